// Grouped GEMMs of the SwiGLU experts (Appendix E) over the E expert buffers.
// Expert-choice gives every expert the same number of rows M = K_tot
// (Section 2.2: each expert processes exactly its capacity), so the group is
// a uniform batch of E problems; ragged per-group capacities only change M.
//
// bf16: one pipelined kernel (gemm_dma_kernel) for every product of the
// forward and backward.  v_mfma_f32_16x16x32_bf16 with fp32 accumulation; a
// 256 x 256 output tile per workgroup (the forward products take 192-, 128- or 64-row
// tiles when those pad short expert buffers less).  K advances 64 at a time through an
// LDS ring of two stages (three for buffers of one short row block) filled straight from
// global memory by buffer_load_dwordx4 ... lds (no VGPR staging, one offset register per
// load).  K-contiguous operands sit in LDS as 128-byte rows with XOR-swizzled 16-byte
// chunks (conflict-free fragment reads); K-major operands (the weight gradients' token-row
// contractions, and the weights in the dA and dX products) stay K-major in LDS and are read
// with the transposing ds_read_b64_tr_b16.  The MFMAs alternate with the next sub-step's
// fragment reads and, once the barrier has freed a stage, with its refill's DMA (with two
// stages half of it then, three quarters where both operands are K-contiguous, the rest in
// the next step), so LDS latency hides behind MFMAs in flight.  The MFMAs take the B
// fragment first, so each lane ends with four consecutive output columns of a row, staged
// through LDS with 16-byte writes for coalesced stores.  Tiles are numbered so that
// consecutive ones share an expert and stay on one XCD.
//
// What bounds it: at 8 x 2048 tokens the chip's power limit and the LDS port, which a
// k-step keeps busy about as long as the matrix cores (64 KiB written, 128 KiB read by
// four waves of 128 x 128 or 192 KiB by eight of 64 x 128).  Hence 16x16x32 MFMAs, which
// move half the accumulator bytes per product of 32x32x16 ones and so let the clock
// rise, buffer loads (with global_load_lds the compiler waits for every LDS read in
// flight, lgkmcnt(0), before each use; with buffer loads it counts), and four waves
// where both operands are K-contiguous, the contraction is long and the tiles are many
// (fwd_eight_waves).  K-major operands keep eight: their fragments
// take twice the reads, and one wave per SIMD leaves those exposed (dW1/dW3 of one
// 2048-token sequence 207 us against 226).  Measured on one card, 64 experts x 2071
// rows, d 2048, h 1024, against 32x32x16 MFMAs, eight waves and global loads: W1/W3 1053
// -> 1008 us, W2 532 -> 533, dA 642 -> 608, dW2 512 -> 450, dX 1015 -> 934, dW1/dW3 1043
// -> 906 (the kernels share one power budget), 1.2 PFLOP/s over the six where a loop of
// nothing but MFMAs sustains 1.6 on such data; the step 5127 -> 4770.  128 x 128 tiles,
// two workgroups a CU, for the weight gradients of few rows are slower (256 rows: dW1/dW3
// 207 -> 252), as are four row blocks per tile group (one sequence's step 870 -> 887).
//
// The products that read the selected tokens' rows (of X, or of the output
// gradient dY) gather them in the operand load: the W1/W3 and dA products per
// row of their K-contiguous A, the dW2 and dW1/dW3 products per k row of their
// K-major operand, so no gathered copy is ever written.
//
// fp32: gemm_f32_kernel, v_mfma_f32_32x32x2_f32 tiles with the same operand
// conventions and gathers.
#include <type_traits>

#include "ec_common.h"
#include "ec_kernels.h"

namespace ec {

namespace {

enum { EPI_STORE = 0, EPI_SWIGLU = 1, EPI_SWIGLU_BWD = 2, EPI_STORE_ADD = 3 };

// Stage tags: every product gets its own kernel symbol, so that traces and
// counters attribute each launch to its stage.
enum { G_W13 = 1, G_W2, G_DA, G_DXE, G_DW2, G_DW13, G_ROUTER_DX, G_ROUTER_DWG,
       G_SH_W13, G_SH_W2, G_SH_DA, G_SH_DXE, G_SH_DW2, G_SH_DW13, G_TC_W13, G_TC_W2 };

struct GemmParams {
  // A operand, element (m, k) of batch e:
  //   K-contiguous:  A[e*a_bs + m*lda + k];   M-contiguous: A[e*a_bs + k*lda + m]
  const void* A;
  long a_bs;
  int lda;
  // K-contiguous A only (may be null): row m of batch e is row
  // a_rows[e*a_rows_bs + r0 + m] of A itself (r0: the batch's first packed row
  // with var_rows, else 0), so the gather of the selected tokens happens in the
  // operand load
  const int32_t* a_rows;
  long a_rows_bs;
  // B operand, element (n, k) of batch e:
  //   K-contiguous:  B[e*b_bs + n*ldb + k]  (SwiGLU: rows of W1 and W3 side by side)
  //   N-contiguous:  B[e*b_bs + k*ldb + n]; rows k >= k_split come from B2
  //                  instead (B2[e*b_bs + (k-k_split)*ldb + n]; the bf16 kernel
  //                  needs k_split to be a multiple of its k-step)
  const void* B;
  const void* B2;
  long b_bs;
  int ldb;
  int k_split;
  int M, N, K;        // per batch (SwiGLU: N = h, the output width)
  int kv_a, kv_b;     // k >= kv reads as zero
  int batches, MT, NT;
  // output (dtype, or fp32 when out_f32): rows m >= c_split go to C2 at m - c_split
  void* C;
  void* C2;
  long c_bs;
  int ldc;
  int c_split;
  // SwiGLU: H1/H3 [batch][M][h] saved (forward, optional) or read (backward)
  void* H1;
  void* H3;
  long h_bs;
  int ldh;
  // K-major operands (used with the OPT_GA / OPT_GB instantiations): row k
  // of batch e's A is row ka_rows[e*k_rows_bs + k] of A itself (kb_rows: of
  // B), so the gather of the selected tokens happens in the operand load when
  // the contraction runs over an expert's rows
  const int32_t* ka_rows;
  const int32_t* kb_rows;
  long k_rows_bs;
  // SwiGLU forward and backward, uniform batches only (may be null): a factor
  // per output row, g = gate[e*gate_bs + m] for row m of batch e.  The forward
  // writes A = g SiLU(H1) H3 (H1, H3 unscaled); the backward takes dA = g (the
  // product) before the SwiGLU backward.
  const float* gate;
  long gate_bs;
  // SwiGLU backward only (may be null): the gate-gradient partials.  For row m
  // of batch e and each column block q of the output (128 columns in the bf16
  // kernel, 64 in the fp32 one), dsp[(e M + m) dsp_ld + q] = sum over the block
  // of dA * A with dA as above and A = SiLU(H1) H3 recomputed from the saved
  // H1, H3 (so the sum over all blocks is g times the gate's gradient when the
  // product is dY W2).
  float* dsp;
  int dsp_ld;
  // Variable rows per batch (token choice): batch e owns rows
  // [var_rows[e], var_rows[e+1]) of A, C and H (row strides lda, ldc, ldh) and
  // tiles [var_tiles[e], var_tiles[e+1]) of the launch; both device arrays of
  // batches + 1 entries, null for a uniform batch of M rows.
  const int* var_rows;
  const int* var_tiles;
};

// Where one output tile sits: batch, first row and column, the batch's rows,
// and the element offsets of the batch in A, C and H.
struct TileCoord {
  int e, m0, n0, M, row0;
  size_t a_off, c_off, h_off;
};

// ------------------------------------------------------------------ bf16 MFMA, pipelined

// 16 bytes per lane from global memory straight into LDS at lds + 16 * lane.
// (The builtin exists only for the device; the host pass must not see it or it
// drops the kernel's launch stub.)
__device__ __forceinline__ void dma16(const void* g, void* lds) {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_global_load_lds(g, lds, 16, 0, 0);
#endif
}

// The same from a buffer resource: a uniform base, a 32-bit byte offset per lane and a
// uniform one, so a K-contiguous operand's loads need one register each and no vector
// arithmetic per step.
// What a base reaches ends below BUF_BYTES: the operands that are read gathered, X and dY,
// are below 2^31 bytes (N 2 d < 2^31 elements), and run_dma checks the others.  Only the
// router's dZ, [N, E rounded up to 64], passes 2^32 bytes: its base is the tile's first row
// (OPT_TILE_BASE; for every product that costs W2 of 128 experts x 1024 rows 420 -> 427 us).
// A load at BUF_PAST reads zero.
constexpr uint32_t BUF_BYTES = 0xffffff80u, BUF_PAST = 0xfffffff0u;
#if defined(__HIP_DEVICE_COMPILE__)
using Rsrc = __amdgpu_buffer_rsrc_t;
__device__ __forceinline__ Rsrc make_rsrc(const void* base) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, BUF_BYTES, 0x00020000);
}
__device__ __forceinline__ void dma16_buf(Rsrc r, uint32_t voff, int soff, void* lds) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)lds, 16,
                                           (int)voff, soff, 0, 0);
}
#else
using Rsrc = int;
__device__ inline Rsrc make_rsrc(const void*) { return 0; }
__device__ inline void dma16_buf(Rsrc, uint32_t, int, void*) {}
#endif

constexpr int vmcnt_imm(int n) { return (n & 15) | (((n >> 4) & 3) << 14) | (7 << 4) | (15 << 8); }

// Each operand is K-contiguous (stored [rows][K]) or K-major (stored
// [K][rows]: the backward's transposed products).  A K-major tile is kept
// K-major in LDS (64 rows of k, its columns contiguous, 16-byte chunks
// XOR-swizzled by k) and read with the transposing ds_read_b64_tr_b16: in each 16-lane group, lane j addresses the
// 4 consecutive columns 4*(j%4).. of row kbase + j/4, and lane i receives
// column i of rows kbase..kbase+3 -- two such reads make one MFMA fragment.
// Rows past the valid K (ragged tail) read as exact zeros.

typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4i16 lds_v4i16;

__device__ __attribute__((aligned(16))) bf16_t g_zero_block[4096];  // stays zero

__device__ __forceinline__ v4i16 ds_read_tr16(const char* __restrict__ p) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)(p));
#else
  return v4i16{0, 0, 0, 0};
#endif
}

template <int R, bool KC, int NT, int KSTEP>
struct DmaOperand {
  static constexpr int BYTES = R * KSTEP * 2;               // per stage
  static constexpr int LOADS = R * KSTEP / 8 / NT;          // 16-byte chunks per thread
  static constexpr int CPR = KC ? KSTEP / 8 : R / 8;        // chunks per LDS row
  static_assert(R * KSTEP / 8 % NT == 0, "whole chunks per thread");
  static_assert(KC || (R % 128 == 0), "K-major tiles are multiples of 128 wide");
};

// Chunk swizzles, for the fragment-read patterns (SQ_LDS_BANK_CONFLICT reads zero in the
// main loops): 128-byte K-contiguous rows, whose 16 (fp32: 32) rows of a fragment read two
// to a 256-byte bank line, and K-major rows (by k), whose four 16-lane groups read 32
// bytes of four rows each.
__device__ __forceinline__ int kc_swz(int row) { return (row >> 1) & 7; }
__device__ __forceinline__ int km_swz(int k) { return ((k & 3) << 2) | ((k >> 2) & 2); }

// Options of an instantiation (bf16; see GemmParams): OPT_GA / OPT_GB gather
// the rows of a K-major A / B through p.ka_rows / p.kb_rows.  OPT_TAILS:
// the last row block and column block take a smaller tile where one holds them.
// OPT_TILE_BASE: an ungathered K-contiguous A of any size, addressed tile by tile.
enum { OPT_GA = 1, OPT_GB = 2, OPT_TAILS = 4, OPT_TILE_BASE = 8 };
template <int BM, int BN, int WGM, int WGN, int KSTEP, int STAGES, bool A_KC, bool B_KC, int EPI,
          bool OUT_F32, int OPT>
__device__ __forceinline__ void gemm_dma_tile(const GemmParams& p, const TileCoord& tc,
                                              char* smem) {
  constexpr int NT = 64 * WGM * WGN;
  constexpr int WM = BM / WGM, WN = BN / WGN;
  constexpr int MB = WM / 16, NB = WN / 16, MH = MB / 2, NH = NB / 2;
  constexpr int KK = KSTEP / 32;
  static_assert(KSTEP == 64 && MB % 2 == 0 && NB % 2 == 0, "two 32-wide sub-steps, whole halves");
  static_assert(STAGES == 2 || (STAGES == 3 && A_KC && B_KC), "ring depth");
  using OA = DmaOperand<BM, A_KC, NT, KSTEP>;
  using OB = DmaOperand<BN, B_KC, NT, KSTEP>;
  constexpr int STAGE_BYTES = OA::BYTES + OB::BYTES;
  constexpr int LOADS = OA::LOADS + OB::LOADS;
  constexpr int SLD = WN + 4;
  static_assert(EPI != EPI_SWIGLU || (NB % 2 == 0), "SwiGLU needs W1 and W3 blocks per wave");
  static_assert(EPI != EPI_SWIGLU || B_KC, "SwiGLU forward has K-contiguous weights");
  const int e = tc.e, M = tc.M, m0 = tc.m0, n0 = tc.n0;

  const int tid = threadIdx.x, lane = tid & 63;
  // the wave index is uniform: read into a scalar register so that the LDS
  // destinations of the DMA loads (M0) are formed with scalar arithmetic
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % WGM, wn = wave / WGM;
  // SwiGLU: the row factors of this wave's rows (lane l holds row wm*WM + 64 t
  // + l), read before the main loop so the epilogue finds them in registers (after it in
  // the forward's eight-wave tiles, which have none to spare)
  constexpr bool GATED = EPI == EPI_SWIGLU || EPI == EPI_SWIGLU_BWD;
  constexpr bool LATE_GATE = EPI == EPI_SWIGLU && NT == 512;
  constexpr int GR = GATED ? (WM + 63) / 64 : 1;
  float gate_r[GR];
  if constexpr (GATED && !LATE_GATE) {
#pragma unroll
    for (int t = 0; t < GR; ++t) {
      const int m = m0 + wm * WM + 64 * t + lane;
      gate_r[t] = (p.gate && m < M) ? p.gate[(size_t)e * p.gate_bs + m] : 1.f;
    }
  }
  const bf16_t* Ab = reinterpret_cast<const bf16_t*>(p.A) + tc.a_off;
  const bf16_t* Bb = reinterpret_cast<const bf16_t*>(p.B) + (size_t)e * p.b_bs;
  const bf16_t* B2b = p.B2 ? reinterpret_cast<const bf16_t*>(p.B2) + (size_t)e * p.b_bs : nullptr;

  // ---- DMA sources.  Load q of a thread fills 1 KiB block (wave*L + q) of
  // the operand's stage area: 64 chunks, lane -> chunk.
  // Every load has one byte offset from a uniform base (see BUF_BYTES), the step's offset
  // being uniform.  K-contiguous: the chunk in its row (clamped: rows past the end produce
  // outputs that are not stored).
  // K-major: the chunk at k-step 0, its column clamped into the operand likewise; rows
  // past the valid K ask for an offset past the buffer, which reads as zero.
  // K-major gathered (OPT_GA / OPT_GB): the chunk's column; the source rows of
  // the next k-step's 64 rows are held one per lane (fetched one step ahead,
  // the first two at set-up so that the prologue waits for no index) and each
  // load takes its row's with a lane read.  Rows past the valid K re-read a
  // valid row: the other operand, never gathered, reads zeros there.
  constexpr bool GA = (OPT & OPT_GA) != 0 && !A_KC, GB = (OPT & OPT_GB) != 0 && !B_KC;
  constexpr bool TILE_BASE = (OPT & OPT_TILE_BASE) != 0;
  static_assert(!TILE_BASE || A_KC, "a K-contiguous A");
  static_assert(((OPT & OPT_GA) == 0 || GA) && ((OPT & OPT_GB) == 0 || GB), "K-major gathers");
  static_assert(!(GA && GB), "one gathered operand: the other zero-fills the ragged K");
  static_assert((!GA || OA::CPR == 32) && (!GB || OB::CPR == 32),
                "a gathered load covers two k rows of 256 columns");
  static_assert(!(GA || GB) || KSTEP == 64, "one source row per lane and k-step");
  uint32_t a_off[OA::LOADS], b_off[OB::LOADS];
  // source row of row k (< K) of a gathered operand; rows past kv re-read the last
  auto k_row = [&](const int32_t* rows, int k, int kv) -> int {
    return rows[(size_t)e * p.k_rows_bs + (k < kv ? k : kv - 1)];
  };
  int a_kidx = 0, a_kidx1 = 0, b_kidx = 0, b_kidx1 = 0;
  if constexpr (GA) {
    if (p.kv_a > 0) {
      a_kidx = k_row(p.ka_rows, lane, p.kv_a);
      a_kidx1 = k_row(p.ka_rows, KSTEP + lane, p.kv_a);
    }
  }
  if constexpr (GB) {
    if (p.kv_b > 0) {
      b_kidx = k_row(p.kb_rows, lane, p.kv_b);
      b_kidx1 = k_row(p.kb_rows, KSTEP + lane, p.kv_b);
    }
  }
  // the source row of k row 2 j + (lane >= 32) of the step (j uniform)
  auto pick_row = [&](int kidx, int j) -> int {
    const int lo = __builtin_amdgcn_readlane(kidx, 2 * j);
    const int hi = __builtin_amdgcn_readlane(kidx, 2 * j + 1);
    return lane < 32 ? lo : hi;
  };
#pragma unroll
  for (int q = 0; q < OA::LOADS; ++q) {
    const int id = (wave * OA::LOADS + q) * 64 + lane;
    if constexpr (A_KC) {
      const int row = id / OA::CPR, lc = (id % OA::CPR) ^ kc_swz(row);
      int r = m0 + row;
      r = r < M ? r : M - 1;
      if (p.a_rows) {
        const int tok = p.a_rows[(size_t)e * p.a_rows_bs + tc.row0 + r];
        a_off[q] = ((uint32_t)tok * (uint32_t)p.lda + lc * 8) * 2;
      } else {
        a_off[q] = ((uint32_t)(TILE_BASE ? r - m0 : r) * (uint32_t)p.lda + lc * 8) * 2;
      }
    } else {
      const int row = id / OA::CPR, lc = (id % OA::CPR) ^ km_swz(row);
      const int col = m0 + lc * 8 < M ? m0 + lc * 8 : (M - 1) & ~7;   // first column of the chunk
      a_off[q] = ((GA ? 0u : (uint32_t)row * (uint32_t)p.lda) + col) * 2;
    }
  }
#pragma unroll
  for (int q = 0; q < OB::LOADS; ++q) {
    const int id = (wave * OB::LOADS + q) * 64 + lane;
    if constexpr (B_KC) {
      const int row = id / OB::CPR, lc = (id % OB::CPR) ^ kc_swz(row);
      int r = n0 + (EPI == EPI_SWIGLU ? row % (BN / 2) : row);
      r = r < p.N ? r : p.N - 1;
      b_off[q] = ((uint32_t)r * (uint32_t)p.ldb + lc * 8) * 2;
    } else {
      const int row = id / OB::CPR, lc = (id % OB::CPR) ^ km_swz(row);
      const int col = n0 + lc * 8 < p.N ? n0 + lc * 8 : (p.N - 1) & ~7;
      b_off[q] = ((GB ? 0u : (uint32_t)row * (uint32_t)p.ldb) + col) * 2;
    }
  }
  // a SwiGLU wave's rows all lie in W1 or all in W3
  static_assert(EPI != EPI_SWIGLU || (BN / 2) % (OB::LOADS * 8) == 0, "one weight per wave");
  const bf16_t* const a_base = TILE_BASE ? Ab + (size_t)m0 * p.lda : Ab;
  const Rsrc a_rsrc = make_rsrc((A_KC ? p.a_rows != nullptr : GA) ? p.A : (const void*)a_base);
  const Rsrc b_rsrc = make_rsrc(EPI == EPI_SWIGLU && wave * OB::LOADS * 8 >= BN / 2 ? B2b : Bb);
  // Issues k-step kt; the calls come with kt = 0, 1, 2, ... in order.
  // Loads [lo, hi) of k-step kt (A's loads first, then B's); each load of a
  // k-step is issued exactly once and the k-steps in order.
  // K-major rows past the valid K read zero (see BUF_PAST); with full_step (a step
  // known to lie below both kv) the per-load check is skipped.  first: k-step
  // 0 (its successor's source rows are already at hand).
  auto issue_part = [&](int kt, int stage, int lo, int hi, auto full_step, auto first) {
    constexpr bool FULL = decltype(full_step)::value;
    constexpr bool FIRST = decltype(first)::value;
    char* base = smem + stage * STAGE_BYTES;
    // the loads of a K-major operand: rows past the valid K ask for an offset past the
    // buffer, which reads as zero
    auto km_load = [&](Rsrc r, uint32_t off, int row, int k0, int kv, uint32_t ld, void* lds) {
      const uint32_t step = (uint32_t)k0 * ld * 2u;
      if constexpr (FULL) dma16_buf(r, off, (int)step, lds);
      else dma16_buf(r, k0 + row < kv ? off + step : BUF_PAST, 0, lds);
    };
#pragma unroll
    for (int q = 0; q < OA::LOADS; ++q) {
      if (q < lo || q >= hi) continue;
      char* lds = base + (wave * OA::LOADS + q) * 1024;
      if constexpr (A_KC)
        dma16_buf(a_rsrc, a_off[q], kt * KSTEP * 2, lds);
      else if constexpr (GA)
        dma16_buf(a_rsrc, a_off[q] + (uint32_t)pick_row(a_kidx, wave * OA::LOADS + q) * (uint32_t)p.lda * 2u, 0, lds);
      else
        km_load(a_rsrc, a_off[q], ((wave * OA::LOADS + q) * 64 + lane) / OA::CPR, kt * KSTEP, p.kv_a, p.lda, lds);
    }
    // K-major B split at k_split (a multiple of the k-step): steps from there on read B2
    // (selected, not branched to: a branch would split the interleaved group)
    const bool second = !B_KC && !GB && kt * KSTEP >= p.k_split;
    const int bk0 = kt * KSTEP - (second ? p.k_split : 0), bkv = p.kv_b - (second ? p.k_split : 0);
    const Rsrc bk_rsrc = make_rsrc(second ? B2b : Bb);
    if constexpr (GA) {   // every A load of step kt has gone out: rows of step kt + 1
      if (lo < OA::LOADS && hi >= OA::LOADS)
        a_kidx = FIRST ? a_kidx1 : k_row(p.ka_rows, (kt + 1) * KSTEP + lane, p.kv_a);
    }
#pragma unroll
    for (int q = 0; q < OB::LOADS; ++q) {
      if (OA::LOADS + q < lo || OA::LOADS + q >= hi) continue;
      char* lds = base + OA::BYTES + (wave * OB::LOADS + q) * 1024;
      if constexpr (B_KC) {
        dma16_buf(b_rsrc, b_off[q], kt * KSTEP * 2, lds);
      } else if constexpr (GB) {
        dma16_buf(b_rsrc, b_off[q] + (uint32_t)pick_row(b_kidx, wave * OB::LOADS + q) * (uint32_t)p.ldb * 2u, 0, lds);
      } else {
        const int row = ((wave * OB::LOADS + q) * 64 + lane) / OB::CPR;
        km_load(bk_rsrc, b_off[q], row, bk0, bkv, p.ldb, lds);
      }
    }
    if constexpr (GB) {
      if (hi >= OA::LOADS + OB::LOADS)
        b_kidx = FIRST ? b_kidx1 : k_row(p.kb_rows, (kt + 1) * KSTEP + lane, p.kv_b);
    }
  };
  auto issue = [&](int kt, int stage, auto first) {
    issue_part(kt, stage, 0, OA::LOADS + OB::LOADS, std::false_type{}, first);
  };

  auto b_lds_col = [&](int ni) -> int {
    if constexpr (EPI == EPI_SWIGLU) {
      constexpr int HWN = BN / 2 / WGN;
      return (ni < NH) ? wn * HWN + ni * 16 : BN / 2 + wn * HWN + (ni - NH) * 16;
    } else {
      return wn * WN + ni * 16;
    }
  };
  // Fragment addressing (16 rows or columns x 32 k).  K-contiguous: lane l reads row
  // base + l % 16 of the tile, base a multiple of 16 (uniform over the wave), so the
  // row's chunk swizzle is a per-lane value.  K-major:
  // lane l reads 4 columns from column base + lp of k rows km_k and km_k + 4 (of each
  // 32-wide sub-step); the swizzled chunk is base / 8 XOR a per-lane value.  Nothing
  // per fragment is held in registers.
  const int g16 = lane >> 4, l15 = lane & 15;
  const int km_k = 8 * g16 + (l15 >> 2);            // k row (within a sub-step) of a K-major read
  const int km_lp = 4 * (l15 & 3);
  const int km_inner = (km_lp & 7) * 2;             // byte offset inside the chunk
  const int km_u = (km_lp >> 3) | km_swz(km_k);     // chunk bits from the lane and the k swizzle

  bf16x8 af[MB], bfr[NB];
  auto kc_frag = [&](const char* tile, int base, int kk) -> bf16x8 {
    const int lc = kk * 4 + g16;
    return __builtin_bit_cast(
        bf16x8, *reinterpret_cast<const u32x4*>(tile + (base + l15) * (KSTEP * 2) +
                                                ((lc ^ (l15 >> 1)) << 4)));
  };
  auto km_frag = [&](const char* tile, int rowbytes, int base, int kk) -> bf16x8 {
    const char* p0 = tile + (kk * 32 + km_k) * rowbytes + (((base >> 3) ^ km_u) << 4) + km_inner;
    const v4i16 lo = ds_read_tr16(p0);
    const v4i16 hi = ds_read_tr16(p0 + 4 * rowbytes);
    const v4i16 both[2] = {lo, hi};
    return __builtin_bit_cast(bf16x8, both);
  };
  // half of the A (B) fragments of sub-step kk
  auto load_a = [&](int stage, int kk, int half) {
    const char* sa = smem + stage * STAGE_BYTES;
#pragma unroll
    for (int i = 0; i < MH; ++i) {
      const int mi = half * MH + i;
      if constexpr (A_KC) af[mi] = kc_frag(sa, wm * WM + mi * 16, kk);
      else af[mi] = km_frag(sa, BM * 2, wm * WM + mi * 16, kk);
    }
  };
  auto load_b = [&](int stage, int kk, int half) {
    const char* sb = smem + stage * STAGE_BYTES + OA::BYTES;
#pragma unroll
    for (int i = 0; i < NH; ++i) {
      const int ni = half * NH + i;
      if constexpr (B_KC) bfr[ni] = kc_frag(sb, b_lds_col(ni), kk);
      else bfr[ni] = km_frag(sb, BN * 2, b_lds_col(ni), kk);
    }
  };

  f32x4 acc[MB][NB];
#pragma unroll
  for (int mi = 0; mi < MB; ++mi)
#pragma unroll
    for (int ni = 0; ni < NB; ++ni) acc[mi][ni] = f32x4{0.f, 0.f, 0.f, 0.f};

  constexpr bool EARLY = A_KC && B_KC;   // read order, see below
  // Ring: steps 0..STAGES-1 are issued up front; the end of step kt refills
  // stage kt % STAGES with step kt + STAGES once every wave has read it.  When
  // waiting for step j, the steps issued after it number min(STAGES-1, KT-1-j)
  // for j = 0 and min(STAGES-2, KT-1-j) afterwards (vmcnt counts this wave's
  // outstanding loads, which complete in order).
  auto wait_younger = [&](int younger) {
    if (STAGES > 2 && younger == 2) __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * LOADS));
    else if (younger >= 1) __builtin_amdgcn_s_waitcnt(vmcnt_imm(LOADS));
    else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
  };
  static_assert((STAGES - 1) * LOADS <= 63, "vmcnt range");
  const int KT = (p.K + KSTEP - 1) / KSTEP;
  if (KT > 0) issue(0, 0, std::true_type{});
#pragma unroll
  for (int s2 = 1; s2 < STAGES; ++s2)
    if (s2 < KT) issue(s2, s2, std::false_type{});
  if (KT > 0) {
    wait_younger(KT - 1 < STAGES - 1 ? KT - 1 : STAGES - 1);
    __builtin_amdgcn_s_barrier();
    load_a(0, 0, 0);
    load_b(0, 0, 0);
    if constexpr (EARLY) load_b(0, 0, 1);
  }
  // a quadrant: half of the A blocks times half of the B blocks.  B fragment first: the
  // 16 x 16 block comes out transposed, each lane holding four consecutive output
  // columns of one row (16-byte staging writes in the epilogue)
  constexpr int NMQ = MH * NH;
  auto quad = [&](int ha, int hb) {
#pragma unroll
    for (int j = 0; j < NH; ++j)
#pragma unroll
      for (int i = 0; i < MH; ++i) {
        const int mi = ha * MH + i, ni = hb * NH + j;
        acc[mi][ni] =
            __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[ni], af[mi], acc[mi][ni], 0, 0, 0);
      }
  };

  // A 32-wide sub-step runs as four quadrants, A0 Bx, A0 By, A1 By, A1 Bx (x alternating
  // between sub-steps), so that half operands die one by one and one set of fragment
  // registers is enough.  A1 is read during the first quadrant, the next sub-step's A0
  // during the third.  EARLY (both operands K-contiguous): its By and Bx are read during
  // the third and fourth, each fragment after the last MFMA of the one it replaces, a
  // whole quadrant before their use; K-major operands' twice as many reads are
  // spread instead, By over the fourth and Bx over the next first (reading them early
  // costs dW2 12% and dA 6%).  In a stage's last sub-step the waits and the barrier
  // stand between the second and third quadrants (the stage's last reads are then done),
  // and the refill's DMA follows in the other two.  Steps with and without a refill (or
  // a refill's second half) run in separate straight-line segments, so that no branch
  // splits an interleaved group.
  constexpr int RA = MH * (A_KC ? 1 : 2), RB = NH * (B_KC ? 1 : 2);   // read instructions
  // A stage's refill is issued in two parts: DMA_HEAD loads after the barrier that frees
  // the stage, the rest in the next step's first sub-step (two stages only: the wait at
  // every step end is then for all outstanding loads).  K-major fragment reads leave
  // room for half of it after the barrier; K-contiguous ones, half as many, for three
  // quarters (against half: one 2048-token sequence's forward 357 -> 349 us, 4 x 4096
  // tokens 1250 -> 1244, a step of 8 x 2048 4795 -> 4770; all of it: 345, 1280, 4828;
  // K-major with three quarters: dW2 450 -> 473, dW1/dW3 897 -> 923).
  constexpr bool SPLIT_DMA = STAGES == 2;
  constexpr int DMA_HEAD = !SPLIT_DMA ? LOADS : (EARLY ? LOADS * 3 / 4 : LOADS / 2);
  constexpr int DMA_Q3 = DMA_HEAD / 2;
  // orders a quadrant: after each MFMA its share of the LDS reads and DMA loads
  auto order = [&](auto reads, auto dmas) {
    constexpr int RD = decltype(reads)::value, DM = decltype(dmas)::value;
#pragma unroll
    for (int q = 0; q < NMQ; ++q) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                     // MFMA
      if constexpr (DM > 0) __builtin_amdgcn_sched_group_barrier(0x010, (DM + NMQ - 1) / NMQ, 0);   // DMA
      if constexpr (RD > 0) __builtin_amdgcn_sched_group_barrier(0x100, (RD + NMQ - 1) / NMQ, 0);   // LDS read
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto kstep = [&](int kt, auto refill, auto tail_part, auto full_refill) {
    constexpr bool RF = decltype(refill)::value;
    constexpr bool TAIL = SPLIT_DMA && decltype(tail_part)::value;
    const int stage = kt % STAGES;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      const int x = kk & 1;
      const bool last = kk == KK - 1;
      using RB_ = std::integral_constant<int, RB>;
      using NONE_ = std::integral_constant<int, 0>;
      const int nstage = last ? (kt + 1) % STAGES : stage, nkk = last ? 0 : kk + 1;
      quad(0, x);
      if constexpr (!EARLY) load_b(stage, kk, x ^ 1);
      load_a(stage, kk, 1);
      order(std::integral_constant<int, EARLY ? RA : RA + RB>{}, NONE_{});
      quad(0, x ^ 1);
      if (!last) {
        // TAIL: the second part of the previous step's refill
        if constexpr (TAIL) {
          issue_part(kt - 1 + STAGES, (kt - 1) % STAGES, DMA_HEAD, LOADS, full_refill,
                     std::false_type{});
          order(NONE_{}, std::integral_constant<int, LOADS - DMA_HEAD>{});
        } else {
          __builtin_amdgcn_sched_barrier(0);
        }
      } else {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0): this wave's reads are done
        if (kt + 1 < KT) wait_younger(KT - 2 - kt < STAGES - 2 ? KT - 2 - kt : STAGES - 2);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
      }
      // after the final step these read a stale stage, harmlessly
      quad(1, x ^ 1);
      if constexpr (RF)
        if (last) issue_part(kt + STAGES, stage, 0, DMA_Q3, full_refill, std::false_type{});
      load_a(nstage, nkk, 0);
      if constexpr (EARLY) load_b(nstage, nkk, x ^ 1);
      if (RF && last) order(std::integral_constant<int, EARLY ? RA + RB : RA>{}, std::integral_constant<int, DMA_Q3>{});
      else order(std::integral_constant<int, EARLY ? RA + RB : RA>{}, NONE_{});
      quad(1, x);
      if constexpr (RF)
        if (last) issue_part(kt + STAGES, stage, DMA_Q3, DMA_HEAD, full_refill, std::false_type{});
      load_b(nstage, nkk, EARLY ? x : x ^ 1);
      if (RF && last) order(RB_{}, std::integral_constant<int, DMA_HEAD - DMA_Q3>{});
      else order(RB_{}, NONE_{});
    }
  };
  // Straight-line segments, so that no branch splits an interleaved group:
  // step 0 (refill, no tail), steps that refill and finish the previous
  // refill, the step that only finishes it, then the last steps.
  {
    using T_ = std::true_type;
    using F_ = std::false_type;
    int kt = 0;
    if constexpr (SPLIT_DMA) {
      // refills of the steps below KT - 1 skip the K-major row check when
      // every such step lies below both kv (the usual case: only the last step
      // is ragged), and so does the second part of such a refill in the next step
      const bool full_ok = p.kv_a >= (KT - 1) * KSTEP && p.kv_b >= (KT - 1) * KSTEP;
      const int n_full = full_ok ? KT - STAGES - 1 : 0;
      if (KT > STAGES) {
        kstep(0, T_{}, F_{}, F_{});
        if constexpr (!A_KC || !B_KC)
          for (kt = 1; kt < n_full; ++kt) kstep(kt, T_{}, T_{}, T_{});
        for (kt = kt > 1 ? kt : 1; kt + STAGES < KT; ++kt) kstep(kt, T_{}, T_{}, F_{});
        kstep(kt, F_{}, T_{}, F_{});
        ++kt;
      }
    } else {
      for (; kt + STAGES < KT; ++kt) kstep(kt, T_{}, F_{}, F_{});
    }
    for (; kt < KT; ++kt) kstep(kt, F_{}, F_{}, F_{});
  }
  if constexpr (LATE_GATE) {
#pragma unroll
    for (int t = 0; t < GR; ++t) {
      const int m = m0 + wm * WM + 64 * t + lane;
      gate_r[t] = (p.gate && m < M) ? p.gate[(size_t)e * p.gate_bs + m] : 1.f;
    }
  }
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
  __syncthreads();

  // ---- epilogue: stage 32-row slices of the wave tile through LDS ----
  // The accumulators of a slice go to LDS (fp32, row-major); then every lane
  // reads its 16-byte output chunks back in batches of EQ with no branch
  // between the reads (their LDS addresses always lie inside the slice), and
  // only then converts and stores the chunks that fall inside the matrix.
  float* stage_f = reinterpret_cast<float*>(smem) + wave * 32 * SLD;
  constexpr int HW = WN / 2;                                    // SwiGLU: outputs per row
  constexpr int CPR = (EPI == EPI_SWIGLU) ? HW / 8 : WN / 8;    // chunks per slice row
  constexpr int NCH = 32 * CPR;                                 // chunks per slice
  constexpr int NQ = (NCH + 63) / 64;                           // chunks per lane
  constexpr int EQ = (EPI == EPI_SWIGLU_BWD && NQ > 4) ? 4 : NQ;  // chunks per batch
  static_assert(NQ % EQ == 0, "whole batches");
  static_assert(EPI != EPI_SWIGLU_BWD || (CPR == 16 && NCH % 64 == 0),
                "the chunks of a 128-column block of a row sit in one 16-lane DPP row");
  // SwiGLU backward: the H1/H3 chunks of slice 0 are loaded before it is
  // staged; those of slice mi + 1 batch by batch as slice mi's batches finish
  // with theirs, so their latency overlaps slice mi's work (rows or columns past
  // the matrix read element 0 and are not stored).
  constexpr int HQ = (EPI == EPI_SWIGLU_BWD) ? NQ : 1;
  u32x4 h1raw[2][HQ], h3raw[2][HQ];
  auto load_h = [&](int mi, int q) {
    if constexpr (EPI == EPI_SWIGLU_BWD) {
      const int mb = m0 + wm * WM + mi * 32;
      const int c = lane + q * 64;
      const int m = mb + c / CPR, n = n0 + wn * WN + (c % CPR) * 8;
      const size_t ho = (m < M && n < p.N) ? tc.h_off + (size_t)m * p.ldh + n : 0;
      // read once: streaming loads
      h1raw[mi & 1][q] =
          __builtin_nontemporal_load(reinterpret_cast<const u32x4*>((const bf16_t*)p.H1 + ho));
      h3raw[mi & 1][q] =
          __builtin_nontemporal_load(reinterpret_cast<const u32x4*>((const bf16_t*)p.H3 + ho));
    }
  };
  if constexpr (EPI == EPI_SWIGLU_BWD) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) load_h(0, q);
  }
#pragma unroll
  for (int mi = 0; mi < WM / 32; ++mi) {
    const int mbase = m0 + wm * WM + mi * 32;
    // acc[2 mi + b][ni][i] is row 16 b + lane % 16 of the slice, column
    // 16 ni + 4 (lane / 16) + i
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int ni = 0; ni < NB; ++ni)
        *reinterpret_cast<f32x4*>(&stage_f[(b * 16 + l15) * SLD + ni * 16 + g16 * 4]) =
            acc[2 * mi + b][ni];
    __builtin_amdgcn_s_waitcnt(0xc07f);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int q0 = 0; q0 < NQ; q0 += EQ) {
      // chunk q of this lane: slice row c / CPR, columns (c % CPR) * 8 .. + 7
      float v[EQ][8], v3[EPI == EPI_SWIGLU ? EQ : 1][8];
#pragma unroll
      for (int e = 0; e < EQ; ++e) {
        int c = lane + (q0 + e) * 64;
        c = c < NCH ? c : NCH - 1;
        const float* src = stage_f + (c / CPR) * SLD + (c % CPR) * 8;
#pragma unroll
        for (int u = 0; u < 8; ++u) v[e][u] = src[u];
        if constexpr (EPI == EPI_SWIGLU) {
#pragma unroll
          for (int u = 0; u < 8; ++u) v3[e][u] = src[HW + u];
        }
      }
      float dots[EPI == EPI_SWIGLU_BWD ? EQ : 1];
#pragma unroll
      for (int e = 0; e < (EPI == EPI_SWIGLU_BWD ? EQ : 1); ++e) dots[e] = 0.f;
#pragma unroll
      for (int e = 0; e < EQ; ++e) {
        const int q = q0 + e;
        const int c = lane + q * 64;
        const int m = mbase + c / CPR;
        const int n = n0 + wn * (EPI == EPI_SWIGLU ? HW : WN) + (c % CPR) * 8;
        // the row factor, from the lane that holds it (every lane takes part)
        float g = 1.f;
        if constexpr (GATED) {
          const int rr = (c < NCH ? c : NCH - 1) / CPR;   // row within the slice
          g = __shfl(gate_r[(mi * 32) / 64], (mi * 32) % 64 + rr, 64);
        }
        if (c >= NCH || m >= M || n >= p.N) continue;
        if constexpr (EPI == EPI_STORE || EPI == EPI_STORE_ADD) {
          const bool second = m >= p.c_split;
          const int mm = second ? m - p.c_split : m;
          const size_t off = tc.c_off + (size_t)mm * p.ldc + n;
          if constexpr (OUT_F32) {
            float* dst = (float*)(second ? p.C2 : p.C) + off;
            if constexpr (EPI == EPI_STORE_ADD) {
              float old[8];
              Elem<float>::load8(dst, old);
#pragma unroll
              for (int u = 0; u < 8; ++u) v[e][u] += old[u];
            }
            Elem<float>::store8(dst, v[e]);
          } else {
            bf16_t* dst = (bf16_t*)(second ? p.C2 : p.C) + off;
            if constexpr (EPI == EPI_STORE_ADD) {
              float old[8];
              Elem<bf16_t>::load8(dst, old);
#pragma unroll
              for (int u = 0; u < 8; ++u) v[e][u] += old[u];
            }
            Elem<bf16_t>::store8(dst, v[e]);
          }
        } else if constexpr (EPI == EPI_SWIGLU) {
          float a[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) a[u] = silu_f(v[e][u]) * v3[e][u] * g;
          Elem<bf16_t>::store8((bf16_t*)p.C + tc.c_off + (size_t)m * p.ldc + n, a);
          if (p.H1) {
            const size_t ho = tc.h_off + (size_t)m * p.ldh + n;
            Elem<bf16_t>::store8((bf16_t*)p.H1 + ho, v[e]);
            Elem<bf16_t>::store8((bf16_t*)p.H3 + ho, v3[e]);
          }
        } else {  // EPI_SWIGLU_BWD
          float d1[8], d3[8];
          float dot = 0.f;
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            const uint32_t w1 = h1raw[mi & 1][q][u >> 1], w3 = h3raw[mi & 1][q][u >> 1];
            const float h1 = bf16_to_f32((u & 1) ? (w1 >> 16) : (w1 & 0xffffu));
            const float h3 = bf16_to_f32((u & 1) ? (w3 >> 16) : (w3 & 0xffffu));
            const float da = v[e][u] * g;
            const float sg = sigmoid_f(h1);
            const float s1 = h1 * sg;   // SiLU(h1)
            d3[u] = da * s1;
            d1[u] = da * h3 * sg * (1.0f + h1 * (1.0f - sg));
            dot = fmaf(da, s1 * h3, dot);
          }
          dots[e] = dot;
          const size_t off = tc.c_off + (size_t)m * p.ldc + n;
          Elem<bf16_t>::store8((bf16_t*)p.C + off, d1);
          Elem<bf16_t>::store8((bf16_t*)p.C2 + off, d3);
        }
      }
      if constexpr (EPI == EPI_SWIGLU_BWD) {
        // gate-gradient partials: the 16 lanes of a DPP row hold the chunks of
        // one row's 128-column block (columns past N hold clamped duplicates
        // and count as zero)
        if (p.dsp) {
#pragma unroll
          for (int e = 0; e < EQ; ++e) {
            const int c = lane + (q0 + e) * 64;
            const int m = mbase + c / CPR;
            const int n = n0 + wn * WN + (c % CPR) * 8;
            const float t = row16_sum(n < p.N ? dots[e] : 0.f);
            if ((lane & 15) == 0 && m < M && n < p.N)
              p.dsp[((size_t)tc.e * p.M + m) * p.dsp_ld + (n >> 7)] = t;
          }
        }
        if (mi + 1 < WM / 32) {
#pragma unroll
          for (int e = 0; e < EQ; ++e) load_h(mi + 1, q0 + e);
        }
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// smem bytes of gemm_dma_tile's configuration
template <int BM, int BN, int WGM, int WGN, int KSTEP, int STAGES, bool A_KC, bool B_KC>
constexpr int dma_smem_bytes() {
  constexpr int NT = 64 * WGM * WGN;
  constexpr int STAGE_BYTES = (BM + BN) * KSTEP * 2;
  constexpr int STAGE_EPI = NT / 64 * 32 * (BN / WGN + 4) * 4;
  return STAGES * STAGE_BYTES > STAGE_EPI ? STAGES * STAGE_BYTES : STAGE_EPI;
}

// One output tile per workgroup; consecutive tile ids (same expert) are kept
// on one XCD so that its L2 serves their shared A rows and B columns.
template <int BM, int BN, int WGM, int WGN, int KSTEP, int STAGES, bool A_KC, bool B_KC, int EPI,
          bool OUT_F32, int TAG, int OPT>
__global__ __launch_bounds__(64 * WGM * WGN, 1) void gemm_dma_kernel(GemmParams p) {
  __shared__ __attribute__((aligned(1024)))
  char smem[dma_smem_bytes<BM, BN, WGM, WGN, KSTEP, STAGES, A_KC, B_KC>()];
  TileCoord tc;
  int rem, MT;
  if (p.var_rows) {
    // the tile count is known only on the device: the grid is an upper bound,
    // and the XCD-contiguous numbering uses the actual count
    const int total = p.var_tiles[p.batches];
    const int per_xcd = (total + 7) >> 3;
    const int j = blockIdx.x >> 3;
    if (j >= per_xcd) return;
    const int t = (blockIdx.x & 7) * per_xcd + j;
    if (t >= total) return;
    int lo = 0, hi = p.batches;          // var_tiles[lo] <= t < var_tiles[hi]
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (p.var_tiles[mid] <= t) lo = mid; else hi = mid;
    }
    const int row0 = p.var_rows[lo];
    tc.e = lo;
    tc.row0 = row0;
    tc.M = p.var_rows[lo + 1] - row0;
    MT = (tc.M + BM - 1) / BM;
    rem = t - p.var_tiles[lo];
    tc.a_off = (size_t)row0 * p.lda;
    tc.c_off = (size_t)row0 * p.ldc;
    tc.h_off = (size_t)row0 * p.ldh;
  } else {
    const int t = xcd_tile_id(blockIdx.x, gridDim.x);
    if (t >= p.batches * p.MT * p.NT) return;
    const int per_b = p.MT * p.NT;
    tc.e = t / per_b;
    tc.row0 = 0;
    tc.M = p.M;
    MT = p.MT;
    rem = t - tc.e * per_b;
    tc.a_off = (size_t)tc.e * p.a_bs;
    tc.c_off = (size_t)tc.e * p.c_bs;
    tc.h_off = (size_t)tc.e * p.h_bs;
  }
  // Tiles go in groups of GROUP_M row blocks, row block fastest inside a
  // group: the workgroups resident on one XCD then share few A row blocks and
  // B column blocks at a time (fewer L2 misses than a full column of row blocks).
  constexpr int GROUP_M = 3;
  const int grp = rem / (GROUP_M * p.NT), in_grp = rem - grp * GROUP_M * p.NT;
  const int gm = (MT - grp * GROUP_M) < GROUP_M ? (MT - grp * GROUP_M) : GROUP_M;
  tc.m0 = (grp * GROUP_M + in_grp % gm) * BM;
  tc.n0 = in_grp / gm * (EPI == EPI_SWIGLU ? BN / 2 : BN);
  // Short last blocks: a whole 256 x 256 tile for 23 rows (64 experts x 2071 rows) is
  // a ninth of the product spent on padding.  The smaller tiles hold the same sums, so
  // the results are the same bits; measured there W1/W3 1.10 -> 1.07 ms, W2 0.57 -> 0.54,
  // dX 1.08 -> 1.04, and a step of 40 experts x 681 rows, d 1472, h 832 893 -> 869 us
  // (less than the share of padding: under the power limit padding is cheap).
  if constexpr ((OPT & OPT_TAILS) != 0) {
    constexpr int NW = WGM * WGN;
    static_assert(BM == 256 && BN == 256 && (NW == 4 || NW == 8), "tails of 256 x 256 tiles");
    const int left = tc.M - tc.m0;
    // a K-major operand's tiles are multiples of 128 wide (256 when gathered), and a
    // SwiGLU backward wave covers 128 columns
    constexpr bool ROWS = (OPT & OPT_GA) == 0, COLS = (OPT & OPT_GB) == 0;
    constexpr bool BWD = EPI == EPI_SWIGLU_BWD, FINE = ROWS && A_KC && !BWD;
    if constexpr (FINE) {
      if (left <= 64) {
        gemm_dma_tile<64, 256, NW / 4, 4, KSTEP, STAGES, A_KC, B_KC, EPI, OUT_F32, OPT>(p, tc, smem);
        return;
      }
    }
    if constexpr (ROWS) {
      if (left <= 128) {
        constexpr int GM = BWD ? NW / 2 : 2;
        gemm_dma_tile<128, 256, GM, NW / GM, KSTEP, STAGES, A_KC, B_KC, EPI, OUT_F32, OPT>(p, tc, smem);
        return;
      }
    }
    if constexpr (FINE && B_KC) {   // (a K-major B beside three row blocks would spill)
      if (left <= 192) {
        gemm_dma_tile<192, 256, 2, NW / 2, KSTEP, STAGES, A_KC, B_KC, EPI, OUT_F32, OPT>(p, tc, smem);
        return;
      }
    }
    if constexpr (COLS) {
      if (p.N - tc.n0 <= (EPI == EPI_SWIGLU ? 64 : 128)) {
        constexpr int GN = BWD ? 1 : 2;
        gemm_dma_tile<256, 128, NW / GN, GN, KSTEP, STAGES, A_KC, B_KC, EPI, OUT_F32, OPT>(p, tc, smem);
        return;
      }
    }
  }
  gemm_dma_tile<BM, BN, WGM, WGN, KSTEP, STAGES, A_KC, B_KC, EPI, OUT_F32, OPT>(p, tc, smem);
}

// The operands that a tile addresses from their batch's start are within BUF_BYTES (a
// batch of variable rows has no more of them than p.M).
template <bool A_KC, bool B_KC, int OPT>
bool operands_in_reach(const GemmParams& p) {
  const bool a_far = (OPT & OPT_GA) || (A_KC && p.a_rows) || (OPT & OPT_TILE_BASE);
  const long a = a_far ? 0 : 2L * (A_KC ? p.M : p.kv_a) * p.lda;
  const long b = (OPT & OPT_GB) ? 0 : 2L * (B_KC ? p.N : p.kv_b) * p.ldb;
  return a <= (long)BUF_BYTES && b <= (long)BUF_BYTES;
}

// OPT: the options of the instantiation; the pointers of each option must be
// set exactly when it is.
template <int BM, int BN, int WGM, int WGN, int KSTEP, int STAGES, bool A_KC, bool B_KC, int EPI,
          bool OUT_F32, int TAG, int OPT = 0>
hipError_t run_dma(GemmParams p, hipStream_t st) {
  if (((OPT & OPT_GA) != 0) != (p.ka_rows != nullptr) ||
      ((OPT & OPT_GB) != 0) != (p.kb_rows != nullptr))
    return hipErrorInvalidValue;
  if (!operands_in_reach<A_KC, B_KC, OPT>(p)) return hipErrorInvalidValue;
  p.MT = (p.M + BM - 1) / BM;
  p.NT = (EPI == EPI_SWIGLU) ? (p.N + BN / 2 - 1) / (BN / 2) : (p.N + BN - 1) / BN;
  const long ntile = (long)p.batches * p.MT * p.NT;
  if (ntile == 0) return hipSuccess;
  const long grid = (ntile + 7) / 8 * 8;
  if constexpr ((OPT & OPT_TAILS) != 0) {
    // without a short last block the kernel that knows none is the faster by a percent
    const int mr = p.M % BM, nr = (EPI == EPI_SWIGLU ? 2 * p.N : p.N) % BN;
    const bool mtail = mr > 0 && mr <= (A_KC && B_KC ? 192 : 128);
    if (!((mtail && !(OPT & OPT_GA)) || (nr > 0 && nr <= 128 && !(OPT & OPT_GB))))
      return run_dma<BM, BN, WGM, WGN, KSTEP, STAGES, A_KC, B_KC, EPI, OUT_F32, TAG,
                     OPT & ~OPT_TAILS>(p, st);
  }
  gemm_dma_kernel<BM, BN, WGM, WGN, KSTEP, STAGES, A_KC, B_KC, EPI, OUT_F32, TAG, OPT>
      <<<dim3((unsigned)grid), 64 * WGM * WGN, 0, st>>>(p);
  return hipGetLastError();
}

// Variable rows per batch (p.var_rows / p.var_tiles on the device): the grid
// covers max_rows rows in total plus one partial row block per batch.
template <int BM, int BN, int WGM, int WGN, int KSTEP, int STAGES, bool A_KC, bool B_KC, int EPI,
          bool OUT_F32, int TAG, int OPT>
hipError_t run_dma_var(GemmParams p, long max_rows, hipStream_t st) {
  if (!operands_in_reach<A_KC, B_KC, OPT>(p)) return hipErrorInvalidValue;
  p.MT = 0;
  p.NT = (EPI == EPI_SWIGLU) ? (p.N + BN / 2 - 1) / (BN / 2) : (p.N + BN - 1) / BN;
  const long ntile = ((max_rows + BM - 1) / BM + p.batches) * p.NT;
  if (ntile == 0 || p.batches == 0) return hipSuccess;
  const long grid = (ntile + 7) / 8 * 8;
  gemm_dma_kernel<BM, BN, WGM, WGN, KSTEP, STAGES, A_KC, B_KC, EPI, OUT_F32, TAG, OPT>
      <<<dim3((unsigned)grid), 64 * WGM * WGN, 0, st>>>(p);
  return hipGetLastError();
}

// Row blocks of the forward expert products: 192 when they pad the expert buffers to less
// than 6/7 of what whole blocks of 256 would (one 2048-token sequence at c(t) = 12 - 8t has
// 373 rows per expert: 384 instead of 512).  Equal blocks are the faster also where blocks
// of 256 with a short last one compute no more rows, or fewer, as every round of tiles then
// takes as long as its fullest: two blocks of 192 against 256 and a short one, 257 rows
// W2 of 64 experts, d 2048, h 1024 106 and 117 us, of 8 experts 21.5 and 26.3, W1/W3 193
// and 191, 34.3 and 40.4; 384 rows 115 and 121, 22.0 and 26.8, 198 and 197, 35.0 and 39.5;
// three, 513 rows 168 and 166, 22.8 and 27.9, 279 and 286, 36.3 and 45.5.  (W1/W3 of many
// experts is the exception, by up to 4%: 40 experts, d 1472, h 832, 300 rows 98 and 95.)
// Every choice keeps an expert's row blocks side by side on one XCD, so its weights are
// fetched once.
// Buffers of at most 128 or 64 rows (that sequence at t = 1; a short sequence) are one
// row block that only streams the weights: what counts is loads in flight, so three
// stages instead of two, and for 64 rows 64 x 128 tiles, two workgroups a CU.  Measured
// with 64 experts, d 2048, h 1024 (805 MB of weights; 128-row tiles of two stages and
// eight waves before): 30 rows W1/W3 131 -> 108 us (4.9 TB/s) and W2 57 -> 50, 128 rows 134
// -> 128 and 65 -> 57.  Two stages are slower at 128 rows (64 experts 132 and 61); 64-wide
// columns, four stages and 32-row tiles were, with 32x32x16 MFMAs.
int fwd_block_rows(int M) {
  if (M <= 64) return 64;
  if (M <= 128) return 128;
  const long r256 = (M + 255) / 256 * 256L, r192 = (M + 191) / 192 * 192L;
  return r192 * 7 < r256 * 6 ? 192 : 256;
}

// Waves of the forward products' 256- and 192-row tiles: four of 128 x 128 read a third
// less LDS, draw less power and store wider rows (128 bytes of each W1/W3 output where
// eight store 64), which pays while the chip is full for long and where H1 and H3 are
// saved; eight of 128 x 64 share a tile's prologue and epilogue out further and hide more
// latency, which pays where the tiles fill half the chip once, and in W1/W3 without saved
// outputs where a contraction is short.  Measured, four against eight: W1/W3 of 64 experts
// x 2048 rows, d 2048, h 1024 847 and 872 us; d 1024, h 512 237 and 246 (512 rows 63.3 and
// 60.5, saving 69.8 and 75.6); d 640, h 384, 1400 rows 105 and 97; d 512, h 256, 256 rows
// 19.6 and 17.4, 1024 rows 39.5 and 36.0, saving 46.7 and 59.3; 32 experts, d 768, h 1536,
// 512 rows (768 tiles) 77.6 and 81.5; 8 experts, d 2048, h 1024, 512 rows (128 tiles) 44.0
// and 42.3, saving 46.1 and 44.2; W2 there 27.4 and 26.2 (d 1024, h 512 17.4 and 16.2),
// but of 64 experts x 256 rows, d 1024, h 512 (256 tiles) 22.0 and, on some cards, 26.5.
bool fwd_eight_waves(int epi, long tiles, int k, bool saves) {
  if (tiles <= 128) return true;
  return epi == EPI_SWIGLU && !saves && (k <= 704 || (k <= 1024 && tiles <= 512));
}

// A forward product in BM x 256 tiles of four or eight waves.
template <int BM, int EPI, int TAG, int OPT, bool VAR = false>
hipError_t run_fwd(const GemmParams& p, hipStream_t st, long max_rows = 0) {
  constexpr int WIDTH = EPI == EPI_SWIGLU ? 128 : 256;   // output columns of a tile
  // variable rows: the row blocks of max_rows in one and half a block more per batch
  const long blocks = VAR ? max_rows / BM + (p.batches + 1) / 2
                          : (long)p.batches * ((p.M + BM - 1) / BM);
  const long tiles = blocks * ((p.N + WIDTH - 1) / WIDTH);
  auto run = [&](auto wgn) -> hipError_t {
    constexpr int WGN = decltype(wgn)::value;
    if constexpr (VAR)
      return run_dma_var<BM, 256, 2, WGN, 64, 2, true, true, EPI, false, TAG, OPT>(p, max_rows, st);
    else
      return run_dma<BM, 256, 2, WGN, 64, 2, true, true, EPI, false, TAG, OPT>(p, st);
  };
  return fwd_eight_waves(EPI, tiles, p.K, p.H1 != nullptr) ? run(std::integral_constant<int, 4>{})
                                                             : run(std::integral_constant<int, 2>{});
}

// Buffers of one 128-row block (three stages): 128 x 128 tiles of four waves while there
// is at most one per CU; 128 x 256 of eight, which read the rows half as often, where
// those are at most one per CU.  Past that W1/W3 takes the narrow and W2 the wide ones, by
// measurement alone.  128 rows, narrow against wide: W1/W3 of 64 experts, d 512, h 256 (256
// narrow tiles) 10.5 and 12.4 us, d 1024, h 512 (512) 28.2 and 23.8, 24 experts, d 2048,
// h 1024 (384) 49.6 and 41.9, 64 experts (1024) 127 and 131; W2 of 8 experts, d 2048, h
// 1024 (128) 13.0 and 16.1, 64 experts (1024) 63 and 57.
template <int EPI, int TAG>
hipError_t run_fwd_128(const GemmParams& p, hipStream_t st) {
  const int width = EPI == EPI_SWIGLU ? 2 * p.N : p.N;
  const long narrow = (long)p.batches * ((width + 127) / 128);
  const long wide = (long)p.batches * ((width + 255) / 256);
  if (narrow <= 256 || (EPI == EPI_SWIGLU && wide > 256))
    return run_dma<128, 128, 2, 2, 64, 3, true, true, EPI, false, TAG>(p, st);
  return run_dma<128, 256, 2, 4, 64, 3, true, true, EPI, false, TAG>(p, st);
}

// ------------------------------------------------------------------ fp32 MFMA
//
// v_mfma_f32_32x32x2_f32 over the same operand conventions: every product and sum in
// fp32.  A k-step is 32 wide (128-byte rows, the layout and swizzle of the bf16
// kernel's K-contiguous tiles); a lane's 16-byte chunk holds four consecutive k of its
// row, MFMA i of a sub-step taking element i of both lane halves (k = 8 s + i and
// 8 s + 4 + i).  K-major tiles stay K-major, read with four 4-byte reads per fragment.
// The matrix cores bound it: a k-step of a 64 x 64 wave tile is 4096 MFMA cycles, far
// more than its LDS reads (1/8 of the port) or its DMA, so one barrier per step and
// two stages suffice, and accumulators go straight to memory (16 bytes a lane).
// Measured, 16 experts x 512 rows, d 1024, h 512: W1/W3 484 -> 150 us (115 TFLOP/s, MFMA
// busy 78% of the cycles), W2 240 -> 79, dA 268 -> 98, dX 530 -> 155, dW1/dW3 520 -> 158,
// against a 64 x 64 tile of scalar FMAs; a plain 8192^3 library product reaches 154.
constexpr int FK = 32;   // k-step
// 128 x 128 tiles from one per CU on (the same problem in 64 x 64 tiles, whose waves
// read a third more LDS per MFMA and meet at twice as many barriers: 1037 against 795 us
// a training step); below that 64 x 64 tiles keep more CUs busy.
constexpr long F32_BIG_TILES = 256;

template <int BM, int BN, int WGM, int WGN, bool A_KC, bool B_KC, int EPI, int OPT>
__global__ __launch_bounds__(64 * WGM * WGN) void gemm_f32_kernel(GemmParams p) {
  constexpr int NT = 64 * WGM * WGN;
  constexpr int WM = BM / WGM, WN = BN / WGN, MB = WM / 32, NB = WN / 32;
  constexpr int A_BYTES = BM * FK * 4, STAGE_BYTES = (BM + BN) * FK * 4;
  constexpr int AL = BM * 8 / NT, BL = BN * 8 / NT;   // 16-byte chunks per thread and step
  static_assert(BM * 8 % NT == 0 && BN * 8 % NT == 0, "whole chunks per thread");
  static_assert(EPI != EPI_SWIGLU || (B_KC && NB == 2), "a W1 and a W3 block per wave");
  static_assert(EPI != EPI_SWIGLU_BWD || WN == 64, "a wave covers one 64-column partial");
  constexpr bool GA = (OPT & OPT_GA) != 0;
  static_assert(!(GA && A_KC) && (OPT & ~OPT_GA) == 0, "a K-major A may be gathered");
  __shared__ __attribute__((aligned(1024))) char smem[2 * STAGE_BYTES];

  const int t = xcd_tile_id(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
  const int per_b = p.MT * p.NT;
  if (t >= p.batches * per_b) return;
  const int e = t / per_b, rem = t - e * per_b;
  const int m0 = rem % p.MT * BM;
  const int n0 = rem / p.MT * (EPI == EPI_SWIGLU ? BN / 2 : BN);
  // rows of this batch: uniform (M), or [var_rows[e], var_rows[e+1]) of packed buffers
  int M = p.M, row0 = 0;
  size_t a_off = (size_t)e * p.a_bs, c_off = (size_t)e * p.c_bs, h_off = (size_t)e * p.h_bs;
  if (p.var_rows) {
    row0 = p.var_rows[e];
    M = p.var_rows[e + 1] - row0;
    a_off = (size_t)row0 * p.lda;
    c_off = (size_t)row0 * p.ldc;
    h_off = (size_t)row0 * p.ldh;
  }
  if (m0 >= M) return;
  const float* A = (const float*)p.A + a_off;
  const float* B = (const float*)p.B + (size_t)e * p.b_bs;
  const float* B2 = p.B2 ? (const float*)p.B2 + (size_t)e * p.b_bs : nullptr;
  const float* zero = reinterpret_cast<const float*>(g_zero_block);

  const int tid = threadIdx.x, lane = tid & 63, l31 = lane & 31, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % WGM, wn = wave / WGM;

  // DMA sources: load q of a thread fills the 16 bytes at (wave L + q) 1024 + 16 lane
  // of the operand's area.  K-contiguous: the chunk's address at k-step 0.  K-major: the
  // chunk's column; its row is formed per step (a gathered row's index is read a
  // step ahead); rows past the valid K and columns past the width read zeros.
  const float* a_src[AL];
  const float* b_src[BL];
  int a_idx[AL];
  auto km_idx = [&](int k) -> int {
    return p.ka_rows[(size_t)e * p.k_rows_bs + (k < p.kv_a ? k : p.kv_a - 1)];
  };
#pragma unroll
  for (int q = 0; q < AL; ++q) {
    const int id = (wave * AL + q) * 64 + lane;
    if constexpr (A_KC) {
      const int row = id >> 3, lc = (id & 7) ^ kc_swz(row);
      int r = m0 + row;
      r = r < M ? r : M - 1;
      a_src[q] = p.a_rows ? (const float*)p.A +
                                (size_t)p.a_rows[(size_t)e * p.a_rows_bs + row0 + r] * p.lda + lc * 4
                          : A + (size_t)r * p.lda + lc * 4;
    } else {
      const int col = m0 + id % (BM / 4) * 4;
      a_src[q] = col < M ? (GA ? (const float*)p.A : A) + col : nullptr;
      if constexpr (GA) a_idx[q] = p.kv_a > 0 ? km_idx(id / (BM / 4)) : 0;
    }
  }
#pragma unroll
  for (int q = 0; q < BL; ++q) {
    const int id = (wave * BL + q) * 64 + lane;
    if constexpr (B_KC) {
      const int row = id >> 3, lc = (id & 7) ^ kc_swz(row);
      if constexpr (EPI == EPI_SWIGLU) {
        int r = n0 + row % (BN / 2);
        r = r < p.N ? r : p.N - 1;
        b_src[q] = (row < BN / 2 ? B : B2) + (size_t)r * p.ldb + lc * 4;
      } else {
        int r = n0 + row;
        r = r < p.N ? r : p.N - 1;
        b_src[q] = B + (size_t)r * p.ldb + lc * 4;
      }
    } else {
      const int col = n0 + id % (BN / 4) * 4;
      b_src[q] = col < p.N ? B + col : nullptr;
    }
  }
  const long b2_off = B2 ? B2 - B : 0;
  auto issue = [&](int kt, int stage) {
    char* base = smem + stage * STAGE_BYTES;
#pragma unroll
    for (int q = 0; q < AL; ++q) {
      const float* g;
      if constexpr (A_KC) {
        g = a_src[q] + kt * FK;
      } else {
        const int k = kt * FK + ((wave * AL + q) * 64 + lane) / (BM / 4);
        g = (k < p.kv_a && a_src[q]) ? a_src[q] + (size_t)(GA ? a_idx[q] : k) * p.lda : zero;
        if constexpr (GA) a_idx[q] = km_idx(k + FK);
      }
      dma16(g, base + (wave * AL + q) * 1024);
    }
#pragma unroll
    for (int q = 0; q < BL; ++q) {
      const float* g;
      if constexpr (B_KC) {
        g = b_src[q] + kt * FK;
      } else {
        const int k = kt * FK + ((wave * BL + q) * 64 + lane) / (BN / 4);
        const float* s = b_src[q] + (k < p.k_split ? 0 : b2_off);
        const int kr = k < p.k_split ? k : k - p.k_split;
        g = (k < p.kv_b && b_src[q]) ? s + (size_t)kr * p.ldb : zero;
      }
      dma16(g, base + A_BYTES + (wave * BL + q) * 1024);
    }
  };
  // the four k of sub-step s that this lane holds, for tile row (or column) base + lane % 32
  auto frag = [&](const char* __restrict__ tile, auto kc, int width, int base, int s) -> f32x4 {
    if constexpr (decltype(kc)::value) {
      const int row = base + l31;
      return *reinterpret_cast<const f32x4*>(tile + row * (FK * 4) +
                                             (((2 * s + half) ^ kc_swz(row)) << 4));
    } else {
      const float* c = reinterpret_cast<const float*>(tile) + (8 * s + 4 * half) * width + base + l31;
      return f32x4{c[0], c[width], c[2 * width], c[3 * width]};
    }
  };
  auto b_col = [&](int ni) -> int {
    return EPI == EPI_SWIGLU ? ni * (BN / 2) + wn * (WN / 2) : wn * WN + ni * 32;
  };

  f32x16 acc[MB][NB];
#pragma unroll
  for (int mi = 0; mi < MB; ++mi)
#pragma unroll
    for (int ni = 0; ni < NB; ++ni)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mi][ni][r] = 0.f;

  const int KT = (p.K + FK - 1) / FK;
  if (KT > 0) issue(0, 0);
  for (int kt = 0; kt < KT; ++kt) {
    // step kt has landed for every wave, and every wave has read step kt - 1
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    __syncthreads();
    if (kt + 1 < KT) issue(kt + 1, (kt + 1) & 1);
    const char* sa = smem + (kt & 1) * STAGE_BYTES;
    const char* sb = sa + A_BYTES;
    // the fragments of sub-step s + 1 are requested before the MFMAs of sub-step s
    f32x4 af[2][MB], bf[2][NB];
    auto load = [&](int s) {
#pragma unroll
      for (int mi = 0; mi < MB; ++mi)
        af[s & 1][mi] = frag(sa, std::integral_constant<bool, A_KC>{}, BM, wm * WM + mi * 32, s);
#pragma unroll
      for (int ni = 0; ni < NB; ++ni)
        bf[s & 1][ni] = frag(sb, std::integral_constant<bool, B_KC>{}, BN, b_col(ni), s);
    };
    load(0);
#pragma unroll
    for (int s = 0; s < FK / 8; ++s) {
      if (s + 1 < FK / 8) load(s + 1);
      __builtin_amdgcn_sched_barrier(0);
      // B first: each lane ends with four consecutive output columns of a row
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int mi = 0; mi < MB; ++mi)
#pragma unroll
          for (int ni = 0; ni < NB; ++ni)
            acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(
                bf[s & 1][ni][i], af[s & 1][mi][i], acc[mi][ni], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // acc[mi][ni][4 g + i]: row lane % 32 of the block, column 8 g + 4 (lane / 32) + i
#pragma unroll
  for (int mi = 0; mi < MB; ++mi) {
    const int m = m0 + wm * WM + mi * 32 + l31;
    const bool row_ok = m < M;
    const float gate =
        ((EPI == EPI_SWIGLU || EPI == EPI_SWIGLU_BWD) && p.gate && row_ok)
            ? p.gate[(size_t)e * p.gate_bs + m] : 1.f;
    float dsum = 0.f;   // SwiGLU backward: the row's gate-gradient partial
#pragma unroll
    for (int ni = 0; ni < (EPI == EPI_SWIGLU ? 1 : NB); ++ni) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int n = n0 + (EPI == EPI_SWIGLU ? wn * (WN / 2) : wn * WN + ni * 32) + 8 * g + 4 * half;
        if (!row_ok || n >= p.N) continue;
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = acc[mi][ni][4 * g + i];
        if constexpr (EPI == EPI_STORE || EPI == EPI_STORE_ADD) {
          const bool second = m >= p.c_split;
          float4* dst = reinterpret_cast<float4*>((float*)(second ? p.C2 : p.C) + c_off +
                                                  (size_t)(second ? m - p.c_split : m) * p.ldc + n);
          float4 o = make_float4(v[0], v[1], v[2], v[3]);
          if constexpr (EPI == EPI_STORE_ADD) {
            const float4 old = *dst;
            o = make_float4(old.x + o.x, old.y + o.y, old.z + o.z, old.w + o.w);
          }
          *dst = o;
        } else if constexpr (EPI == EPI_SWIGLU) {
          float a[4], h3[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            h3[i] = acc[mi][NB - 1][4 * g + i];
            a[i] = silu_f(v[i]) * h3[i] * gate;
          }
          *reinterpret_cast<float4*>((float*)p.C + c_off + (size_t)m * p.ldc + n) =
              make_float4(a[0], a[1], a[2], a[3]);
          if (p.H1) {
            const size_t ho = h_off + (size_t)m * p.ldh + n;
            *reinterpret_cast<float4*>((float*)p.H1 + ho) = make_float4(v[0], v[1], v[2], v[3]);
            *reinterpret_cast<float4*>((float*)p.H3 + ho) = make_float4(h3[0], h3[1], h3[2], h3[3]);
          }
        } else {
          const size_t ho = h_off + (size_t)m * p.ldh + n;
          const float4 h1v = *reinterpret_cast<const float4*>((const float*)p.H1 + ho);
          const float4 h3v = *reinterpret_cast<const float4*>((const float*)p.H3 + ho);
          const float h1a[4] = {h1v.x, h1v.y, h1v.z, h1v.w}, h3a[4] = {h3v.x, h3v.y, h3v.z, h3v.w};
          float d1[4], d3[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float da = v[i] * gate, sg = sigmoid_f(h1a[i]);
            d1[i] = da * h3a[i] * sg * (1.0f + h1a[i] * (1.0f - sg));
            d3[i] = da * h1a[i] * sg;
            dsum = fmaf(da, h1a[i] * sg * h3a[i], dsum);
          }
          const size_t off = c_off + (size_t)m * p.ldc + n;
          *reinterpret_cast<float4*>((float*)p.C + off) = make_float4(d1[0], d1[1], d1[2], d1[3]);
          *reinterpret_cast<float4*>((float*)p.C2 + off) = make_float4(d3[0], d3[1], d3[2], d3[3]);
        }
      }
    }
    if constexpr (EPI == EPI_SWIGLU_BWD) {
      // the two lanes of a row hold its 64-column block (N is a multiple of 64)
      const float tsum = dsum + __shfl_xor(dsum, 32, 64);
      const int nb = n0 + wn * WN;
      if (p.dsp && half == 0 && row_ok && nb < p.N)
        p.dsp[((size_t)e * p.M + m) * p.dsp_ld + (nb >> 6)] = tsum;
    }
  }
}

template <int BM, int BN, int WGM, int WGN, bool A_KC, bool B_KC, int EPI, int OPT>
hipError_t launch_f32_tile(GemmParams p, hipStream_t st) {
  p.MT = (p.M + BM - 1) / BM;
  p.NT = (EPI == EPI_SWIGLU) ? (p.N + BN / 2 - 1) / (BN / 2) : (p.N + BN - 1) / BN;
  const long ntile = (long)p.batches * p.MT * p.NT;
  if (ntile == 0) return hipSuccess;
  if (ntile >= (1l << 30)) return hipErrorInvalidValue;   // 2^26 at the size limits
  // One dimension of a launch ends below 2^32 threads, which token choice passes (its
  // grid covers every token for every expert): rows of at most 2^23 workgroups, whole
  // rounds of the XCDs each.
  const long rows = (ntile + (1l << 23) - 1) >> 23;
  const long per_row = ((ntile + rows - 1) / rows + 7) / 8 * 8;
  gemm_f32_kernel<BM, BN, WGM, WGN, A_KC, B_KC, EPI, OPT>
      <<<dim3((unsigned)per_row, (unsigned)rows), 64 * WGM * WGN, 0, st>>>(p);
  return hipGetLastError();
}

// OPT: as in run_dma.
template <bool A_KC, bool B_KC, int EPI, int OPT = 0>
hipError_t run_f32(const GemmParams& p, hipStream_t st) {
  if (((OPT & OPT_GA) != 0) != (p.ka_rows != nullptr)) return hipErrorInvalidValue;
  const int nw = EPI == EPI_SWIGLU ? 2 * p.N : p.N;
  const long big = (long)p.batches * ((p.M + 127) / 128) * ((nw + 127) / 128);
  if (big >= F32_BIG_TILES) return launch_f32_tile<128, 128, 2, 2, A_KC, B_KC, EPI, OPT>(p, st);
  return launch_f32_tile<64, 64, 2, 1, A_KC, B_KC, EPI, OPT>(p, st);
}

GemmParams base_params() {
  GemmParams p = {};
  p.k_split = 1 << 30;
  p.c_split = 1 << 30;
  return p;
}

// Deterministic split-K reduction (partials added in the order of the splits) into
// the output type, with the output's row split: row r < c_split goes to C, the others
// to C2 at r - c_split.  Four columns a thread (N is a multiple of 64), eight partials
// in flight: it moves at memory speed (8 fp32 partials of 2048 x 2048: 34 -> 12 us with
// one element a thread; 32 of 64 x 2048: 10 -> 5).
template <typename T>
__global__ __launch_bounds__(64) void splitk_store_kernel(const float* __restrict__ part,
                                                          int splits, int M, int N, int c_split,
                                                          T* __restrict__ C, T* __restrict__ C2,
                                                          int ldc) {
  const long i = ((long)blockIdx.x * 64 + threadIdx.x) * 4;
  const long n = (long)M * N;
  if (i >= n) return;
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
  for (int q = 0; q < splits; ++q) s += *reinterpret_cast<const f32x4*>(part + (size_t)q * n + i);
  const int r = (int)(i / N), c = (int)(i % N);
  T* dst = (r < c_split ? C + (size_t)r * ldc : C2 + (size_t)(r - c_split) * ldc) + c;
  if constexpr (sizeof(T) == 4)
    *reinterpret_cast<f32x4*>(dst) = s;
  else
    *reinterpret_cast<uint2*>(dst) = make_uint2(pack_bf16x2(s[0], s[1]), pack_bf16x2(s[2], s[3]));
}

template <typename T>
hipError_t run_splitk_store(const float* part, int splits, int M, int N, int c_split, T* C, T* C2,
                            int ldc, hipStream_t st) {
  const long n4 = (long)M * N / 4;
  splitk_store_kernel<T><<<(unsigned)((n4 + 63) / 64), 64, 0, st>>>(part, splits, M, N, c_split, C,
                                                                    C2, ldc);
  return hipGetLastError();
}

}  // namespace

// ---------------------------------------------------------------- launchers

int dsp_parts(int dtype, int h) { return dtype == DT_F32 ? (h + 63) / 64 : (h + 127) / 128; }

hipError_t launch_gemm_w13(int dtype, const void* Xe, const void* W1, const void* W3, void* A,
                           void* H1, void* H3, int E, int M, int d, int h, hipStream_t st,
                           bool shared, const int32_t* rows, const float* gate) {
  GemmParams p = base_params();
  p.gate = gate; p.gate_bs = M;
  p.A = Xe; p.a_bs = (long)M * d; p.lda = d;
  if (rows) {   // Xe is X itself, row m of expert e is X[rows[e M + m]]
    p.a_bs = 0; p.a_rows = rows; p.a_rows_bs = M;
  }
  p.B = W1; p.B2 = W3; p.b_bs = (long)h * d; p.ldb = d;
  p.M = M; p.N = h; p.K = d; p.kv_a = d; p.kv_b = d; p.batches = E;
  p.C = A; p.c_bs = (long)M * h; p.ldc = h;
  p.H1 = H1; p.H3 = H3; p.h_bs = (long)M * h; p.ldh = h;
  if (M == 0) return hipSuccess;
  if (dtype == DT_F32) {
    return run_f32<true, true, EPI_SWIGLU>(p, st);
  }
  if (shared) {
    if (rows) return hipErrorInvalidValue;   // the shared experts read X as is
    return run_fwd<256, EPI_SWIGLU, G_SH_W13, 0>(p, st);
  }
  switch (fwd_block_rows(M)) {
    case 64: return run_dma<64, 128, 2, 2, 64, 3, true, true, EPI_SWIGLU, false, G_W13>(p, st);
    case 128: return run_fwd_128<EPI_SWIGLU, G_W13>(p, st);
    case 192: return run_fwd<192, EPI_SWIGLU, G_W13, 0>(p, st);
    default: return run_fwd<256, EPI_SWIGLU, G_W13, OPT_TAILS>(p, st);
  }
}

hipError_t launch_gemm_w2(int dtype, const void* A, const void* W2, void* O, int E, int M, int d,
                          int h, hipStream_t st, bool shared) {
  GemmParams p = base_params();
  p.A = A; p.a_bs = (long)M * h; p.lda = h;
  p.B = W2; p.b_bs = (long)d * h; p.ldb = h;
  p.M = M; p.N = d; p.K = h; p.kv_a = h; p.kv_b = h; p.batches = E;
  p.C = O; p.c_bs = (long)M * d; p.ldc = d;
  if (M == 0) return hipSuccess;
  if (dtype == DT_F32) return run_f32<true, true, EPI_STORE>(p, st);
  if (shared) return run_fwd<256, EPI_STORE, G_SH_W2, 0>(p, st);
  switch (fwd_block_rows(M)) {
    case 64: return run_dma<64, 128, 2, 2, 64, 3, true, true, EPI_STORE, false, G_W2>(p, st);
    case 128: return run_fwd_128<EPI_STORE, G_W2>(p, st);
    case 192: return run_fwd<192, EPI_STORE, G_W2, 0>(p, st);
    default: return run_fwd<256, EPI_STORE, G_W2, OPT_TAILS>(p, st);
  }
}

hipError_t launch_gemm_dA(int dtype, const void* dO, const void* W2, const void* H1,
                          const void* H3, void* dH, int E, int M, int d, int h, hipStream_t st,
                          bool shared, float* dsp, const int32_t* rows, const float* gate) {
  // dA[m, n] = g_m sum_k dO[m, k] W2[k, n]  (k over d, n over h); epilogue -> dH1, dH3
  GemmParams p = base_params();
  p.A = dO; p.a_bs = (long)M * d; p.lda = d;
  if (rows) {   // dO is dY itself, row m of expert e is dY[rows[e M + m]]
    p.a_bs = 0; p.a_rows = rows; p.a_rows_bs = M;
  }
  p.gate = gate; p.gate_bs = M;
  p.B = W2; p.b_bs = (long)d * h; p.ldb = h;
  p.M = M; p.N = h; p.K = d; p.kv_a = d; p.kv_b = d; p.batches = E;
  const size_t esz = dtype == DT_F32 ? 4 : 2;
  p.C = dH; p.C2 = (char*)dH + (size_t)h * esz; p.c_bs = (long)M * 2 * h; p.ldc = 2 * h;
  p.H1 = (void*)H1; p.H3 = (void*)H3; p.h_bs = (long)M * h; p.ldh = h;
  p.dsp = dsp; p.dsp_ld = dsp_parts(dtype, h);
  if (M == 0) return hipSuccess;
  if (dtype == DT_F32) {
    return run_f32<true, false, EPI_SWIGLU_BWD>(p, st);
  }
  if (shared && rows) return hipErrorInvalidValue;
  // B = W2 K-major: B(n, k) = W2[k, n]
  if (shared)
    return run_dma<256, 256, 4, 2, 64, 2, true, false, EPI_SWIGLU_BWD, false, G_SH_DA>(p, st);
  return run_dma<256, 256, 4, 2, 64, 2, true, false, EPI_SWIGLU_BWD, false, G_DA, OPT_TAILS>(p, st);
}

hipError_t launch_gemm_dXe(int dtype, const void* dH, const void* W1, const void* W3, void* dXe,
                           int E, int M, int d, int h, hipStream_t st, bool shared) {
  // dXe[m, n] = sum_k dH[m, k] W13[k, n], k < h from W1, k >= h from W3
  GemmParams p = base_params();
  p.A = dH; p.a_bs = (long)M * 2 * h; p.lda = 2 * h;
  p.B = W1; p.B2 = W3; p.b_bs = (long)h * d; p.ldb = d; p.k_split = h;
  p.M = M; p.N = d; p.K = 2 * h; p.kv_a = 2 * h; p.kv_b = 2 * h; p.batches = E;
  p.C = dXe; p.c_bs = (long)M * d; p.ldc = d;
  if (M == 0) return hipSuccess;
  if (dtype == DT_F32) return shared ? run_f32<true, false, EPI_STORE_ADD>(p, st)
                                     : run_f32<true, false, EPI_STORE>(p, st);
  // bf16: B K-major, rows k >= h from W3 (h is a multiple of the k-step); the
  // shared experts' input gradient is added to dX
  if (h % 64 != 0) return hipErrorInvalidValue;
  if (shared)
    return run_dma<256, 256, 4, 2, 64, 2, true, false, EPI_STORE_ADD, false, G_SH_DXE>(p, st);
  return run_dma<256, 256, 4, 2, 64, 2, true, false, EPI_STORE, false, G_DXE, OPT_TAILS>(p, st);
}

hipError_t launch_gemm_dW2(int dtype, const void* dO, const void* A, void* dW2, int E, int M,
                           int d, int h, hipStream_t st, const int32_t* rows) {
  // dW2[m, n] = sum_k dO[k, m] A[k, n]  (m over d, n over h, k over the M expert rows)
  GemmParams p = base_params();
  p.A = dO; p.a_bs = (long)M * d; p.lda = d;
  p.B = A; p.b_bs = (long)M * h; p.ldb = h;
  p.M = d; p.N = h; p.K = M; p.kv_a = M; p.kv_b = M; p.batches = E;
  p.C = dW2; p.c_bs = (long)d * h; p.ldc = h;
  if (rows) {   // dO is dY itself, row k of expert e is dY[rows[e M + k]]
    p.a_bs = 0; p.ka_rows = rows; p.k_rows_bs = M;
    if (dtype == DT_F32) return run_f32<false, false, EPI_STORE, OPT_GA>(p, st);
    return run_dma<256, 256, 4, 2, 64, 2, false, false, EPI_STORE, false, G_DW2, OPT_GA | OPT_TAILS>(p, st);
  }
  if (dtype == DT_F32) return run_f32<false, false, EPI_STORE>(p, st);
  return hipErrorInvalidValue;   // bf16 gathers the rows of dO
}

hipError_t launch_gemm_dW13(int dtype, const void* dH, const void* Xe, void* dW1, void* dW3,
                            int E, int M, int d, int h, hipStream_t st, const int32_t* rows) {
  // [dW1; dW3][m, n] = sum_k dH[k, m] Xe[k, n]  (m over 2h, n over d)
  GemmParams p = base_params();
  p.A = dH; p.a_bs = (long)M * 2 * h; p.lda = 2 * h;
  p.B = Xe; p.b_bs = (long)M * d; p.ldb = d;
  p.M = 2 * h; p.N = d; p.K = M; p.kv_a = M; p.kv_b = M; p.batches = E;
  p.C = dW1; p.C2 = dW3; p.c_split = h; p.c_bs = (long)h * d; p.ldc = d;
  if (rows) {   // Xe is X itself, row k of expert e is X[rows[e M + k]]
    if (dtype == DT_F32) return hipErrorInvalidValue;   // fp32 reads the saved Xe
    p.b_bs = 0; p.kb_rows = rows; p.k_rows_bs = M;
    return run_dma<256, 256, 4, 2, 64, 2, false, false, EPI_STORE, false, G_DW13, OPT_GB | OPT_TAILS>(p, st);
  }
  if (dtype == DT_F32) return run_f32<false, false, EPI_STORE>(p, st);
  return hipErrorInvalidValue;   // bf16 gathers the rows of X
}

hipError_t launch_router_dx(int dtype, const void* dZ, const void* Wg, void* dX, int N, int E,
                            int EP, int d, hipStream_t st) {
  // dX[i, n] = sum_j dZ[i, j] Wg[j, n]; dZ is [N, EP], zero padded
  GemmParams p = base_params();
  p.A = dZ; p.a_bs = 0; p.lda = EP;
  p.B = Wg; p.b_bs = 0; p.ldb = d;
  p.M = N; p.N = d; p.K = EP; p.kv_a = EP; p.kv_b = E; p.batches = 1;
  p.C = dX; p.c_bs = 0; p.ldc = d;
  if (N == 0) return hipSuccess;
  if (dtype == DT_F32) return run_f32<true, false, EPI_STORE>(p, st);
  return run_dma<256, 256, 4, 2, 64, 2, true, false, EPI_STORE, false, G_ROUTER_DX, OPT_TILE_BASE>(
      p, st);
}

hipError_t launch_router_dwg(int dtype, const void* dZ, const void* X, float* dWg, float* part,
                             int splits, int N, int E, int EP, int d, hipStream_t st) {
  // dWg[j, n] = sum_i dZ[i, j] X[i, n], split over i in at most `splits` chunks
  if (N == 0 || splits < 1) return launch_zero(dWg, (size_t)E * d * sizeof(float), st);
  const RowSplit rs = split_rows(N, splits, 1);
  const size_t esz = dtype == DT_F32 ? 4 : 2;
  // `batches` chunks from row `row0` on, of which `rows` rows each are there
  auto run = [&](int batches, long row0, int rows, float* out) -> hipError_t {
    GemmParams p = base_params();
    p.A = (const char*)dZ + row0 * EP * esz; p.a_bs = (long)rs.chunk * EP; p.lda = EP;
    p.B = (const char*)X + row0 * d * esz; p.b_bs = (long)rs.chunk * d; p.ldb = d;
    p.M = E; p.N = d; p.K = rs.chunk; p.kv_a = rows; p.kv_b = rows; p.batches = batches;
    p.C = out; p.c_bs = (long)E * d; p.ldc = d;
    if (dtype == DT_F32) return run_f32<false, false, EPI_STORE>(p, st);
    return run_dma<128, 256, 2, 4, 64, 2, false, false, EPI_STORE, true, G_ROUTER_DWG>(p, st);
  };
  hipError_t err = rs.full > 0 ? run(rs.full, 0, rs.chunk, part) : hipSuccess;
  if (err == hipSuccess && rs.last > 0)
    err = run(1, (long)rs.full * rs.chunk, rs.last, part + (size_t)rs.full * E * d);
  if (err != hipSuccess) return err;
  return run_splitk_store<float>(part, rs.parts(), E, d, E, dWg, dWg, d, st);
}

namespace {

// C[m, n] = sum_k A[k, m] B[k, n] over K rows (both operands K-major), split
// over the rows into `splits` fp32 partials (part [splits, M, N]) added in a
// fixed order into C (rows < c_split) and C2 (the others).  One batch only.
template <int TAG>
hipError_t run_wgrad_splitk(const void* A, int lda, const void* B, int ldb, int M, int N, int K,
                            void* C, void* C2, int c_split, int ldc, float* part, int splits,
                            hipStream_t st) {
  if (K == 0 || splits < 1) {
    // no rows: the gradient is zero
    hipError_t e = launch_zero(C, (size_t)(c_split < M ? c_split : M) * ldc * 2, st);
    if (e != hipSuccess || c_split >= M) return e;
    return launch_zero(C2, (size_t)(M - c_split) * ldc * 2, st);
  }
  const RowSplit rs = split_rows(K, splits, 64);
  const int chunk = rs.chunk, full = rs.full, last = rs.last;
  GemmParams p = base_params();
  p.A = A; p.a_bs = (long)chunk * lda; p.lda = lda;
  p.B = B; p.b_bs = (long)chunk * ldb; p.ldb = ldb;
  p.M = M; p.N = N; p.K = chunk; p.kv_a = chunk; p.kv_b = chunk;
  p.C = part; p.c_bs = (long)M * N; p.ldc = N;
  hipError_t err = hipSuccess;
  if (full > 0) {
    p.batches = full;
    err = run_dma<256, 256, 4, 2, 64, 2, false, false, EPI_STORE, true, TAG>(p, st);
    if (err != hipSuccess) return err;
  }
  if (last > 0) {
    GemmParams q = p;
    q.A = (const bf16_t*)A + (size_t)full * chunk * lda;
    q.B = (const bf16_t*)B + (size_t)full * chunk * ldb;
    q.C = part + (size_t)full * M * N;
    q.K = last; q.kv_a = last; q.kv_b = last; q.batches = 1;
    err = run_dma<256, 256, 4, 2, 64, 2, false, false, EPI_STORE, true, TAG>(q, st);
    if (err != hipSuccess) return err;
  }
  return run_splitk_store<bf16_t>(part, rs.parts(), M, N, c_split, (bf16_t*)C, (bf16_t*)C2, ldc, st);
}

}  // namespace

hipError_t launch_shared_dW2(int dtype, const void* dY, const void* A, void* dW2, int N, int d,
                             int h, float* part, int splits, hipStream_t st) {
  // dW2[m, n] = sum_i dY[i, m] A[i, n]  (m over d, n over h, i over all N tokens)
  if (dtype == DT_F32) return launch_gemm_dW2(dtype, dY, A, dW2, 1, N, d, h, st);
  return run_wgrad_splitk<G_SH_DW2>(dY, d, A, h, d, h, N, dW2, dW2, 1 << 30, h, part, splits, st);
}

hipError_t launch_shared_dW13(int dtype, const void* dH, const void* X, void* dW1, void* dW3,
                              int N, int d, int h, float* part, int splits, hipStream_t st) {
  // [dW1; dW3][m, n] = sum_i dH[i, m] X[i, n]  (m over 2h, n over d)
  if (dtype == DT_F32) return launch_gemm_dW13(dtype, dH, X, dW1, dW3, 1, N, d, h, st);
  return run_wgrad_splitk<G_SH_DW13>(dH, 2 * h, X, d, 2 * h, d, N, dW1, dW3, h, d, part, splits,
                                     st);
}

int tc_col_blocks_w13(int h) { return (h + 127) / 128; }
int tc_col_blocks_w2(int d) { return (d + 255) / 256; }

hipError_t launch_gemm_w13_var(int dtype, const void* Xe, const void* W1, const void* W3, void* A,
                               int E, const int32_t* rows, const int32_t* tiles, long max_rows,
                               int max_rows_per_expert, int d, int h, hipStream_t st,
                               const int32_t* sel) {
  GemmParams p = base_params();
  p.A = Xe; p.lda = d;
  if (sel) {   // Xe is X itself, packed row r is X[sel[r]]
    p.a_rows = sel; p.a_rows_bs = 0;
  }
  p.B = W1; p.B2 = W3; p.b_bs = (long)h * d; p.ldb = d;
  p.M = max_rows_per_expert; p.N = h; p.K = d; p.kv_a = d; p.kv_b = d; p.batches = E;
  p.C = A; p.ldc = h; p.ldh = h;
  p.var_rows = rows; p.var_tiles = tiles;
  if (max_rows == 0) return hipSuccess;
  if (dtype == DT_F32) return run_f32<true, true, EPI_SWIGLU>(p, st);
  return run_fwd<256, EPI_SWIGLU, G_TC_W13, OPT_TAILS, true>(p, st, max_rows);
}

hipError_t launch_gemm_w2_var(int dtype, const void* A, const void* W2, void* O, int E,
                              const int32_t* rows, const int32_t* tiles, long max_rows,
                              int max_rows_per_expert, int d, int h, hipStream_t st) {
  GemmParams p = base_params();
  p.A = A; p.lda = h;
  p.B = W2; p.b_bs = (long)d * h; p.ldb = h;
  p.M = max_rows_per_expert; p.N = d; p.K = h; p.kv_a = h; p.kv_b = h; p.batches = E;
  p.C = O; p.ldc = d;
  p.var_rows = rows; p.var_tiles = tiles;
  if (max_rows == 0) return hipSuccess;
  if (dtype == DT_F32) return run_f32<true, true, EPI_STORE>(p, st);
  return run_fwd<256, EPI_STORE, G_TC_W2, OPT_TAILS, true>(p, st, max_rows);
}

}  // namespace ec
