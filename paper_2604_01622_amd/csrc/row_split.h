// Host arithmetic of the contractions over all tokens that are split into partial sums
// (the router's and the shared experts' weight gradients).
#pragma once

namespace ec {

// n rows in chunks: `full` chunks of `chunk` rows, then one of `last` rows (0: none).
struct RowSplit {
  int chunk, full, last;
  int parts() const { return full + (last > 0); }
};

// At most `splits` chunks of a multiple of `step` rows; n, splits, step >= 1.  Rounding a
// chunk up can leave fewer than `splits` of them (131073 rows by 512: 510 chunks of 257
// and one of 3), so the whole chunks are counted from the rows.
inline RowSplit split_rows(int n, int splits, int step) {
  RowSplit s;
  s.chunk = ((n + splits - 1) / splits + step - 1) / step * step;
  s.full = n / s.chunk;
  s.last = n - s.full * s.chunk;
  return s;
}

// Planned splits of the router's weight gradient over N tokens: 512 tiles of 128 columns,
// chunks of 256 tokens or more.
inline int router_dwg_splits(int N, int d) {
  const int tiles = (d + 127) / 128, s = (512 + tiles - 1) / tiles, most = (N + 255) / 256;
  return s < most ? s : most > 1 ? most : 1;
}

// Planned splits of a shared expert's M x N weight gradient over K tokens: one 256 x 256
// tile per CU (every further split writes and reads another M x N fp32 partial), chunks of
// 256 tokens or more.
inline int wgrad_splits(int M, int N, int K) {
  const int tiles = ((M + 255) / 256) * ((N + 255) / 256);
  const int s = (256 + tiles - 1) / tiles, most = (K + 255) / 256;
  return s < most ? s : most > 1 ? most : 1;
}

}  // namespace ec
