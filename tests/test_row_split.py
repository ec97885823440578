"""The split of a contraction over all tokens (CPU only): the header's arithmetic,
compiled for the host, covers every row exactly once and stays inside the rows and the
planned partial sums."""
import os
import shutil
import subprocess

import pytest

from paper_2604_01622_amd import build

PROGRAM = r"""
#include <cstdio>
#include "row_split.h"

static long bad = 0, fewer = 0;

static void check(int n, int splits, int step) {
  const ec::RowSplit r = ec::split_rows(n, splits, step);
  const bool ok = r.chunk >= 1 && r.chunk % step == 0 && r.full >= 0 && r.last >= 0 &&
                  r.last < r.chunk && (long)r.full * r.chunk + r.last == n &&
                  r.parts() >= 1 && r.parts() <= splits;
  if (!ok) ++bad;
  if (r.parts() < splits) ++fewer;
}

int main() {
  for (int n = 1; n <= 600000; ++n)
    for (int d = 64; d <= 1024; d *= 2) check(n, ec::router_dwg_splits(n, d), 1);
  for (int n = 1; n <= 5000; ++n)
    for (int m = 64; m <= 4096; m *= 2) check(n, ec::wgrad_splits(m, 192, n), 64);
  for (long n = (1l << 24) - 3000; n < (1l << 24); ++n) check((int)n, ec::router_dwg_splits((int)n, 64), 1);
  const ec::RowSplit r = ec::split_rows(131073, 512, 1);
  std::printf("%ld %ld %d %d %d\n", bad, fewer, r.chunk, r.full, r.last);
}
"""


def test_every_row_in_one_chunk(tmp_path):
    cc = shutil.which("g++")
    if cc is None:
        pytest.skip("needs g++")
    src, exe = tmp_path / "split.cpp", tmp_path / "split"
    src.write_text(PROGRAM)
    subprocess.run([cc, "-std=c++17", "-O2", "-Wall", "-Werror", "-I", build.CSRC, str(src), "-o",
                    str(exe)], check=True, capture_output=True, text=True)
    r = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=120)
    bad, fewer, chunk, full, last = (int(x) for x in r.stdout.split())
    assert bad == 0
    assert fewer > 0            # sizes whose chunks come out fewer than planned are among them
    assert (chunk, full, last) == (257, 510, 3)
