"""The rules that share a store's bucket table among workgroups (csrc/work_split.h),
compiled for the host: every bucket is walked once, no workgroup walks group
after group of a sparse store while others are left out, and dense stores keep
one workgroup per so many rows."""
import os
import shutil
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2603_08883_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include "work_split.h"
using namespace iqcc;
int main() {
  long long rows, buckets, grid, threads, cand;
  char kind;
  while (std::scanf(" %c %lld %lld %lld %lld %lld", &kind, &rows, &buckets, &grid, &threads, &cand) == 6) {
    if (kind == 'l') {
      std::printf("%d\n", doublings(rows, buckets));
      continue;
    }
    if (kind == 'i') {   // rows, pairs, most pairs of an item, stash, waves
      std::printf("%d\n", 1 << item_pairs_log2(rows, buckets, log2_floor(grid), (int)threads, cand));
      continue;
    }
    if (kind == 'd') {   // grid: most ranges; threads: compute units
      std::printf("%lld\n", (long long)dis_range_buckets(rows, buckets, (int)grid, 0, cand, (int)threads));
      continue;
    }
    const BucketSplit s = kind == 'e' ? energy_buckets(rows, buckets, grid, (int)threads)
                                      : gradient_buckets(rows, buckets, grid, (int)threads);
    std::printf("%lld %lld %lld\n", (long long)s.G, (long long)s.ngroups, (long long)s.active);
  }
}
"""

ROWS = [0, 1, 100, 1000, 30000, 1_000_000, 50_000_000, 4_000_000_000]
BUCKETS = [1 << k for k in (0, 1, 5, 8, 9, 10, 13, 16, 19, 24, 28)]


def ceil(a, b):
    return -(-a // b)


@pytest.fixture(scope="module")
def split(tmp_path_factory):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("split")
    (d / "driver.cpp").write_text(DRIVER)
    subprocess.run([cxx, "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(d / "driver.cpp"), "-o", str(d / "driver")], check=True)

    def run(cases):
        text = "\n".join(f"{k} " + " ".join(str(v) for v in c) for k, *c in cases)
        out = subprocess.run([str(d / "driver")], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(int(v) for v in line.split()) for line in out.splitlines()]

    return run


@pytest.mark.parametrize("kind,grid,threads,most,rows_each", [
    ("e", 1024, 512, 512, 1024), ("e", 256, 1024, 1024, 1024), ("e", 1, 512, 512, 1024),
    ("g", 256, 768, 256, 768), ("g", 256, 384, 256, 384)])
def test_sums(split, kind, grid, threads, most, rows_each):
    cases = [(kind, r, b, grid, threads, 0) for r in ROWS for b in BUCKETS]
    for (_, r, b, *_), (G, ngroups, active) in zip(cases, split(cases)):
        assert 1 <= G <= most and ngroups == ceil(b, G), (r, b)
        assert 1 <= active <= min(grid, ngroups), (r, b)
        # groups a workgroup walks: one, or as few as the whole grid can have
        assert ceil(ngroups, active) <= max(1, 2 * ceil(b, most * grid)), (r, b, G, ngroups, active)
        if r >= 4 * b:   # dense: by the rows
            want = min(ceil(r, rows_each), grid, b)
            assert ceil(b, G) <= max(want, ceil(b, most)) and active >= min(want, ceil(b, ceil(b, want)))


@pytest.mark.parametrize("n_cand", [1, 40, 1000, 100_000])
def test_dis_ranges(split, n_cand):
    most = int(np.clip(ceil(2048, ceil(n_cand, 256)), 1, 4096))
    cases = [("d", r, b, most, 256, n_cand) for r in ROWS for b in BUCKETS]
    for (_, r, b, *_), (per,) in zip(cases, split(cases)):
        assert 1 <= per <= b and ceil(b, per) <= most, (r, b, per)
        assert per <= max(256, ceil(b, most)), (r, b, per)   # one chunk of buckets, or the ranges run out
        if r >= 8 * b and per > ceil(b, most):               # dense: a pass of 512 to 2048 terms
            assert min(b, 512 / 1.02 * b / r - 1) <= per <= 2048 / 1.02 * b / r, (r, b, per)


@pytest.mark.parametrize("waves", [12, 3072])
@pytest.mark.parametrize("cap", [40, 200, 400])
def test_inplace_items(split, waves, cap):
    cases = []
    for p in range(0, 28):
        for per in (0.01, 0.3, 1, 6, 20, 60, 300):      # terms a pair
            most = 1
            while most * 2 <= 32 and most * 2 * max(per, 2) <= 1.5 * cap:
                most *= 2
            cases.append(("i", int(per * (1 << p)), 1 << p, most, cap, waves))
    for (_, rows, pairs, most, *_), (n,) in zip(cases, split(cases)):
        assert 1 <= n <= most and n & (n - 1) == 0
        items, per = ceil(pairs, n), rows / pairs
        fits = [m for m in (1, 2, 4, 8, 16, 32) if m <= most and (m == 1 or m * per <= min(128, cap / 2))]
        if ceil(pairs, fits[-1]) <= waves:      # one round, of items as small as that allows
            assert items <= waves and (n == 1 or ceil(pairs, n // 2) > waves), (rows, pairs, most, n)
        elif n > 1:                             # at least two items a wave
            assert items >= 2 * waves, (rows, pairs, most, n)
        if items < 2 * waves and n > 1:         # never by items that may pass the stash
            assert n * per <= cap / 2, (rows, pairs, most, n)
        if items >= 4 * waves:                  # and no smaller than that needs
            assert n == most, (rows, pairs, most, n)


def test_doublings(split):
    cases = [("l", a, b, 0, 0, 0) for a in (1, 2, 3, 5, 8, 100, 12_345_678) for b in (1, 2, 3, 4, 7, 300, 301, 1 << 40)]
    for (_, a, b, *_), (e,) in zip(cases, split(cases)):
        assert e >= 0 and (e == 0 or a << e <= b) and a << (e + 1) > b, (a, b, e)
