// How the kernels that walk a store's bucket table share it among workgroups.
// Plain C++ (constexpr functions serve the device too), so that the rules can be
// checked on the host over all sizes.
//
// A workgroup walks its buckets in groups of at most as many as it has threads
// for, one group after another, and a group costs a chain of loads (about
// 2.6 us) even where its buckets are empty.  So the rows alone do not decide: an
// in-place store may have far more buckets than terms, and then there are as
// many workgroups as groups.  1000 two-word terms in 2^16 / 2^19 buckets: energy
// 32 / 39 us (393 / 3082 with the rows alone, and 48 / 50 with up to four groups a
// workgroup), angle gradient 38 / 63 us (519 / 2713), DIS of 40
// candidates 114 / 320 us (7540 / 25250).
#pragma once

#include <stdint.h>

namespace iqcc {

// Groups of G consecutive buckets; workgroup g of the `active` ones takes the
// groups g, g + active, ...  (a store has at most 2^28 buckets)
struct BucketSplit {
  int G, ngroups, active;
};

// One workgroup per rows_each rows or per group of `most` buckets, whichever
// are more, at most grid.
constexpr BucketSplit split_buckets(int64_t rows, int64_t buckets, int64_t grid, int64_t rows_each, int64_t most) {
  const int64_t by_rows = (rows + rows_each - 1) / rows_each;
  const int64_t by_buckets = (buckets + most - 1) / most;
  int64_t want64 = by_rows > by_buckets ? by_rows : by_buckets;
  want64 = want64 < 1 ? 1 : (want64 > grid ? grid : want64);
  // (32 bits: a 64-bit division is a good part of a microsecond on the device)
  const uint32_t B = (uint32_t)buckets, want = want64 > buckets ? B : (uint32_t)want64;
  uint32_t G = (B + want - 1) / want;
  G = G > (uint32_t)most ? (uint32_t)most : G;
  const uint32_t ngroups = (B + G - 1) / G;
  return {(int)G, (int)ngroups, (int)(ngroups < want ? ngroups : want)};
}

// Energy.  rows_each: a call over the stores of a 32-Hamiltonian batch takes
// 10.4 us with 512 rows, 10.3 with 1024, 11.5 with 2048.
constexpr int64_t kEnergyRows = 1024;
constexpr BucketSplit energy_buckets(int64_t rows, int64_t buckets, int64_t grid, int threads) {
  return split_buckets(rows, buckets, grid, kEnergyRows, threads);
}

// Angle gradient, a row per thread.
constexpr int kBwdGroup = 256;     // most buckets per group of one flat range
constexpr BucketSplit gradient_buckets(int64_t rows, int64_t buckets, int64_t grid, int threads) {
  return split_buckets(rows, buckets, grid, threads, kBwdGroup);
}

constexpr int kDisB = 256;          // threads per workgroup of the batched DIS kernel
constexpr int kDisR = 8;            // terms per lane of a full pass
constexpr int kDisChunk = kDisB;    // buckets whose prefix sums are staged at once
constexpr int kDisPass = kDisB * kDisR;
constexpr int kDisRun = 16;         // least candidates of a workgroup's run, if there are as many

// Buckets per term range of a batched DIS launch: as many as fill one pass (with
// 2 % to spare, so that uneven buckets seldom spill a few terms into a second
// pass: on 1e6 terms in 4096 buckets, ranges of 8.4 buckets took 2320 us, of 8
// 1902 us), but no more than max_ranges ranges; `fixed`: max_ranges ranges.
// Where that leaves CUs without a run of candidates, the ranges are halved, to
// 4 and to 2 terms a lane: then a workgroup's loads, not its candidates, are the
// time (200,000 two-word terms x 16 candidates 54 us with 98 ranges, 30 with
// 391; x 64, which fill the chip, 69 and 78).  And no more than one chunk of
// buckets.
constexpr int64_t dis_range_buckets(int64_t rows, int64_t buckets, int max_ranges, int fixed, int64_t n_cand,
                                    int n_cu) {
  const int64_t least = (buckets + max_ranges - 1) / max_ranges;
  if (fixed || rows <= 0) return least;
  int pass = kDisPass;
  while (pass > 2 * kDisB && (rows / pass + 1) * ((n_cand + kDisRun - 1) / kDisRun) < n_cu) pass /= 2;
  int64_t fill = (int64_t)((double)buckets * (pass / 1.02) / (double)rows);
  fill = fill > kDisChunk ? kDisChunk : fill;
  return fill < least ? least : (fill > buckets ? buckets : fill);
}

// floor(log2(v)), v >= 1
constexpr int log2_floor(uint64_t v) { return 63 - __builtin_clzll(v); }

// The largest e >= 0 with a 2^e <= b (0 if there is none); a, b >= 1 below 2^62.
constexpr int doublings(uint64_t a, uint64_t b) {
  int e = log2_floor(b) - log2_floor(a);
  if (e > 0 && a << e > b) --e;
  return e > 0 ? e : 0;
}

// Pairs per item of an in-place step of `rows` terms in `npairs` pairs (a power of
// two), as a power of two up to 2^most (whose anticommuting terms the stash of
// `cap` entries of a wave is expected to hold), for nw waves.  A wave's chain of loads, join and stores takes about as
// long for 6 terms as for the 128 that it loads at once.  So where items of at most
// that many, and of half the stash if all of them anticommute (a larger set goes
// to the store's pool, which costs more than a round), make one round of the
// waves, the smallest such are taken: 4096 buckets of 3 terms: 64 items of 32
// pairs on 64 waves 24 to 38 us a step, 2048 of one pair 13 us; 65536 buckets of 3
// two-word terms: 8192 items 51 us with the host's part, 2048 of 16 pairs 39.  Else
// at least two items a wave (2^18 buckets of 4 terms: 92 us with 4096 items for
// 3072 waves, 80 us with 8192).
// (No loops: every wave works this out before its first load.)
constexpr int item_pairs_log2(int64_t rows, int64_t npairs, int most, int cap, int64_t nw) {
  const int p = log2_floor(npairs);
  const int64_t terms = cap / 2 < 128 ? cap / 2 : 128;
  int one = doublings(rows > 0 ? rows : 1, terms * npairs);
  one = one < most ? one : most;
  const int round = p - log2_floor(nw);             // so that the items are no more than the waves
  if (round <= one) return round > 0 ? round : 0;
  const int two = p - log2_floor(2 * nw - 1) - 1;   // twice the waves or more
  return two < 0 ? 0 : (two < most ? two : most);
}

}  // namespace iqcc
