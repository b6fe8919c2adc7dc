// Term-limit compression: keep the M terms of largest |c| (the maximum-terms
// limit of the paper's Ru-catalyst runs, Results, next to the coefficient
// cutoff; ties broken by the smaller canonical key so that the kept set is
// unique).
//
// Radix selection on the IEEE bits of |c|, which order non-negative doubles
// like their values: six digit passes (11, 11, 11, 11, 11, 9 bits, most
// significant first) each build a histogram of the digit over the terms whose
// higher digits equal the prefix chosen so far, and pick the digit where the
// running count from the top reaches the number still needed.  After the first
// digit only the terms that share it can matter, so the second pass copies
// their |c| bits aside (into the output's arena, which holds nothing yet, at
// the rows of their bucket: no append counter) and the later passes read those
// alone.  If the second digit leaves few terms, one workgroup settles the other
// four from a list of them.  That fixes the threshold T (the M-th largest |c|),
// the number of terms above it and the number to take among the terms equal to
// T.  When not all ties are taken, the tie keys are collected (in the output's
// arena too) and the same selection runs on their canonical key words (x words,
// then z words, most significant first), from the bottom.  A last pass copies
// every bucket's kept terms, in input order, to the same rows of the output
// arena.
//
// A pass is one launch: the workgroup that adds its histogram last picks the
// digit.  A wavefront streams a bucket, several slices of 64 terms in flight,
// with no barrier (workgroups of 256 that scanned the bucket together, one
// append counter and a kernel per pick: 24, 40 and 81 us for the two full
// passes and the copy on 3e6 two-word terms and 40 us for the picks and later
// passes, now 17, 17, 48 and 16).  Bound: HBM in the copy, 80 bytes per kept term.
#include "iqcc_internal.h"

namespace iqcc {

constexpr int kSelBins = 2048;
constexpr int kSelBlock = 1024;   // few workgroups: each adds its bins to the same counters
constexpr int kSelWaves = kSelBlock / 64;

__device__ __forceinline__ uint64_t abs_bits(double c) {
  return (uint64_t)__double_as_longlong(c) & 0x7fffffffffffffffull;
}

// The digit at which the count reaches need, scanning from the largest digit
// down (descending) or from 0 up; count(d) gives a digit's terms (need >= 1 and
// need <= the sum).  Every thread of the workgroup calls and gets the result.
struct Pick {
  int digit;
  unsigned at;      // terms of the digit
  int64_t before;   // terms passed over
};

template <class Count>
__device__ Pick block_pick(int width, int descending, int64_t need, Count count) {
  __shared__ uint64_t scan_tmp[kSelWaves];
  __shared__ Pick found;
  const int nb = 1 << width;
  constexpr int kPer = kSelBins / kSelBlock;   // consecutive digits per thread
  unsigned v[kPer];
  uint64_t mine = 0;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int r = threadIdx.x * kPer + k;   // rank in scan order
    v[k] = r < nb ? count(descending ? nb - 1 - r : r) : 0u;
    mine += v[k];
  }
  uint64_t total;
  int64_t before = (int64_t)block_exclusive_scan_n<kSelWaves>(mine, scan_tmp, total);
  if (before < need && before + (int64_t)mine >= need) {   // one thread
    int k = 0;
    while (k < kPer - 1 && before + (int64_t)v[k] < need) before += v[k++];
    const int r = threadIdx.x * kPer + k;
    unsigned at = v[0];
#pragma unroll
    for (int j = 1; j < kPer; ++j) at = j == k ? v[j] : at;
    found = Pick{descending ? nb - 1 - r : r, at, before};
  }
  __syncthreads();
  const Pick p = found;
  __syncthreads();
  return p;
}

// True in every thread of the workgroup that arrives last.
__device__ bool block_arrive(double* slot) {
  __shared__ int s_last;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // every wave's stores and atomics are done
  __syncthreads();
  if (threadIdx.x < 64) {
    const bool last = finish_arrive(slot, blockIdx.x, gridDim.x);
    if (threadIdx.x == 0) s_last = last;
  }
  __syncthreads();
  return s_last != 0;
}

// Adds the workgroup's histogram h to hist; the workgroup that arrives last
// picks the digit and clears hist.  need >= 0 starts a selection of that many
// terms.
struct PickArgs {
  SelState* ss;
  unsigned* hist;
  double* slot;
  int64_t need;
  int width, descending, last, key_word;
};

__device__ void add_and_pick(const unsigned* h, const PickArgs& a) {
  __syncthreads();
  for (int i = threadIdx.x; i < kSelBins; i += kSelBlock)
    if (h[i]) atomicAdd(&a.hist[i], h[i]);
  if (!block_arrive(a.slot)) return;
  SelState* ss = a.ss;
  const bool start = a.need >= 0;
  const int64_t need = start ? a.need : ss->need;
  const Pick p = block_pick(a.width, a.descending, need, [&](int d) {
    const unsigned v = __hip_atomic_load(&a.hist[d], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    a.hist[d] = 0u;
    return v;
  });
  if (threadIdx.x) return;
  const uint64_t chosen = ((start ? 0ull : ss->prefix) << a.width) | (uint64_t)p.digit;
  ss->need = need - p.before;
  ss->passed = (start ? 0 : ss->passed) + p.before;
  ss->at = p.at;
  ss->prefix = a.last ? 0ull : chosen;
  if (start) {
    ss->key_mode = 0;
    ss->listed = 0;
    ss->done = 0;
  }
  if (a.last) {
    ss->done = 1;
    if (a.key_word < 0) {
      ss->T = chosen;
      ss->ties = p.at;
    } else {
      ss->kthr[a.key_word] = chosen;
      ss->key_mode = 1;
    }
  }
}

// Streams val rows off[b] .. off[b] + cnt[b] of every bucket, one wavefront per
// bucket, kSelU slices of 64 values loaded at a time: f(b, w, active, value) for
// each slice, in order, by whole wavefronts (active: the lane has a value), and
// end(b, w) after each bucket; w starts at 0 in every bucket and is f's to move.
constexpr int kSelU = 4;

template <class F, class E>
__device__ __forceinline__ void each_value(const uint64_t* val, const int64_t* cnt, const int64_t* off0, int m, F f,
                                           E end) {
  const int lane = threadIdx.x & 63;
  const int64_t B = 1ll << m;
  const int64_t step = (int64_t)gridDim.x * kSelWaves;
  int64_t b = (int64_t)blockIdx.x * kSelWaves + (threadIdx.x >> 6);
  int64_t n = b < B ? cnt[b] : 0, off = b < B ? off0[b] : 0;
  for (; b < B; b += step) {
    const bool more = b + step < B;
    const int64_t nn = more ? cnt[b + step] : 0, noff = more ? off0[b + step] : 0;
    int64_t w = 0;
    for (int64_t i0 = 0; i0 < n; i0 += 64 * kSelU) {
      uint64_t u[kSelU];
#pragma unroll
      for (int k = 0; k < kSelU; ++k) {
        const int64_t i = i0 + 64 * k + lane;
        u[k] = i < n ? val[off + i] : 0ull;
      }
#pragma unroll
      for (int k = 0; k < kSelU; ++k)
        if (i0 + 64 * k < n) f(off, w, i0 + 64 * k + lane < n, u[k]);
    }
    end(b, w);
    n = nn;
    off = noff;
  }
}

__device__ __forceinline__ uint64_t magnitude(uint64_t bits) { return bits & 0x7fffffffffffffffull; }

// First digit over every live term.  An invalid store, and one that needs no
// selection (all or none of its terms stay), is left alone: `keep` stands for
// the following passes and the copy, which the host launches with them.  It reads
// the state once, after the copy, and goes on only where the selection was not
// settled (a call that keeps every one of 1000 terms takes 41 us, 49 with
// the count read before and 53 with the state read before the copy).
__global__ __launch_bounds__(kSelBlock) void k_abs_hist(StoreDev st, int shift, PickArgs a) {
  __shared__ unsigned h[kSelBins];
  const int64_t n = *st.total;
  const int err = *st.err;
  const int keep = err ? kKeepInvalid : n <= a.need ? 1 : a.need == 0 ? -1 : 0;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    a.ss->n = n;
    a.ss->err = err;
    a.ss->keep = keep;
  }
  if (keep) return;
  for (int i = threadIdx.x; i < kSelBins; i += kSelBlock) h[i] = 0;
  __syncthreads();
  each_value((const uint64_t*)st.c, st.cnt, st.off, *st.m,
             [&](int64_t, int64_t&, bool active, uint64_t u) {
               if (active) atomicAdd(&h[magnitude(u) >> shift], 1u);
             },
             [](int64_t, int64_t) {});
  add_and_pick(h, a);
}

// Second digit: the histogram over the terms that share the first, whose |c|
// bits go to the first of their bucket's rows in cand, their number to ncand.
__global__ __launch_bounds__(kSelBlock) void k_abs_collect(StoreDev st, int shift, uint64_t* cand, int64_t* ncand,
                                                           PickArgs a) {
  __shared__ unsigned h[kSelBins];
  if (a.ss->keep) return;
  for (int i = threadIdx.x; i < kSelBins; i += kSelBlock) h[i] = 0;
  __syncthreads();
  const uint64_t prefix = a.ss->prefix;
  const uint64_t dmask = (1ull << a.width) - 1;
  each_value((const uint64_t*)st.c, st.cnt, st.off, *st.m,
             [&](int64_t off, int64_t& w, bool active, uint64_t bits) {
               const uint64_t u = magnitude(bits);
               const bool match = active && (u >> (shift + a.width)) == prefix;
               const uint64_t mask = __ballot(match);
               if (match) {
                 atomicAdd(&h[(u >> shift) & dmask], 1u);
                 cand[off + w + lanes_below(mask)] = u;
               }
               w += __popcll(mask);
             },
             [&](int64_t b, int64_t w) {
               if ((threadIdx.x & 63) == 0) ncand[b] = w;
             });
  add_and_pick(h, a);
}

static const int kDigitWidth[6] = {11, 11, 11, 11, 11, 9};
static const int kDigitShift[6] = {53, 42, 31, 20, 9, 0};

// The other four digits at once if the first two left at most kSelList terms
// (64 KB of LDS; four passes and one more synchronisation otherwise: 38 us
// against 16 on 3e6 terms): each workgroup lists its matches, the one that
// arrives last reads the whole list back and selects from it.
constexpr int kSelList = 8192;

__global__ __launch_bounds__(kSelBlock) void k_cand_finish(StoreDev st, const uint64_t* cand, const int64_t* ncand,
                                                           uint64_t* list, PickArgs a) {
  __shared__ uint64_t mine[kSelList];
  __shared__ unsigned h[kSelBins];
  __shared__ unsigned n_mine;
  __shared__ unsigned long long base;
  SelState* ss = a.ss;
  if (ss->keep || ss->at > kSelList) return;   // the same in every workgroup
  if (threadIdx.x == 0) n_mine = 0;
  __syncthreads();
  uint64_t prefix = ss->prefix;
  int shift = 64 - 22;
  each_value(cand, ncand, st.off, *st.m,
             [&](int64_t, int64_t&, bool active, uint64_t u) {
               if (active && (u >> shift) == prefix) mine[atomicAdd(&n_mine, 1u)] = u;
             },
             [](int64_t, int64_t) {});
  __syncthreads();
  if (threadIdx.x == 0 && n_mine) base = atomicAdd((unsigned long long*)&ss->listed, (unsigned long long)n_mine);
  __syncthreads();
  for (unsigned i = threadIdx.x; i < n_mine; i += kSelBlock)
    __hip_atomic_store(&list[base + i], mine[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (!block_arrive(a.slot)) return;
  const int n = (int)ss->at;
  for (int i = threadIdx.x; i < n; i += kSelBlock)
    mine[i] = __hip_atomic_load(&list[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  int64_t need = ss->need, passed = ss->passed;
  unsigned at = 0;
  while (shift > 0) {
    const int width = shift < 11 ? shift : 11;
    const uint64_t dmask = (1ull << width) - 1;
    for (int i = threadIdx.x; i < kSelBins; i += kSelBlock) h[i] = 0;
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += kSelBlock)
      if ((mine[i] >> shift) == prefix) atomicAdd(&h[(mine[i] >> (shift - width)) & dmask], 1u);
    __syncthreads();
    const Pick p = block_pick(width, 1, need, [&](int d) { return h[d]; });
    need -= p.before;
    passed += p.before;
    at = p.at;
    prefix = (prefix << width) | (uint64_t)p.digit;
    shift -= width;
  }
  if (threadIdx.x) return;
  ss->need = need;
  ss->passed = passed;
  ss->at = ss->ties = at;
  ss->T = prefix;
  ss->prefix = 0;
  ss->listed = 0;   // (counts the ties' keys next)
  ss->done = 1;
}

// Later digits one by one, over the collected |c| bits.
__global__ __launch_bounds__(kSelBlock) void k_cand_hist(StoreDev st, const uint64_t* cand, const int64_t* ncand,
                                                         int shift, PickArgs a) {
  __shared__ unsigned h[kSelBins];
  for (int i = threadIdx.x; i < kSelBins; i += kSelBlock) h[i] = 0;
  __syncthreads();
  const uint64_t prefix = a.ss->prefix;
  const uint64_t dmask = (1ull << a.width) - 1;
  each_value(cand, ncand, st.off, *st.m,
             [&](int64_t, int64_t&, bool active, uint64_t u) {
               if (active && (u >> (shift + a.width)) == prefix) atomicAdd(&h[(u >> shift) & dmask], 1u);
             },
             [](int64_t, int64_t) {});
  add_and_pick(h, a);
}

// Canonical key word q of a term: x[W-1], ..., x[0], z[W-1], ..., z[0].
template <int W>
__device__ __forceinline__ uint64_t canon_word(const StoreDev& st, int64_t row, int q) {
  return q < W ? st.x[(W - 1 - q) * st.cap + row] : st.z[(2 * W - 1 - q) * st.cap + row];
}

// Keys of the terms with |c| bits == T, as the first rows of `keys`.
template <int W>
__global__ __launch_bounds__(kBlock) void k_collect_ties(StoreDev st, SelState* ss, StoreDev keys) {
  const uint64_t T = ss->T;
  const int64_t B = 1ll << *st.m;
  for (int64_t b = blockIdx.x; b < B; b += gridDim.x) {
    const int64_t n = st.cnt[b], off = st.off[b];
    for (int64_t i = threadIdx.x; i < n; i += kBlock) {
      if (abs_bits(st.c[off + i]) != T) continue;
      const int64_t r = (int64_t)atomicAdd((unsigned long long*)&ss->listed, 1ull);
      if (r < keys.cap) {
#pragma unroll
        for (int w = 0; w < W; ++w) {
          keys.x[w * keys.cap + r] = st.x[w * st.cap + off + i];
          keys.z[w * keys.cap + r] = st.z[w * st.cap + off + i];
        }
      }
    }
  }
}

// Digit of key word q over the tie keys whose earlier words equal kthr[0..q)
// and whose bits of word q above shift + width equal the prefix.
template <int W>
__global__ __launch_bounds__(kSelBlock) void k_key_hist(StoreDev keys, int64_t n, int q, int shift, int first,
                                                        PickArgs a) {
  __shared__ unsigned h[kSelBins];
  for (int i = threadIdx.x; i < kSelBins; i += kSelBlock) h[i] = 0;
  __syncthreads();
  const uint64_t dmask = (1ull << a.width) - 1;
  for (int64_t i = blockIdx.x * (int64_t)kSelBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kSelBlock) {
    bool match = true;
    for (int p = 0; p < q; ++p) match = match && canon_word<W>(keys, i, p) == a.ss->kthr[p];
    const uint64_t word = canon_word<W>(keys, i, q);
    if (match && (first || (word >> (shift + a.width)) == a.ss->prefix))
      atomicAdd(&h[(word >> shift) & dmask], 1u);
  }
  add_and_pick(h, a);
}

// Copy the kept terms of every bucket, in input order, to the same rows of
// the output arena; the output keeps the input's bucket table shape.  One
// wavefront per bucket (positions from ballots); the workgroup that arrives
// last writes the output's counters.  keep: see launch_select_compact.
template <int W>
__global__ __launch_bounds__(kBlock) void k_select_compact(StoreDev in, StoreDev out, const SelState* ss,
                                                           int keep, double* slot) {
  constexpr int U = 2;
  __shared__ int64_t s_kept[kWaves];
  __shared__ int s_last;
  __shared__ uint64_t scan_tmp[kWaves];
  if (keep == kKeepAuto) {
    if (ss->keep == kKeepInvalid || !sel_settled(*ss)) return;
    keep = ss->keep;
  }
  const uint64_t T = keep == 0 ? ss->T : 0ull;
  const int key_mode = keep == 0 ? ss->key_mode : 0;
  const int m = *in.m;
  const int64_t B = 1ll << m;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int64_t kept = 0;
  for (int64_t b = (int64_t)blockIdx.x * kWaves + wave; b < B; b += (int64_t)gridDim.x * kWaves) {
    const int64_t n = in.cnt[b], off = in.off[b];
    int64_t w = 0;
    for (int64_t i0 = 0; i0 < n && keep >= 0; i0 += 64 * U) {
      uint64_t kx[U][W], kz[U][W];
      double kc[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t i = i0 + 64 * u + lane;
        if (i < n) load_key<W>(in, off + i, kx[u], kz[u], kc[u]);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        bool kept_here = i0 + 64 * u + lane < n;
        if (kept_here && !keep) {
          const uint64_t v = abs_bits(kc[u]);
          kept_here = v >= T;
          if (v == T && key_mode) {
            // keep ties whose canonical key is <= kthr
            bool decided = false;
#pragma unroll
            for (int q = 0; q < 2 * W; ++q) {
              const uint64_t word = q < W ? kx[u][W - 1 - q] : kz[u][2 * W - 1 - q];
              if (!decided && word != ss->kthr[q]) {
                kept_here = word < ss->kthr[q];
                decided = true;
              }
            }
          }
        }
        const uint64_t mask = __ballot(kept_here);
        if (kept_here) store_key<W>(out, off + w + lanes_below(mask), kx[u], kz[u], kc[u]);
        w += __popcll(mask);
      }
    }
    if (lane == 0) {
      out.off[b] = off;
      out.cnt[b] = w;
      out.lim[b] = off + n;   // the input bucket's rows
    }
    kept += w;
  }
  if (lane == 0) s_kept[wave] = kept;
  __syncthreads();
  if (wave == 0) {
    if (lane == 0) {
      int64_t k = 0;
      for (int i = 0; i < kWaves; ++i) k += s_kept[i];
      finish_put(slot, blockIdx.x, __longlong_as_double(k));
    }
    const bool last = finish_arrive(slot, blockIdx.x, gridDim.x);
    if (lane == 0) s_last = last;
  }
  __syncthreads();
  if (!s_last) return;
  uint64_t mine = 0, total;
  for (unsigned i = threadIdx.x; i < gridDim.x; i += kBlock) mine += (uint64_t)__double_as_longlong(finish_get(slot, i));
  block_exclusive_scan(mine, scan_tmp, total);
  if (threadIdx.x == 0) {
    *out.m = m;
    *out.total = (int64_t)total;
    *out.top = *in.top;
    *out.err = 0;
    out.stats[0] = out.stats[1] = 0;
  }
}

void launch_abs_select(const StoreDev& st, SelState* ss, unsigned* hist, int n_cu, int64_t need, const StoreDev& tmp,
                       double* slot, hipStream_t s) {
  for (int p = 0; p < 3; ++p) {
    const PickArgs a{ss, hist, slot, p == 0 ? need : -1, kDigitWidth[p], 1, 0, -1};
    if (p == 0) hipLaunchKernelGGL(k_abs_hist, dim3(n_cu), dim3(kSelBlock), 0, s, st, kDigitShift[p], a);
    else if (p == 1) hipLaunchKernelGGL(k_abs_collect, dim3(n_cu), dim3(kSelBlock), 0, s, st, kDigitShift[p], tmp.x, tmp.cnt, a);
    else hipLaunchKernelGGL(k_cand_finish, dim3(n_cu), dim3(kSelBlock), 0, s, st, tmp.x, tmp.cnt, tmp.z, a);
  }
}

void launch_abs_select_rest(const StoreDev& st, SelState* ss, unsigned* hist, int n_cu, const StoreDev& tmp,
                            double* slot, hipStream_t s) {
  for (int p = 2; p < 6; ++p) {
    const PickArgs a{ss, hist, slot, -1, kDigitWidth[p], 1, p == 5, -1};
    hipLaunchKernelGGL(k_cand_hist, dim3(n_cu), dim3(kSelBlock), 0, s, st, tmp.x, tmp.cnt, kDigitShift[p], a);
  }
}

template <int W>
static void launch_ties_w(const StoreDev& st, const StoreDev& keys, int64_t n, SelState* ss, unsigned* hist, int n_cu,
                          double* slot, hipStream_t s) {
  hipLaunchKernelGGL(k_collect_ties<W>, dim3(4 * n_cu), dim3(kBlock), 0, s, st, ss, keys);
  const int64_t g = (n + kSelBlock - 1) / kSelBlock;
  const int grid = (int)(g < 1 ? 1 : g > 256 ? 256 : g);
  for (int q = 0; q < 2 * W; ++q)
    for (int p = 0; p < 6; ++p) {
      // (need goes on from the number of ties to take; the prefix starts anew per word)
      const PickArgs a{ss, hist, slot, -1, kDigitWidth[p], 0, p == 5, q};
      hipLaunchKernelGGL(k_key_hist<W>, dim3(grid), dim3(kSelBlock), 0, s, keys, n, q, kDigitShift[p], p == 0, a);
    }
}

void launch_select_ties(int W, const StoreDev& st, const StoreDev& keys, int64_t n, SelState* ss, unsigned* hist,
                        int n_cu, double* slot, hipStream_t s) {
  switch (W) {
    case 1: launch_ties_w<1>(st, keys, n, ss, hist, n_cu, slot, s); break;
    case 2: launch_ties_w<2>(st, keys, n, ss, hist, n_cu, slot, s); break;
    case 3: launch_ties_w<3>(st, keys, n, ss, hist, n_cu, slot, s); break;
    default: launch_ties_w<4>(st, keys, n, ss, hist, n_cu, slot, s); break;
  }
}

void launch_select_compact(int W, const StoreDev& in, const StoreDev& out, const SelState* ss, int keep, int grid,
                           double* slot, hipStream_t s) {
  switch (W) {
    case 1: hipLaunchKernelGGL(k_select_compact<1>, dim3(grid), dim3(kBlock), 0, s, in, out, ss, keep, slot); break;
    case 2: hipLaunchKernelGGL(k_select_compact<2>, dim3(grid), dim3(kBlock), 0, s, in, out, ss, keep, slot); break;
    case 3: hipLaunchKernelGGL(k_select_compact<3>, dim3(grid), dim3(kBlock), 0, s, in, out, ss, keep, slot); break;
    default: hipLaunchKernelGGL(k_select_compact<4>, dim3(grid), dim3(kBlock), 0, s, in, out, ss, keep, slot); break;
  }
}

}  // namespace iqcc
