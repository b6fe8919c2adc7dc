// Kernels of one iQCC iteration (Sec. II, iterative procedure) beyond the
// dressing step itself:
//   * the distinct flip sets of a Hamiltonian (x parts of its terms, App. A: DIS
//     candidates must share the flip set of some term) and the candidates on
//     them, one per qubit of a set: Y there, X on the rest;
//   * the candidates of largest |g|;
//   * the two sums over the terms that anticommute with a generator P that fix
//     its single-generator energy E(tau) = a + b cos(tau) + c sin(tau) (Eq. 5):
//     b = sum of c_K <Omega|K|Omega> (Eq. 3 restricted) and c = the DIS gradient
//     of P (Eq. 7).
// The iteration keeps flip sets, candidates, gradients and the selection on the
// device: the host sees two counts, the selected generators and, per step, b, c
// and the energy.
#include "iqcc_internal.h"

#pragma clang fp contract(off)

namespace iqcc {

// Distinct flip sets with 1 <= |F| <= w_max, appended to fx (planes of `ld`) in
// no particular order: every qualifying term looks for its set in an open
// hash table of arena rows (tab, all bits set when empty, a power of two above
// the number of terms); the one whose row gets into the table appends the set.
// count[0] = sets, count[1] = their qubits in all (one candidate each).
template <int W>
__global__ __launch_bounds__(kBlock) void k_flip_unique(StoreDev st, int w_max, unsigned long long* tab,
                                                        uint64_t tmask, uint64_t* fx, int64_t ld,
                                                        unsigned long long* count) {
  const int lane = threadIdx.x & 63;
  const int64_t B = 1ll << *st.m;
  for (int64_t b = blockIdx.x; b < B; b += gridDim.x) {
    const int64_t n = st.cnt[b], off = st.off[b];
    for (int64_t i0 = (threadIdx.x & ~63); i0 < n; i0 += kBlock) {   // wave-uniform
      const int64_t i = i0 + lane;
      uint64_t kx[W];
      int wt = 0;
#pragma unroll
      for (int w = 0; w < W; ++w) {
        kx[w] = i < n ? st.x[w * st.cap + off + i] : 0ull;
        wt += __popcll(kx[w]);
      }
      bool mine = false;
      if (wt >= 1 && wt <= w_max) {
        uint64_t zero[W] = {};
        uint64_t h = table_hash<W>(kx, zero) & tmask;
        for (;;) {
          unsigned long long r = __hip_atomic_load(&tab[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (r == ~0ull) {
            r = atomicCAS(&tab[h], ~0ull, (unsigned long long)(off + i));
            if (r == ~0ull) {
              mine = true;
              break;
            }
          }
          bool eq = true;
#pragma unroll
          for (int w = 0; w < W; ++w) eq = eq && st.x[w * st.cap + (int64_t)r] == kx[w];
          if (eq) break;
          h = (h + 1) & tmask;
        }
      }
      const uint64_t mask = __ballot(mine);
      if (mask == 0) continue;
      int q = mine ? wt : 0;
#pragma unroll
      for (int d = 32; d >= 1; d >>= 1) q += __shfl_xor(q, d, 64);
      unsigned long long base = 0;
      if (lane == 0) {
        base = atomicAdd(&count[0], (unsigned long long)__popcll(mask));
        atomicAdd(&count[1], (unsigned long long)q);
      }
      base = wave_bcast0(base);
      if (mine) {
        const int64_t r = (int64_t)base + lanes_below(mask);
#pragma unroll
        for (int w = 0; w < W; ++w) fx[w * ld + r] = kx[w];
      }
    }
  }
}

__global__ void k_fill_table(unsigned long long* tab, int64_t n, unsigned long long* count) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    tab[i] = ~0ull;
  if (blockIdx.x == 0 && threadIdx.x < 3) count[threadIdx.x] = 0ull;
}

void launch_flip_unique(int W, const StoreDev& st, int w_max, unsigned long long* tab, int64_t table, uint64_t* fx,
                        int64_t ld, unsigned long long* count, int grid, hipStream_t s) {
  int64_t fb = (table + kBlock - 1) / kBlock;
  hipLaunchKernelGGL(k_fill_table, dim3((unsigned)(fb > 4096 ? 4096 : fb)), dim3(kBlock), 0, s, tab, table, count);
  const uint64_t mask = (uint64_t)table - 1;
  switch (W) {
    case 1: hipLaunchKernelGGL(k_flip_unique<1>, dim3(grid), dim3(kBlock), 0, s, st, w_max, tab, mask, fx, ld, count); break;
    case 2: hipLaunchKernelGGL(k_flip_unique<2>, dim3(grid), dim3(kBlock), 0, s, st, w_max, tab, mask, fx, ld, count); break;
    case 3: hipLaunchKernelGGL(k_flip_unique<3>, dim3(grid), dim3(kBlock), 0, s, st, w_max, tab, mask, fx, ld, count); break;
    default: hipLaunchKernelGGL(k_flip_unique<4>, dim3(grid), dim3(kBlock), 0, s, st, w_max, tab, mask, fx, ld, count); break;
  }
}

// Candidates (planes of nc) of nf flip sets, a set's candidates together, in
// ascending order of the Y's qubit; count[2] is the append counter.
template <int W>
__global__ __launch_bounds__(kBlock) void k_candidates(const uint64_t* fx, int64_t ld, int64_t nf, uint64_t* cx,
                                                       uint64_t* cz, int64_t nc, unsigned long long* count) {
  for (int64_t f = blockIdx.x * (int64_t)kBlock + threadIdx.x; f < nf; f += (int64_t)gridDim.x * kBlock) {
    uint64_t x[W];
    int wt = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      x[w] = fx[w * ld + f];
      wt += __popcll(x[w]);
    }
    int64_t r = (int64_t)atomicAdd(&count[2], (unsigned long long)wt);
#pragma unroll
    for (int w = 0; w < W; ++w) {
      for (uint64_t v = x[w]; v; v &= v - 1, ++r) {
#pragma unroll
        for (int u = 0; u < W; ++u) {
          cx[u * nc + r] = x[u];
          cz[u * nc + r] = u == w ? v & (~v + 1) : 0ull;
        }
      }
    }
  }
}

void launch_candidates(int W, const uint64_t* fx, int64_t ld, int64_t nf, uint64_t* cx, uint64_t* cz, int64_t nc,
                       unsigned long long* count, hipStream_t s) {
  int64_t b = (nf + kBlock - 1) / kBlock;
  if (b > 4096) b = 4096;
  switch (W) {
    case 1: hipLaunchKernelGGL(k_candidates<1>, dim3((unsigned)b), dim3(kBlock), 0, s, fx, ld, nf, cx, cz, nc, count); break;
    case 2: hipLaunchKernelGGL(k_candidates<2>, dim3((unsigned)b), dim3(kBlock), 0, s, fx, ld, nf, cx, cz, nc, count); break;
    case 3: hipLaunchKernelGGL(k_candidates<3>, dim3((unsigned)b), dim3(kBlock), 0, s, fx, ld, nf, cx, cz, nc, count); break;
    default: hipLaunchKernelGGL(k_candidates<4>, dim3((unsigned)b), dim3(kBlock), 0, s, fx, ld, nf, cx, cz, nc, count); break;
  }
}

// The k candidates of largest |g| (equal |g|: ascending canonical key; a
// gradient that is no number ranks last), for few of them, one workgroup: every thread keeps
// the best of its share that has not been taken, a tree over the workgroup
// finds the best of those, and only the thread that held it looks for its
// next.  The order is total (candidates are distinct), so "not taken" is
// "after the last one taken".  out: k rows {g, x words, z words}.  A pick takes
// 8 us among 12,000 candidates, so more than kTopCandidates are ranked by the
// host.
constexpr int kTopBlock = 1024;
static_assert(kTopBlock / 64 == 16, "the second tree spans 16 waves");

template <int W>
__global__ __launch_bounds__(kTopBlock) void k_top_candidates(const double* g, const uint64_t* cx, const uint64_t* cz,
                                                              int64_t nc, int k, double* out) {
  __shared__ int64_t s_best[kTopBlock / 64];
  __shared__ double s_val[kTopBlock / 64];
  __shared__ int64_t s_taken;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  auto rank = [&](int64_t i) {
    const double v = fabs(g[i]);
    return v == v ? v : -1.0;
  };
  // candidate a of rank va comes before candidate b of rank vb (none: -1 of
  // rank -2); keys are read only where the ranks are equal
  auto before = [&](double va, int64_t a, double vb, int64_t b) {
    if (va != vb || a < 0 || b < 0) return va > vb;
    for (int w = W - 1; w >= 0; --w)
      if (cx[w * nc + a] != cx[w * nc + b]) return cx[w * nc + a] < cx[w * nc + b];
    for (int w = W - 1; w >= 0; --w)
      if (cz[w * nc + a] != cz[w * nc + b]) return cz[w * nc + a] < cz[w * nc + b];
    return false;
  };
  int64_t mine = -1;
  double vmine = -2.0;
  auto best_after = [&](int64_t last, double vl) {   // last -1: the best of all
    int64_t best = -1;
    double vb = -2.0;
    for (int64_t i = threadIdx.x; i < nc; i += kTopBlock) {
      const double v = rank(i);
      if (v < vb || (last >= 0 && !before(vl, last, v, i))) continue;
      if (before(v, i, vb, best)) {
        best = i;
        vb = v;
      }
    }
    mine = best;
    vmine = vb;
  };
  best_after(-1, 0.0);
  for (int r = 0; r < k; ++r) {
    int64_t b = mine;
    double vb = vmine;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
      const int64_t o = (int64_t)__shfl_xor((long long)b, d, 64);
      const double vo = __shfl_xor(vb, d, 64);
      if (before(vo, o, vb, b)) { b = o; vb = vo; }
    }
    if (lane == 0) {
      s_best[wave] = b;
      s_val[wave] = vb;
    }
    __syncthreads();
    if (wave == 0) {
      b = lane < kTopBlock / 64 ? s_best[lane] : -1;
      vb = lane < kTopBlock / 64 ? s_val[lane] : -2.0;
#pragma unroll
      for (int d = 8; d >= 1; d >>= 1) {
        const int64_t o = (int64_t)__shfl_xor((long long)b, d, 64);
        const double vo = __shfl_xor(vb, d, 64);
        if (before(vo, o, vb, b)) { b = o; vb = vo; }
      }
      if (lane == 0) s_taken = b;   // k <= nc: there is one
      double* row = out + (int64_t)r * (1 + 2 * W);
      b = (int64_t)wave_bcast0((unsigned long long)b);
      if (lane == 0) row[0] = g[b];
      if (lane >= 1 && lane <= W) row[lane] = __longlong_as_double((long long)cx[(lane - 1) * nc + b]);
      if (lane > W && lane <= 2 * W) row[lane] = __longlong_as_double((long long)cz[(lane - 1 - W) * nc + b]);
    }
    __syncthreads();
    if (s_taken == mine && mine >= 0) best_after(mine, vmine);
  }
}

void launch_top_candidates(int W, const double* g, const uint64_t* cx, const uint64_t* cz, int64_t nc, int k,
                           double* out, hipStream_t s) {
  switch (W) {
    case 1: hipLaunchKernelGGL(k_top_candidates<1>, dim3(1), dim3(kTopBlock), 0, s, g, cx, cz, nc, k, out); break;
    case 2: hipLaunchKernelGGL(k_top_candidates<2>, dim3(1), dim3(kTopBlock), 0, s, g, cx, cz, nc, k, out); break;
    case 3: hipLaunchKernelGGL(k_top_candidates<3>, dim3(1), dim3(kTopBlock), 0, s, g, cx, cz, nc, k, out); break;
    default: hipLaunchKernelGGL(k_top_candidates<4>, dim3(1), dim3(kTopBlock), 0, s, g, cx, cz, nc, k, out); break;
  }
}

// *b_out = sum over the terms K that anticommute with P of c_K <K>, and
// (c_out not null) *c_out = sum of +-c_K <K P>, + for K P = i (K ^ P) and - for
// K P = -i (K ^ P).  One pass and one launch: the two products share the
// groups P does not touch, the table is built in every workgroup, and the
// workgroup that arrives last adds the sums in a fixed order.  (Table, sum of
// b, reduction, table, counter and the plain one-candidate gradient were six
// launches: 49 us on 12,007 to 40,000 one-word terms, this takes 10 us.)  C: with
// the second sum; without it only <K> is formed (3e6 one-word terms 64 -> 58 us,
// 3e5 four-word terms in 2^15 bucket regions 401 -> 367).
__device__ __forceinline__ void anti_total(const double* slot, unsigned active, double* red, double* b_out,
                                           double* c_out) {
  double tb = 0.0, tc = 0.0;
  for (unsigned i = threadIdx.x; i < active; i += kBlock) {
    tb += finish_get(slot, i);
    if (c_out) tc += finish_get(slot, active + i);
  }
  tb = block_sum(tb, red);
  if (c_out) tc = block_sum(tc, red);
  if (threadIdx.x == 0) {
    *b_out = tb;
    if (c_out) *c_out = tc;
  }
}

// The second launch of a call without a slot of its stream.
__global__ __launch_bounds__(kBlock) void k_anti_total(StoreDev st, unsigned grid, const double* slot, double* b_out,
                                                       double* c_out) {
  __shared__ double red[kWaves];
  const int64_t B = 1ll << *st.m;
  anti_total(slot, B < grid ? (unsigned)B : grid, red, b_out, c_out);
}

template <int W, bool C>
__global__ __launch_bounds__(kBlock) void k_anti_sums(StoreDev st, Entangler P, int nq, const double* theta,
                                                      const double* phi, SumSlot sums, double* b_out, double* c_out) {
  __shared__ double lut[W * kGroupsPerWord * kLutEntries];
  __shared__ double fq[256 * W];
  __shared__ double red[kWaves];
  __shared__ int s_last;
  const int64_t B = 1ll << *st.m;
  const unsigned active = B < gridDim.x ? (unsigned)B : gridDim.x;   // workgroups with a bucket
  if (blockIdx.x >= active) return;
  build_group_table<W, kBlock>(lut, fq, nq, theta, phi);
  double sb = 0.0, sc = 0.0;
  for (int64_t b = blockIdx.x; b < B; b += active) {
    const int64_t n = st.cnt[b], off = st.off[b];
    for (int64_t i = threadIdx.x; i < n; i += kBlock) {
      uint64_t kx[W], kz[W];
#pragma unroll
      for (int w = 0; w < W; ++w) {
        kx[w] = st.x[w * st.cap + off + i];
        kz[w] = st.z[w * st.cap + off + i];
      }
      double c = 0.0;
      if (C) c = st.c[off + i];   // (beside the key's test)
      if (!anticommutes<W>(kx, kz, P.px, P.pz)) continue;
      if constexpr (C) {
        double ek, ekp;
        expect_split<W>(lut, P, kx, kz, ek, ekp);
        sb += c * ek;
        sc += product_phase<W>(kx, kz, P.px, P.pz) == 1 ? c * ekp : -(c * ekp);
      } else {
        sb += st.c[off + i] * expect_lut<W>(lut, kx, kz);
      }
    }
  }
  sb = block_sum(sb, red);
  if (C) sc = block_sum(sc, red);
  if (threadIdx.x < 64) {
    if (threadIdx.x == 0) {
      finish_put(sums.slot, blockIdx.x, sb);
      if (C) finish_put(sums.slot, active + blockIdx.x, sc);
    }
    const bool last = sums.single && finish_arrive(sums.slot, blockIdx.x, active);
    if (threadIdx.x == 0) s_last = last;
  }
  __syncthreads();
  if (s_last) anti_total(sums.slot, active, red, b_out, c_out);
}

template <int W>
static void launch_anti_w(const StoreDev& st, const Entangler& P, int nq, int grid, const double* theta,
                          const double* phi, const SumSlot& slot, double* b_out, double* c_out, hipStream_t s) {
  if (c_out)
    hipLaunchKernelGGL((k_anti_sums<W, true>), dim3(grid), dim3(kBlock), 0, s, st, P, nq, theta, phi, slot, b_out, c_out);
  else
    hipLaunchKernelGGL((k_anti_sums<W, false>), dim3(grid), dim3(kBlock), 0, s, st, P, nq, theta, phi, slot, b_out, c_out);
}

void launch_anti_sums(int W, const StoreDev& st, const Entangler& P, int nq, int grid, const double* theta,
                      const double* phi, const SumSlot& slot, double* b_out, double* c_out, hipStream_t s) {
  switch (W) {
    case 1: launch_anti_w<1>(st, P, nq, grid, theta, phi, slot, b_out, c_out, s); break;
    case 2: launch_anti_w<2>(st, P, nq, grid, theta, phi, slot, b_out, c_out, s); break;
    case 3: launch_anti_w<3>(st, P, nq, grid, theta, phi, slot, b_out, c_out, s); break;
    default: launch_anti_w<4>(st, P, nq, grid, theta, phi, slot, b_out, c_out, s); break;
  }
  if (!slot.single)
    hipLaunchKernelGGL(k_anti_total, dim3(1), dim3(kBlock), 0, s, st, (unsigned)grid, slot.slot, b_out, c_out);
}

}  // namespace iqcc
