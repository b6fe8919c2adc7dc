// DIS gradient screening (Sec. II, Eq. 7; App. A):
//   g_a = Im <Omega| H P_a |Omega> = sum_k c_k Im(i^e) <Q_k>,  P_k P_a = i^e Q_k,
// so only terms that anticommute with P_a contribute, with +<Q_k> for e = 1
// and -<Q_k> for e = 3.
//
// Batched form: the QMF state is a product state, so for a term K and a
// candidate P_a the ratio <Q>/<K> (Q = K P_a) only involves the qubits in the
// support of P_a.  A table per (qubit, Pauli of P_a there, Pauli of K there)
// gives the factor ratio b_q(Q)/b_q(K), with the sign of the qubit's phase that
// counting leaves open (below); each term carries PK = the product of its
// non-zero qubit factors, and where a state has factors that are exactly zero
// also which of its qubits have one: then <Q> = PK * prod(ratios) when every
// zero factor of K lies in the support of P_a, else 0.  One table lookup per
// support qubit and term, no division in the loop and no special case at zero
// factors.  Plain form: one launch per candidate streaming all terms
// (reference form).
#include "iqcc_internal.h"
#include "work_split.h"

#pragma clang fp contract(off)

namespace iqcc {

constexpr int kDisWaves = kDisB / 64;
constexpr int kDisTile = 256;       // candidates staged at once

// Spread the 16 bits of v to the even bits of a 32-bit word.
__device__ __forceinline__ uint32_t spread16(uint32_t v) {
  v &= 0xffffu;
  v = (v | (v << 8)) & 0x00ff00ffu;
  v = (v | (v << 4)) & 0x0f0f0f0fu;
  v = (v | (v << 2)) & 0x33333333u;
  v = (v | (v << 1)) & 0x55555555u;
  return v;
}

// Sum over the 64 lanes of a wave with DPP moves (no LDS traffic); the total
// lands in lane 63.  Fixed pairing order, so the result is reproducible.
__device__ __forceinline__ double dpp_f64(double v, int ctrl_sel) {
  const uint64_t u = __double_as_longlong(v);
  int lo = (int)(uint32_t)u, hi = (int)(uint32_t)(u >> 32);
  switch (ctrl_sel) {   // constant after inlining
    case 0: lo = __builtin_amdgcn_mov_dpp(lo, 0xB1, 0xF, 0xF, false);   // quad_perm 1,0,3,2
            hi = __builtin_amdgcn_mov_dpp(hi, 0xB1, 0xF, 0xF, false); break;
    case 1: lo = __builtin_amdgcn_mov_dpp(lo, 0x4E, 0xF, 0xF, false);   // quad_perm 2,3,0,1
            hi = __builtin_amdgcn_mov_dpp(hi, 0x4E, 0xF, 0xF, false); break;
    case 2: lo = __builtin_amdgcn_mov_dpp(lo, 0x141, 0xF, 0xF, false);  // row_half_mirror
            hi = __builtin_amdgcn_mov_dpp(hi, 0x141, 0xF, 0xF, false); break;
    case 3: lo = __builtin_amdgcn_mov_dpp(lo, 0x140, 0xF, 0xF, false);  // row_mirror
            hi = __builtin_amdgcn_mov_dpp(hi, 0x140, 0xF, 0xF, false); break;
    case 4: lo = __builtin_amdgcn_update_dpp(0, lo, 0x142, 0xA, 0xF, false);  // row_bcast:15 -> rows 1, 3
            hi = __builtin_amdgcn_update_dpp(0, hi, 0x142, 0xA, 0xF, false); break;
    default: lo = __builtin_amdgcn_update_dpp(0, lo, 0x143, 0xC, 0xF, false); // row_bcast:31 -> rows 2, 3
             hi = __builtin_amdgcn_update_dpp(0, hi, 0x143, 0xC, 0xF, false); break;
  }
  return __longlong_as_double((long long)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo));
}

__device__ __forceinline__ double wave_sum_to_lane63(double v) {
  v += dpp_f64(v, 0);   // pairs within quads
  v += dpp_f64(v, 1);   // quads: every lane holds its quad's sum
  v += dpp_f64(v, 2);   // half rows
  v += dpp_f64(v, 3);   // rows of 16
  v += dpp_f64(v, 4);   // rows 1 and 3 add rows 0 and 2 (other rows add +0)
  v += dpp_f64(v, 5);   // rows 2 and 3 add rows 0..1
  return v;
}

template <int W>
struct DisShared {
  static constexpr int NQ = 64 * W, NS = 4 * W;   // NS: 16-qubit slots
  double ent[NQ * 16];       // [q][p][k]: signed factor ratios (p, k below)
  double pair[NQ / 2 * 16];  // [q / 2][codes of q, q + 1]: product of the non-zero factors
  uint32_t sw[kDisTile * NS];   // candidates as slot words
  double acc[kDisWaves][kDisTile];   // first the factors b_q(k), [q][k]
  int64_t boff[kDisChunk];
  int64_t pre[kDisChunk + 1];
  uint64_t scan_tmp[kDisWaves];
  uint32_t zero[3][NS];      // qubits (even bits of a slot word) whose X, Z, Y factor is exactly 0
};

// Terms r * kDisB + threadIdx.x (r < R) of a pass against `ncand` staged
// candidates.  A term is held as slot words: 16 qubits each, bit 2j the x bit
// and bit 2j + 1 the z bit of qubit j; a candidate's slot words hold its z bit
// at 2j and its x bit at 2j + 1, so that code & sw has one bit per
// anticommuting factor (and two where both are Y, whose ratio carries the sign
// -1 that the second bit would wrongly bring).  With n such bits and the signs
// in the ratios, i^e = i^n, so the pair counts with +1 for n = 1 and -1 for
// n = 3 (mod 4).
// The candidate loop is uniform: slot words sit in scalar registers, the
// support is walked with s_ff1, and every step issues R independent lookups.
template <int W, int R, bool ZERO>
__device__ __forceinline__ void dis_pass(const StoreDev& st, DisShared<W>& sh, int64_t j0, int64_t n_chunk, int nb,
                                         int ncand) {
  constexpr int NS = DisShared<W>::NS;
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint32_t code[R][NS];
  uint32_t zq[ZERO ? R : 1][NS / 2];   // zero factors: qubits of slots 2i (even bits) and 2i + 1 (odd bits)
  double cpk[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t j = j0 + (int64_t)r * kDisB + threadIdx.x;
    uint64_t kx[W], kz[W];
    double c = 0.0;
#pragma unroll
    for (int w = 0; w < W; ++w) kx[w] = kz[w] = 0ull;
    if (j < n_chunk) {
      int lo = 0, hi = nb - 1;   // last bucket with pre <= j (pre[0] = 0)
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (sh.pre[mid] <= j) lo = mid; else hi = mid - 1;
      }
      const int64_t i = sh.boff[lo] + (j - sh.pre[lo]);
#pragma unroll
      for (int w = 0; w < W; ++w) {
        kx[w] = st.x[w * st.cap + i];
        kz[w] = st.z[w * st.cap + i];
      }
      c = st.c[i];
    }
    double p0 = 1.0, p1 = 1.0;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const uint32_t xs = (uint32_t)(kx[s >> 2] >> (16 * (s & 3))), zs = (uint32_t)(kz[s >> 2] >> (16 * (s & 3)));
      const uint32_t cd = spread16(xs) | (spread16(zs) << 1);
      code[r][s] = cd;
#pragma unroll
      for (int i = 0; i < 8; i += 2) {
        p0 *= sh.pair[(8 * s + i) * 16 + ((cd >> (4 * i)) & 15)];
        p1 *= sh.pair[(8 * s + i + 1) * 16 + ((cd >> (4 * i + 4)) & 15)];
      }
      if (ZERO) {
        const uint32_t x = cd & 0x55555555u, z = (cd >> 1) & 0x55555555u;
        uint32_t m = (x & ~z & sh.zero[0][s]) | (z & ~x & sh.zero[1][s]) | (x & z & sh.zero[2][s]);
        asm volatile("" : "+v"(m));
        if (s & 1) zq[ZERO ? r : 0][s >> 1] |= m << 1; else zq[ZERO ? r : 0][s >> 1] = m;
      }
      // the products are needed here: left alone, the compiler holds every
      // looked-up value until the candidate loop and spills
      asm volatile("" : "+v"(p0), "+v"(p1));
    }
    cpk[r] = 0.5 * (c * (p0 * p1));   // (half: the signs below are +-2)
  }
  uint32_t next[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) next[s] = sh.sw[s];
  for (int t = 0; t < ncand; ++t) {
    uint32_t sw[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) sw[s] = (uint32_t)__builtin_amdgcn_readfirstlane((int)next[s]);
    const int tn = t + 1 < ncand ? t + 1 : t;
#pragma unroll
    for (int s = 0; s < NS; ++s) next[s] = sh.sw[tn * NS + s];
    double prod[R];
    uint32_t n[R], dead[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      prod[r] = cpk[r];
      n[r] = dead[r] = 0;
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      if (sw[s]) {
#pragma unroll
        for (int r = 0; r < R; ++r) n[r] += __popc(code[r][s] & sw[s]);
        uint32_t m = (sw[s] | (sw[s] >> 1)) & 0x55555555u;
        const char* slot = reinterpret_cast<const char*>(sh.ent) + s * 2048;
        do {
          const uint32_t b = (uint32_t)__builtin_ctz(m);
          m &= m - 1;
          const char* row = slot + b * 64 + ((sw[s] >> b) & 3u) * 32;
          double e[R];
#pragma unroll
          for (int r = 0; r < R; ++r)
            e[r] = *reinterpret_cast<const double*>(row + __builtin_amdgcn_ubfe(code[r][s], b, 2) * 8);
          // all R reads in flight before the first product waits for its own
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int r = 0; r < R; ++r) prod[r] *= e[r];
        } while (m);
      }
      if (ZERO && (s & 1)) {
        const uint32_t sup = ((sw[s - 1] | (sw[s - 1] >> 1)) & 0x55555555u) | ((sw[s] | (sw[s] << 1)) & 0xAAAAAAAAu);
#pragma unroll
        for (int r = 0; r < R; ++r) dead[r] |= zq[ZERO ? r : 0][s >> 1] & ~sup;
      }
    }
    double v = 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      // +2 for n = 1, -2 for n = 3 (mod 4), else a zero: the low bits of n are the
      // sign and the top exponent bit of the factor, and products by it are exact
      uint32_t f = n[r] << 30;
      if (ZERO) f = dead[r] ? 0u : f;
      v = fma(__hiloint2double((int)f, 0), prod[r], v);
    }
    v = wave_sum_to_lane63(v);
    if (lane == 63) sh.acc[wid][t] += v;
  }
}

// The (range, candidate) pairs are numbered range by range and every workgroup
// takes an equal run of them, so a range's terms are staged once for all the
// candidates of the run and few terms or few candidates still fill the chip.
//
// Bound: VALU issue, and LDS reads close behind.  1e6 two-word terms x 1000
// candidates of 10.8 support qubits: 50 VALU instructions per 64 pairs (3 per
// support qubit, 2 per touched slot, 7 for the sign and the sum) over four
// SIMDs against 11 reads of 512 bytes through one LDS, 1.63 ms (1.68 with the
// sign put together from +-1 and a mask); the former kernel (a second lookup
// per qubit for the phase, 4 terms per lane, ranges of buckets by tiles) took
// 2.38 ms plus 0.13 ms for the sum over ranges.  12,007 one-word terms x 13,472
// candidates: 1113 -> 193 us (its ranges held 307 of 2048
// terms).  233,001 terms x 5 candidates: 298 -> 19 us.
template <int W>
__global__ __launch_bounds__(kDisB, W <= 2 ? 3 : 2) void k_dis_batched(StoreDev st, int nq, const double* __restrict__ theta,
                                                       const double* __restrict__ phi,
                                                       const uint64_t* __restrict__ cx,
                                                       const uint64_t* __restrict__ cz, int64_t n_cand,
                                                       int64_t ld_cand, int tile_size, int max_ranges, int fixed,
                                                       int n_cu, double* __restrict__ partial) {
  constexpr int NQ = 64 * W, NS = 4 * W;
  extern __shared__ __align__(16) unsigned char smem_dis[];
  DisShared<W>& sh = *reinterpret_cast<DisShared<W>*>(smem_dis);
  const int64_t B = 1ll << *st.m;
  const int64_t per = dis_range_buckets(*st.total, B, max_ranges, fixed, n_cand, n_cu);
  const int64_t nr = (B + per - 1) / per;
  int64_t run = (nr * n_cand + gridDim.x - 1) / gridDim.x;
  const int64_t least = n_cand < kDisRun ? n_cand : kDisRun;
  if (run < least) run = least;
  int64_t at = blockIdx.x * run;
  int64_t end = at + run < nr * n_cand ? at + run : nr * n_cand;
  if (at >= end) return;
  // tables
  double* fac = &sh.acc[0][0];
  static_assert(NQ * 4 <= kDisWaves * kDisTile, "the factors fit the accumulators");
  bool zero = false;
  for (int i = threadIdx.x; i < 3 * NS; i += kDisB) (&sh.zero[0][0])[i] = 0u;
  __syncthreads();
  for (int q = threadIdx.x; q < NQ; q += kDisB) {
    double b[4] = {1.0, 1.0, 1.0, 1.0};
    if (q < nq) {
      double st_, ct, sp, cp;
      sincos(theta[q], &st_, &ct);
      sincos(phi[q], &sp, &cp);
#pragma unroll
      for (int op = 1; op < 4; ++op) b[op] = bloch_factor(op, st_, ct, sp, cp);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      fac[4 * q + k] = b[k];
      if (b[k] == 0.0) {
        zero = true;
        atomicOr(&sh.zero[k == 1 ? 0 : k == 2 ? 1 : 2][q >> 4], 1u << (2 * (q & 15)));
      }
    }
  }
  const bool any_zero = __syncthreads_or(zero) != 0;
  for (int i = threadIdx.x; i < NQ * 16; i += kDisB) {
    const int k = i & 3, q = i >> 4;
    const int x1 = k & 1, z1 = k >> 1, z2 = (i >> 2) & 1, x2 = (i >> 3) & 1;
    const int ph = (x1 * z1 + x2 * z2 + 2 * z1 * x2 - (x1 ^ x2) * (z1 ^ z2)) & 3;
    const int bits = (x1 & z2) + (z1 & x2);   // bits of this qubit in code & sw
    const double bk = fac[4 * q + k], bq = fac[4 * q + (k ^ (x2 | (z2 << 1)))];
    const double ratio = bk == 0.0 ? bq : bq / bk;
    sh.ent[i] = ((ph - bits) & 2) ? -ratio : ratio;
  }
  for (int i = threadIdx.x; i < NQ / 2 * 16; i += kDisB) {
    const double f0 = fac[8 * (i >> 4) + (i & 3)], f1 = fac[8 * (i >> 4) + 4 + ((i >> 2) & 3)];
    sh.pair[i] = (f0 == 0.0 ? 1.0 : f0) * (f1 == 0.0 ? 1.0 : f1);
  }
  while (at < end) {
    const int64_t range = at / n_cand, a_lo = at - range * n_cand;
    const int64_t left = end - at, room = n_cand - a_lo;
    const int64_t a_hi = a_lo + (left < room ? left : room);
    at += a_hi - a_lo;
    const int64_t b_lo = range * per, b_hi = b_lo + per < B ? b_lo + per : B;
    for (int64_t a0 = a_lo; a0 < a_hi; a0 += tile_size) {
      const int ncand = (int)(a_hi - a0 < tile_size ? a_hi - a0 : tile_size);   // tile_size <= kDisTile
      __syncthreads();   // tables ready / previous tile written out
      for (int i = threadIdx.x; i < ncand * NS; i += kDisB) {
        const int t = i / NS, s = i % NS;
        const uint32_t xs = (uint32_t)(cx[(s >> 2) * ld_cand + a0 + t] >> (16 * (s & 3)));
        const uint32_t zs = (uint32_t)(cz[(s >> 2) * ld_cand + a0 + t] >> (16 * (s & 3)));
        sh.sw[i] = spread16(zs) | (spread16(xs) << 1);
      }
      for (int i = threadIdx.x; i < kDisWaves * ncand; i += kDisB) sh.acc[i / ncand][i % ncand] = 0.0;
      for (int64_t cb = b_lo; cb < b_hi; cb += kDisChunk) {
        const int nb = (int)((b_hi - cb) < kDisChunk ? (b_hi - cb) : kDisChunk);
        __syncthreads();   // candidates staged / previous chunk done with pre, boff
        uint64_t total;
        const uint64_t n_b = threadIdx.x < nb ? (uint64_t)st.cnt[cb + threadIdx.x] : 0ull;
        const uint64_t ex = block_exclusive_scan_n<kDisWaves>(n_b, sh.scan_tmp, total);
        if (threadIdx.x < nb) {
          sh.pre[threadIdx.x] = (int64_t)ex;
          sh.boff[threadIdx.x] = st.off[cb + threadIdx.x];
        }
        if (threadIdx.x == 0) sh.pre[nb] = (int64_t)total;
        __syncthreads();
        const int64_t n_chunk = (int64_t)total;
        // full passes, then the rest with as few idle lanes as the terms per
        // lane of a pass allow
        for (int64_t j = 0; j < n_chunk;) {
          const int64_t rest = n_chunk - j;
          if (any_zero) {
            if (rest > 2 * kDisB) { dis_pass<W, 4, true>(st, sh, j, n_chunk, nb, ncand); j += 4 * kDisB; }
            else { dis_pass<W, 2, true>(st, sh, j, n_chunk, nb, ncand); j += 2 * kDisB; }
          } else if (rest > 4 * kDisB) {
            dis_pass<W, kDisR, false>(st, sh, j, n_chunk, nb, ncand); j += kDisR * kDisB;
          } else if (rest > 2 * kDisB) {
            dis_pass<W, 4, false>(st, sh, j, n_chunk, nb, ncand); j += 4 * kDisB;
          } else {
            dis_pass<W, 2, false>(st, sh, j, n_chunk, nb, ncand); j += 2 * kDisB;
          }
        }
      }
      __syncthreads();
      for (int t = threadIdx.x; t < ncand; t += kDisB) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < kDisWaves; ++w) s += sh.acc[w][t];
        partial[range * n_cand + a0 + t] = s;
      }
    }
  }
}

int64_t dis_tile() { return kDisTile; }   // the largest tile the batched kernel holds

// Sums the ranges' partials of 16 candidates per workgroup: 16 threads take
// every 16th range of a candidate (reads of 128 bytes), then their sums in
// order.  (One thread per candidate walked all ranges alone: 243 us for 2048
// ranges of 5 candidates.)
__global__ __launch_bounds__(kBlock) void k_dis_reduce(StoreDev st, const double* partial, int max_ranges, int fixed,
                                                       int n_cu, int64_t n_cand, double* g) {
  __shared__ double red[16][17];
  const int64_t B = 1ll << *st.m, per = dis_range_buckets(*st.total, B, max_ranges, fixed, n_cand, n_cu);
  const int64_t nr = (B + per - 1) / per;
  const int t = threadIdx.x & 15, l = threadIdx.x >> 4;
  const int64_t a = blockIdx.x * 16ll + t;
  double s = 0.0;
  if (a < n_cand) {
    int64_t r = l;
    for (; r + 48 < nr; r += 64) {   // four loads in flight, added in order
      const double v0 = partial[r * n_cand + a], v1 = partial[(r + 16) * n_cand + a];
      const double v2 = partial[(r + 32) * n_cand + a], v3 = partial[(r + 48) * n_cand + a];
      s += v0; s += v1; s += v2; s += v3;
    }
    for (; r < nr; r += 16) s += partial[r * n_cand + a];
  }
  red[l][t] = s;
  __syncthreads();
  if (threadIdx.x < 16 && a < n_cand) {
    double v = 0.0;
#pragma unroll
    for (int i = 0; i < 16; ++i) v += red[i][t];
    g[a] = v;
  }
}

// Plain form: one candidate per launch.  Workgroup g takes the groups of G
// consecutive buckets g, g + grid, ... and streams each group's rows as one
// flat range, four terms per thread and pass, so short buckets keep every lane
// busy.  About half the terms anticommute with a candidate; their products
// Q = K P_a go to a per-wavefront ring in LDS, and the expectation of Q is
// formed on full wavefronts of 64 ring entries, so the 44-lookup product is
// not issued for lanes whose term commutes.  The last workgroup to finish
// sums the per-workgroup partials in a fixed order and writes g[a], so a
// candidate costs one launch.
constexpr int kDisOneR = 8;
constexpr int kDisRing = 128;   // ring entries per wavefront (< 64 left + 64 added)

template <int W>
struct DisRing {
  uint64_t x[W][kDisRing], z[W][kDisRing];
  double v[kDisRing];   // +-c: the sign of Im(i^e) for the product phase e
};

template <int W>
__global__ __launch_bounds__(kBlock) void k_dis_one(StoreDev st, const double* lut_g,
                                                    const uint64_t* cx, const uint64_t* cz,
                                                    int64_t ld_cand, int64_t a, double* partial,
                                                    unsigned int* done, double* g) {
  constexpr int R = kDisOneR;
  __shared__ double lut[W * kGroupsPerWord * kLutEntries];
  __shared__ double red[kWaves];
  __shared__ uint64_t scan_tmp[kWaves];
  __shared__ int64_t s_pre[kBlock + 1];
  __shared__ int64_t s_off[kBlock];
  __shared__ DisRing<W> ring_all[kWaves];
  __shared__ int s_last;
  for (int i = threadIdx.x; i < W * kGroupsPerWord * kLutEntries; i += kBlock) lut[i] = lut_g[i];
  uint64_t px[W], pz[W];
#pragma unroll
  for (int w = 0; w < W; ++w) {
    px[w] = cx[w * ld_cand + a];
    pz[w] = cz[w * ld_cand + a];
  }
  const int lane = threadIdx.x & 63;
  DisRing<W>& ring = ring_all[threadIdx.x >> 6];
  int head = 0, fill = 0;   // wave-uniform ring state
  double acc = 0.0;
  // <Q> of 64 ring entries from the head (lanes past `count` add nothing)
  auto drain = [&](int count) {
    // the ring entries were written by other lanes of this wavefront
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int k = (head + lane) & (kDisRing - 1);
    if (lane < count) {
      uint64_t qx[W], qz[W];
#pragma unroll
      for (int w = 0; w < W; ++w) {
        qx[w] = ring.x[w][k];
        qz[w] = ring.z[w][k];
      }
      acc += ring.v[k] * expect_lut<W>(lut, qx, qz);
    }
    head = (head + count) & (kDisRing - 1);
    fill -= count;
    // the drained entries are read before later entries overwrite them
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  const int64_t B = 1ll << *st.m;
  int64_t G = B / gridDim.x;
  G = G < 1 ? 1 : (G > kBlock ? kBlock : G);
  const int64_t ngroups = (B + G - 1) / G;
  __syncthreads();
  for (int64_t grp = blockIdx.x; grp < ngroups; grp += gridDim.x) {
    const int64_t b = grp * G + threadIdx.x;
    const bool mine = threadIdx.x < G && b < B;
    const int64_t cnt = mine ? st.cnt[b] : 0;
    const int64_t off = mine ? st.off[b] : 0;
    uint64_t total;
    // (the scan's barriers also order the previous group's reads of s_pre)
    const uint64_t ex = block_exclusive_scan((uint64_t)cnt, scan_tmp, total);
    s_pre[threadIdx.x] = (int64_t)ex;
    s_off[threadIdx.x] = off;
    if (threadIdx.x == 0) s_pre[kBlock] = (int64_t)total;
    __syncthreads();
    // the group's rows are one range when every bucket starts where the one
    // before it ends (a loaded store); then row = base + i, the row the
    // search below would find (thread 0 holds the group's first bucket)
    const int64_t base = s_off[0];
    const bool contig = __syncthreads_and(!mine || off - (int64_t)ex == base) != 0;
    const int64_t n = (int64_t)total;
    for (int64_t i0 = 0; i0 < n; i0 += kBlock * R) {
      uint64_t kx[R][W], kz[R][W];
      double kc[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int64_t i = i0 + r * kBlock + threadIdx.x;
        kc[r] = 0.0;
#pragma unroll
        for (int w = 0; w < W; ++w) kx[r][w] = kz[r][w] = 0;
        if (i < n) {
          int64_t row = base + i;
          if (!contig) {
            int lo = 0;   // the last bucket of the group whose first row is <= i
#pragma unroll
            for (int step = kBlock / 2; step; step >>= 1)
              if (s_pre[lo + step] <= i) lo += step;
            row = s_off[lo] + (i - s_pre[lo]);
          }
#pragma unroll
          for (int w = 0; w < W; ++w) {
            kx[r][w] = __builtin_nontemporal_load(&st.x[w * st.cap + row]);
            kz[r][w] = __builtin_nontemporal_load(&st.z[w * st.cap + row]);
          }
          kc[r] = __builtin_nontemporal_load(&st.c[row]);
        }
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        // padding lanes (key 0) commute
        const bool anti = anticommutes<W>(kx[r], kz[r], px, pz);
        const uint64_t mask = __ballot(anti);
        if (anti) {
          const int e = product_phase<W>(kx[r], kz[r], px, pz);
          const int k = (head + fill + lanes_below(mask)) & (kDisRing - 1);
#pragma unroll
          for (int w = 0; w < W; ++w) {
            ring.x[w][k] = kx[r][w] ^ px[w];
            ring.z[w][k] = kz[r][w] ^ pz[w];
          }
          ring.v[k] = (e == 1) ? kc[r] : -kc[r];
        }
        fill += __popcll(mask);
        if (fill >= 64) drain(64);   // LDS operations of one wavefront complete in order
      }
    }
  }
  if (fill > 0) drain(fill);
  const double s = block_sum(acc, red);
  if (threadIdx.x == 0) {
    partial[blockIdx.x] = s;
    __threadfence();
    s_last = atomicAdd(done, 1u) == gridDim.x - 1;
  }
  __syncthreads();
  if (s_last) {   // every partial is written: sum them in a fixed order
    __threadfence();
    const volatile double* vp = partial;
    double t = 0.0;
    for (int k = threadIdx.x; k < (int)gridDim.x; k += kBlock) t += vp[k];
    t = block_sum(t, red);
    if (threadIdx.x == 0) {
      g[a] = t;
      *done = 0u;   // ready for the next candidate
    }
  }
}

__global__ void k_zero_u32(unsigned int* p) { *p = 0u; }

// Workgroups of k_dis_one that one CU holds at once (its LDS bounds it): the
// plain launch uses exactly that many per CU, so every workgroup is resident
// and takes one bucket group.
int dis_one_blocks_per_cu(int W) {
  int nb = 0;
  hipError_t e;
  switch (W) {
    case 1: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, (const void*)k_dis_one<1>, kBlock, 0); break;
    case 2: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, (const void*)k_dis_one<2>, kBlock, 0); break;
    case 3: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, (const void*)k_dis_one<3>, kBlock, 0); break;
    default: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, (const void*)k_dis_one<4>, kBlock, 0); break;
  }
  return (e == hipSuccess && nb > 0) ? nb : 1;
}

template <int W>
static void launch_dis_w(const StoreDev& st, const double* theta, const double* phi, int nq, const uint64_t* cx,
                         const uint64_t* cz, int64_t n_cand, int64_t ld_cand, int tile, int n_cu, int max_ranges,
                         int fixed, double* partial, hipStream_t s) {
  const size_t lds = sizeof(DisShared<W>);
  (void)hipFuncSetAttribute((const void*)k_dis_batched<W>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  // three workgroups per CU are resident (two for wide keys; registers); four
  // times as many even out ranges that need a second pass (1e6 terms x 1000
  // candidates: 1903 us with the resident ones alone, 1678 us with four times,
  // 1731 us with eight times as many: each builds its tables)
  hipLaunchKernelGGL(k_dis_batched<W>, dim3(n_cu * (W <= 2 ? 12 : 8)), dim3(kDisB), lds, s, st, nq, theta, phi, cx, cz,
                     n_cand, ld_cand, tile, max_ranges, fixed, n_cu, partial);
}

void launch_dis_batched(int W, const StoreDev& st, const double* theta, const double* phi, int nq, const uint64_t* cx,
                        const uint64_t* cz, int64_t n_cand, int64_t ld_cand, int tile, int n_cu, int max_ranges,
                        int fixed, double* partial, double* g, hipStream_t s) {
  if (n_cand <= 0) return;
  if (tile < 1 || tile > kDisTile) tile = kDisTile;
  switch (W) {
    case 1: launch_dis_w<1>(st, theta, phi, nq, cx, cz, n_cand, ld_cand, tile, n_cu, max_ranges, fixed, partial, s); break;
    case 2: launch_dis_w<2>(st, theta, phi, nq, cx, cz, n_cand, ld_cand, tile, n_cu, max_ranges, fixed, partial, s); break;
    case 3: launch_dis_w<3>(st, theta, phi, nq, cx, cz, n_cand, ld_cand, tile, n_cu, max_ranges, fixed, partial, s); break;
    default: launch_dis_w<4>(st, theta, phi, nq, cx, cz, n_cand, ld_cand, tile, n_cu, max_ranges, fixed, partial, s); break;
  }
  hipLaunchKernelGGL(k_dis_reduce, dim3((unsigned)((n_cand + 15) / 16)), dim3(kBlock), 0, s, st, partial, max_ranges,
                     fixed, n_cu, n_cand, g);
}

void launch_dis_plain(int W, const StoreDev& st, const double* lut, const uint64_t* cx, const uint64_t* cz,
                      int64_t n_cand, int64_t ld_cand, int grid, double* partial, double* g, hipStream_t s) {
  if (n_cand <= 0) return;
  // partial[0, grid) per-workgroup sums, then the finish counter
  unsigned int* done = reinterpret_cast<unsigned int*>(partial + grid);
  hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(1), 0, s, done);
  for (int64_t a = 0; a < n_cand; ++a) {
    switch (W) {
      case 1: hipLaunchKernelGGL(k_dis_one<1>, dim3(grid), dim3(kBlock), 0, s, st, lut, cx, cz, ld_cand, a, partial, done, g); break;
      case 2: hipLaunchKernelGGL(k_dis_one<2>, dim3(grid), dim3(kBlock), 0, s, st, lut, cx, cz, ld_cand, a, partial, done, g); break;
      case 3: hipLaunchKernelGGL(k_dis_one<3>, dim3(grid), dim3(kBlock), 0, s, st, lut, cx, cz, ld_cand, a, partial, done, g); break;
      default: hipLaunchKernelGGL(k_dis_one<4>, dim3(grid), dim3(kBlock), 0, s, st, lut, cx, cz, ld_cand, a, partial, done, g); break;
    }
  }
}

}  // namespace iqcc
