// QMF energy (Sec. II, Eq. 3; energy functional of App. A) and its gradient
// with respect to the Bloch angles.
//
// <K> of the product state is prod_j b_j(sigma_j) with b(I) = 1,
// b(X) = sin t cos f, b(Y) = sin t sin f, b(Z) = cos t.  Terms are streamed
// once; the product uses a table per group of 4 (or 3) qubits in LDS.  Partial
// sums are per workgroup and reduced in a fixed order.
#include <cfloat>

#include "iqcc_internal.h"

#pragma clang fp contract(off)

namespace iqcc {

__global__ void k_build_lut(int W, int nq, const double* theta, const double* phi, double* lut) {
  const int n = W * kGroupsPerWord * kLutEntries;
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < n; e += gridDim.x * blockDim.x) {
    const int idx = e % kLutEntries;
    const int gi = e / kLutEntries;
    const int h = gi / kGroupsPerHalf, g = gi % kGroupsPerHalf;
    double p = 1.0;
    for (int i = 0; i < 3; ++i) {
      const int bitpos = 3 * g + i;          // bit within the 32-bit half
      const int q = 32 * h + bitpos;
      if (bitpos >= 32 || q >= nq) continue;
      const int op = ((idx >> i) & 1) | (((idx >> (3 + i)) & 1) << 1);
      if (op == 0) continue;
      double st, ct, sp, cp;
      sincos(theta[q], &st, &ct);
      sincos(phi[q], &sp, &cp);
      p *= bloch_factor(op, st, ct, sp, cp);
    }
    lut[e] = p;
  }
}

void launch_build_lut(int W, int nq, const double* theta, const double* phi, double* lut,
                      hipStream_t s) {
  hipLaunchKernelGGL(k_build_lut, dim3(16), dim3(kBlock), 0, s, W, nq, theta, phi, lut);
}

// ---------------------------------------------------------------------------
// Fixed-order reduction of per-workgroup partials: out = scale * sum.
// ---------------------------------------------------------------------------
__global__ void k_finalize_sum(const double* partial, int n, const double* scale,
                               const double* base, double* out) {
  __shared__ double red[kWaves];
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) s += partial[i];
  s = block_sum(s, red);
  if (threadIdx.x == 0) {
    if (scale) s *= *scale;
    *out = base ? *base + s : s;
  }
}

void launch_finalize_sum(const double* partial, int n, const double* scale, double* out,
                         hipStream_t s, const double* base) {
  hipLaunchKernelGGL(k_finalize_sum, dim3(1), dim3(kBlock), 0, s, partial, n, scale, base, out);
}

// Exact sum of FixedSum parts (hi, lo, mag as three 8-byte words each).
__global__ void k_finalize_fixed(const double* parts, int n, double* out) {
  __shared__ long long red_hi[kWaves], red_lo[kWaves];
  __shared__ double red_mag[kWaves];
  FixedSum f;
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    f.hi += __double_as_longlong(parts[3 * i]);
    f.lo += __double_as_longlong(parts[3 * i + 1]);
    f.mag += parts[3 * i + 2];
  }
  const FixedSum t = block_fixed_sum<kWaves>(f, red_hi, red_lo, red_mag);
  if (threadIdx.x == 0) *out = fixed_value(t.hi, t.lo, t.mag);
}

void launch_finalize_fixed(const double* parts, int n, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_finalize_fixed, dim3(1), dim3(kBlock), 0, s, parts, n, out);
}

// ---------------------------------------------------------------------------
// Energy of a store in one launch.  Workgroup g takes the groups of G
// consecutive buckets g, g + grid, ... (G = 1 .. 512 so that every workgroup
// has a group); the rows of a group's buckets are streamed as one flat range,
// kEItems terms per thread and pass, so small buckets do not each cost a round
// trip.
//
// The product of a term comes from a table in LDS that every workgroup builds
// from the angles.  Keys of one or two words: 4-qubit groups ("nibbles"), 16
// per key word, 256 entries each (32 KB per word).  A byte of x and the same
// byte of z hold two nibbles; two bit-field inserts per 32-bit half word put
// the codes of its eight groups into the bytes of two registers, and each
// lookup takes one byte extraction.  A code holds the four z bits below the
// four x bits: most groups of a Jordan-Wigner string are Z strings (x = 0),
// whose 16 codes then lie next to each other, in different LDS banks (with
// the x bits low they were 16 entries apart and met in two banks: 156 us
// against XXX us on 1.6e7 two-word terms).  Wider keys: 3-qubit groups, 22 per
// word and 64 entries each, because nibble tables would leave one workgroup
// per CU.
//
// The grid holds what the CUs keep resident (more workgroups would only build
// more tables), and of it only as many workgroups take part ("active") as
// there are passes of kEMinRows rows: below that a workgroup would spend its
// time on its table and its arrival (17.1 us a call over the stores of a
// 32-Hamiltonian batch with one workgroup per bucket, 12.3 us with this rule).
// The active workgroups leave their sums in the finish slot; the last of them
// to arrive adds them in a fixed order, so a call is one launch.
//
// Bound: HBM for large stores (40 bytes a two-word term), the chain of
// latencies (bucket table, rows, table build, arrival) for small ones.
// 1.6e7 two-word terms: 128 us, 5.0 TB/s (table, sums and reduction in three
// launches: 168 us); 361 terms: 6.6 us (23 us).
// ---------------------------------------------------------------------------
constexpr int kEItems = 4;
constexpr int64_t kEMinRows = 2048;
constexpr int kNibbleEntries = 256;
constexpr int kNibblesPerWord = 16;
constexpr int kE4Block = 512;

template <int W>
struct EnergyTable {
  static constexpr bool kNibble = W <= 2;
  static constexpr int kEntries = kNibble ? W * kNibblesPerWord * kNibbleEntries : W * kGroupsPerWord * kLutEntries;
  // scratch of the build: the qubits' factors and, for nibbles, the products
  // of the two qubits of every even/odd pair
  static constexpr int kBuild = 64 * W * 4 + (kNibble ? 32 * W * 16 : 0);
};

// Builds the table (the whole workgroup; ends with a barrier).  Multiplying by
// the identity's factor 1.0 is exact.
template <int W>
__device__ void build_energy_table(double* lut, double* tmp, int nq, const double* theta, const double* phi) {
  double* fac = tmp;   // [64 W][4]: I, X, Z, Y
  for (int q = threadIdx.x; q < 64 * W; q += kE4Block) {
    double st = 0.0, ct = 1.0, sp = 0.0, cp = 1.0;
    const bool live = q < nq;
    if (live) {
      sincos(theta[q], &st, &ct);
      sincos(phi[q], &sp, &cp);
    }
#pragma unroll
    for (int op = 0; op < 4; ++op) fac[4 * q + op] = live ? bloch_factor(op, st, ct, sp, cp) : 1.0;
  }
  __syncthreads();
  if constexpr (EnergyTable<W>::kNibble) {
    double* pair = fac + 64 * W * 4;   // [32 W][16]: z bits low, x bits high
    for (int e = threadIdx.x; e < 32 * W * 16; e += kE4Block) {
      const int q = 2 * (e >> 4), z = e & 3, x = (e >> 2) & 3;
      pair[e] = fac[4 * q + ((x & 1) | ((z & 1) << 1))] * fac[4 * (q + 1) + ((x >> 1) | ((z >> 1) << 1))];
    }
    __syncthreads();
    for (int e = threadIdx.x; e < EnergyTable<W>::kEntries; e += kE4Block) {
      const int z = e & 15, x = (e >> 4) & 15, gi = e >> 8;
      lut[e] = pair[(2 * gi) * 16 + ((z & 3) | ((x & 3) << 2))] * pair[(2 * gi + 1) * 16 + ((z >> 2) | ((x >> 2) << 2))];
    }
  } else {
    for (int e = threadIdx.x; e < EnergyTable<W>::kEntries; e += kE4Block) {
      const int code = e % kLutEntries, gi = e / kLutEntries;
      const int h = gi / kGroupsPerHalf, g = gi % kGroupsPerHalf;
      double p = 1.0;
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        const int bit = 3 * g + r;
        if (bit < 32) p *= fac[4 * (32 * h + bit) + (((code >> (3 + r)) & 1) | (((code >> r) & 1) << 1))];
      }
      lut[e] = p;
    }
  }
  __syncthreads();
}

template <int W>
__device__ __forceinline__ double expect_table(const double* lut, const uint64_t* x, const uint64_t* z) {
  double p[4] = {1.0, 1.0, 1.0, 1.0};
#pragma unroll
  for (int h = 0; h < 2 * W; ++h) {
    const uint32_t xh = (uint32_t)(x[h >> 1] >> (32 * (h & 1)));
    const uint32_t zh = (uint32_t)(z[h >> 1] >> (32 * (h & 1)));
    if constexpr (EnergyTable<W>::kNibble) {
      // byte k: code of nibble 2k (lo) and of nibble 2k + 1 (hi), z bits low
      const uint32_t lo = ((xh << 4) & 0xF0F0F0F0u) | (zh & 0x0F0F0F0Fu);
      const uint32_t hi = ((zh >> 4) & 0x0F0F0F0Fu) | (xh & 0xF0F0F0F0u);
      const double* lh = lut + 8 * h * kNibbleEntries;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        p[k] *= lh[(2 * k) * kNibbleEntries + ((lo >> (8 * k)) & 0xFFu)];
        p[k] *= lh[(2 * k + 1) * kNibbleEntries + ((hi >> (8 * k)) & 0xFFu)];
      }
    } else {
      const double* lh = lut + h * kGroupsPerHalf * kLutEntries;
#pragma unroll
      for (int g = 0; g < kGroupsPerHalf; ++g) {
        const uint32_t code = __builtin_amdgcn_ubfe(zh, 3 * g, 3) | (__builtin_amdgcn_ubfe(xh, 3 * g, 3) << 3);
        p[g & 3] *= lh[g * kLutEntries + code];
      }
    }
  }
  return (p[0] * p[1]) * (p[2] * p[3]);
}

template <int W>
size_t energy_lds_bytes() {
  // table, its build's scratch, first rows and row prefix sums of a group
  return (size_t)(EnergyTable<W>::kEntries + EnergyTable<W>::kBuild) * 8 + (size_t)kE4Block * 8 +
         (size_t)(kE4Block + 1) * 4;
}

template <int W>
__global__ __launch_bounds__(kE4Block) void k_energy(StoreDev st, int nq, const double* theta, const double* phi,
                                                     double* slot, double* out) {
  extern __shared__ __align__(16) unsigned char smem_en[];
  double* lut = (double*)smem_en;
  double* tmp = lut + EnergyTable<W>::kEntries;                  // [kBuild]
  int64_t* s_off = (int64_t*)(tmp + EnergyTable<W>::kBuild);     // [kE4Block]
  uint32_t* s_pre = (uint32_t*)(s_off + kE4Block);               // [kE4Block + 1]
  __shared__ double red[kE4Block / 64];
  __shared__ uint64_t scan_tmp[kE4Block / 64];
  __shared__ int s_last;
  const int64_t B = 1ll << *st.m;
  // at least kEMinRows rows per workgroup (one pass) where the store has them
  int64_t want = (*st.total + kEMinRows - 1) / kEMinRows;
  want = want < 1 ? 1 : (want > gridDim.x ? gridDim.x : want);
  int64_t G = (B + want - 1) / want;
  G = G > kE4Block ? kE4Block : G;
  const int64_t ngroups = (B + G - 1) / G;
  const unsigned active = ngroups < want ? (unsigned)ngroups : (unsigned)want;
  if (blockIdx.x >= active) return;
  bool table = false;
  double acc = 0.0;
  for (int64_t grp = blockIdx.x; grp < ngroups; grp += active) {
    const int64_t b = grp * G + threadIdx.x;
    const bool mine = threadIdx.x < G && b < B;
    const int64_t cnt = mine ? st.cnt[b] : 0;
    const int64_t off = mine ? st.off[b] : 0;
    uint64_t total;
    // (the scan's barriers also order the previous group's reads of s_pre)
    const uint64_t ex = block_exclusive_scan_n<kE4Block / 64>((uint64_t)cnt, scan_tmp, total);
    s_pre[threadIdx.x] = (uint32_t)ex;
    s_off[threadIdx.x] = off;
    if (threadIdx.x == 0) s_pre[kE4Block] = (uint32_t)total;
    __syncthreads();
    // the group's rows are one range when every bucket starts where the one
    // before it ends (a loaded store); then row = base + i, the row the search
    // below would find (thread 0 holds the group's first bucket)
    const int64_t base = s_off[0];
    const bool contig = __syncthreads_and(!mine || off - (int64_t)ex == base) != 0;
    const uint32_t n = (uint32_t)total;
    uint32_t i0 = 0;
    do {
      uint64_t kx[kEItems][W], kz[kEItems][W];
      double kc[kEItems];
#pragma unroll
      for (int r = 0; r < kEItems; ++r) {
        const uint32_t i = i0 + r * kE4Block + threadIdx.x;
        kc[r] = 0.0;
#pragma unroll
        for (int w = 0; w < W; ++w) kx[r][w] = kz[r][w] = 0;
        if (i < n) {
          int64_t row = base + i;
          if (!contig) {
            int lo = 0;   // the last bucket of the group whose first row is <= i
#pragma unroll
            for (int step = kE4Block / 2; step; step >>= 1)
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
      if (!table) {   // built while the first rows are on their way
        build_energy_table<W>(lut, tmp, nq, theta, phi);
        table = true;
      }
#pragma unroll
      for (int r = 0; r < kEItems; ++r) acc += kc[r] * expect_table<W>(lut, kx[r], kz[r]);
      i0 += kE4Block * kEItems;
    } while (i0 < n);
  }
  const double s = block_sum_n<kE4Block / 64>(acc, red);
  if (active == 1) {
    if (threadIdx.x == 0) *out = s;
    return;
  }
  if (threadIdx.x == 0) s_last = finish_arrive(slot, blockIdx.x, s, active);
  __syncthreads();
  if (s_last) {
    double t = 0.0;
    for (unsigned k = threadIdx.x; k < active; k += kE4Block) t += finish_partial(slot, k);
    t = block_sum_n<kE4Block / 64>(t, red);
    if (threadIdx.x == 0) *out = t;
  }
}

template <int W>
static void launch_energy_w(int nq, const StoreDev& st, int n_cu, int per_cu, size_t lds_per_cu, const double* theta,
                            const double* phi, double* slot, double* out, hipStream_t s) {
  const size_t lds = energy_lds_bytes<W>();
  // resident workgroups per CU: LDS (with the static part), 2048 threads
  int fit = (int)(lds_per_cu / (lds + 256));
  fit = fit < 1 ? 1 : (fit > 2048 / kE4Block ? 2048 / kE4Block : fit);
  int grid = n_cu * (per_cu < fit ? per_cu : fit);
  if (grid > kFinishPartials) grid = kFinishPartials;
  (void)hipFuncSetAttribute((const void*)k_energy<W>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL(k_energy<W>, dim3(grid), dim3(kE4Block), lds, s, st, nq, theta, phi, slot, out);
}

void launch_energy(int W, int nq, const StoreDev& st, int n_cu, int per_cu, size_t lds_per_cu, const double* theta,
                   const double* phi, double* slot, double* out, hipStream_t s) {
  switch (W) {
    case 1: launch_energy_w<1>(nq, st, n_cu, per_cu, lds_per_cu, theta, phi, slot, out, s); break;
    case 2: launch_energy_w<2>(nq, st, n_cu, per_cu, lds_per_cu, theta, phi, slot, out, s); break;
    case 3: launch_energy_w<3>(nq, st, n_cu, per_cu, lds_per_cu, theta, phi, slot, out, s); break;
    default: launch_energy_w<4>(nq, st, n_cu, per_cu, lds_per_cu, theta, phi, slot, out, s); break;
  }
}

// ---------------------------------------------------------------------------
// Backward w.r.t. the Bloch angles (derivative of the Eq. 3 energy).
// dE/dtheta_q = sum_sigma S[q][sigma] db_sigma/dtheta (likewise phi), where
// S[q][sigma] adds, over the terms with sigma on qubit q, c times the product
// of the term's other factors.
//
// The product of a term runs over its 3-qubit groups (the energy table L), so
// the derivative is first formed per group table entry:
//   T[g][e] = sum over the terms whose group g has code e != 0 of
//             c * prod_{g' != g} L_g',
// and once per workgroup S[q][sigma] = sum over the codes e of q's group with
// sigma at q's position of T[g][e] * (product of the group's other qubit
// factors of that code).  The product of a term's other groups comes from
// prefix and suffix products -- inside each 32-bit half word over its 11
// groups, and across the half words over their products -- with no division,
// so vanishing factors need no special case.
//
// Summation order does not change the result.  Each value is split into two
// integers, round(v * 2^20) and round((v - that * 2^-20) * 2^60), and added
// to two 64-bit integer tables with LDS atomics, which are exact; per
// workgroup the two sums turn into one double, and the per-workgroup S are
// reduced in a fixed order, so dE/dtheta and dE/dphi are the same on every
// run.  The split is exact for |v| < 2^31 and the sums cannot overflow while
// (largest |c| of the workgroup's terms) * (its term count) < 2^42 and the
// count is below 2^23; a workgroup past these bounds, or one that meets a
// non-finite coefficient or angle, writes NaN instead of its S.  Resolution:
// 2^-61 per added value.
// acc layout per workgroup: [3 * nq] with sigma order X, Z, Y.
// ---------------------------------------------------------------------------
constexpr int kBwdBlock = 512;
constexpr int kBwdGroup = 256;   // most buckets per group of one flat range
// LDS tables of the backward hold each 3-qubit group's 64 entries at a stride
// of 65, so that equal codes of different groups fall in different banks.
constexpr int kBwdStride = kLutEntries + 1;

size_t energy_bwd_lds_bytes(int W) {
  // energy table, the two integer tables (the per-qubit factors of the
  // epilogue reuse the first), bucket-group scan
  return (size_t)3 * W * kGroupsPerWord * kBwdStride * 8 + (size_t)(2 * kBwdGroup + 1) * 8;
}

// Workgroups per CU that the LDS of one CU holds (160 KiB), at most 2048
// threads (32 waves) in all.
int energy_bwd_blocks_per_cu(int W) {
  const int k = (int)((size_t)160 * 1024 / (energy_bwd_lds_bytes(W) + 512));
  const int kmax = 2048 / kBwdBlock;
  return k < 1 ? 1 : k > kmax ? kmax : k;
}

// v as round(v * 2^20) * 2^-20 + round(r * 2^60) * 2^-60 (r the remainder),
// both added to their integer tables.  Adding 1.5 * 2^32 (resp. 1.5 * 2^-8)
// rounds to a multiple of 2^-20 (2^-60), and the difference of the bit
// patterns is that multiple as an integer (both sums stay in the binade of the
// constant, whose low 32 bits are zero).
__device__ __forceinline__ void add_fixed(unsigned long long* hi, unsigned long long* lo, int e, double v) {
  const double k1 = 0x1.8p32, k0 = 0x1.8p-8;
  const double a1 = v + k1;
  const double r = v - (a1 - k1);
  const double a0 = r + k0;
  atomicAdd(&hi[e], (unsigned long long)(__double_as_longlong(a1) - __double_as_longlong(k1)));
  atomicAdd(&lo[e], (unsigned long long)(__double_as_longlong(a0) - __double_as_longlong(k0)));
}

// One term of the backward: T contributions of its non-identity groups and,
// when lam is given, its cotangent.
template <int W>
__device__ __forceinline__ void bwd_term(const double* lut, unsigned long long* thi,
                                         unsigned long long* tlo, const uint64_t* kx,
                                         const uint64_t* kz, double c, double* lam_row,
                                         double scale) {
  constexpr int NH = kGroupsPerHalf * kBwdStride;
  // products of the 2W half words (identity groups read entry 0 = 1.0)
  double hp[2 * W];
#pragma unroll
  for (int h = 0; h < 2 * W; ++h) {
    const uint32_t xh = (uint32_t)(kx[h >> 1] >> (32 * (h & 1)));
    const uint32_t zh = (uint32_t)(kz[h >> 1] >> (32 * (h & 1)));
    const double* lh = lut + h * NH;
    double p0 = 1.0, p1 = 1.0;
#pragma unroll
    for (int g = 0; g < kGroupsPerHalf; ++g) {
      const uint32_t code = __builtin_amdgcn_ubfe(xh, 3 * g, 3) | (__builtin_amdgcn_ubfe(zh, 3 * g, 3) << 3);
      if (g & 1) p1 *= lh[g * kBwdStride + code]; else p0 *= lh[g * kBwdStride + code];
    }
    hp[h] = p0 * p1;
  }
  // <K> for the coefficient cotangent
  if (lam_row) {
    double all = hp[0];
#pragma unroll
    for (int h = 1; h < 2 * W; ++h) all *= hp[h];
    *lam_row = scale * all;
  }
  // c times the product of the other half words, per half word
  double ho[2 * W];
  double pre = c;
#pragma unroll
  for (int h = 0; h < 2 * W; ++h) { ho[h] = pre; pre *= hp[h]; }
  double suf = 1.0;
#pragma unroll
  for (int h = 2 * W - 1; h >= 0; --h) { ho[h] *= suf; suf *= hp[h]; }
  // each half word: prefix and suffix over its groups.  A term visits its
  // half words, and the groups of each, starting at ones picked from its own
  // key bits, so that the lanes of a wave add into different groups' tables
  // at a time (fewer lanes on one LDS address or bank); the values do not
  // depend on where the term sits in the store.
  const uint32_t mix = ((uint32_t)kx[0] ^ (uint32_t)(kz[0] >> 29) ^ (uint32_t)(kx[W - 1] >> 35)) * 0x9E3779B1u;
  const int rot = (int)__umulhi(mix, 2u * W);
#pragma unroll 1
  for (int j = 0; j < 2 * W; ++j) {
    int h = rot + j;
    h = h >= 2 * W ? h - 2 * W : h;
    uint64_t xw = kx[0], zw = kz[0];
    double oh = ho[0];
#pragma unroll
    for (int u = 1; u < 2 * W; ++u) {
      if (u == h) oh = ho[u];
      if ((u & 1) == 0 && u == (h & ~1)) { xw = kx[u >> 1]; zw = kz[u >> 1]; }
    }
    const uint32_t xh = (uint32_t)(xw >> (32 * (h & 1)));
    const uint32_t zh = (uint32_t)(zw >> (32 * (h & 1)));
    const int rg = (int)__umulhi(mix * 0x85EBCA6Bu, (uint32_t)kGroupsPerHalf);
    const uint64_t xr = ((uint64_t)xh | ((uint64_t)xh << 33)) >> (3 * rg);
    const uint64_t zr = ((uint64_t)zh | ((uint64_t)zh << 33)) >> (3 * rg);
    double L[kGroupsPerHalf];
    uint32_t code[kGroupsPerHalf];
    int idx[kGroupsPerHalf];
    // group rg + g of the half, wrapped: the base before and after the wrap
    const int base_lo = h * NH + rg * kBwdStride;
    const int base_hi = base_lo - kGroupsPerHalf * kBwdStride;
#pragma unroll
    for (int g = 0; g < kGroupsPerHalf; ++g) {
      code[g] = (uint32_t)((xr >> (3 * g)) & 7) | ((uint32_t)((zr >> (3 * g)) & 7) << 3);
      idx[g] = (rg < kGroupsPerHalf - g ? base_lo : base_hi) + g * kBwdStride + (int)code[g];
      L[g] = lut[idx[g]];
    }
    double sf[kGroupsPerHalf];
    sf[kGroupsPerHalf - 1] = 1.0;
#pragma unroll
    for (int g = kGroupsPerHalf - 1; g > 0; --g) sf[g - 1] = sf[g] * L[g];
    double pg = oh;
#pragma unroll
    for (int g = 0; g < kGroupsPerHalf; ++g) {
      if (code[g] != 0) add_fixed(thi, tlo, idx[g], pg * sf[g]);
      pg *= L[g];
    }
  }
}

template <int W>
__global__ __launch_bounds__(kBwdBlock, 4) void k_energy_bwd(StoreDev st, int nq, const double* theta,
                                                             const double* phi, const double* lut_g,
                                                             const double* dE, double* lam,
                                                             double* acc_g) {
  constexpr int NE = W * kGroupsPerWord * kBwdStride;
  constexpr int NH = kGroupsPerHalf * kBwdStride;   // entries per half word
  extern __shared__ __align__(16) unsigned char smem_bwd[];
  double* lut = (double*)smem_bwd;                                     // [NE] L per group entry
  unsigned long long* thi = (unsigned long long*)(lut + NE);           // [NE] sums of round(v 2^20)
  unsigned long long* tlo = thi + NE;                                  // [NE] sums of the remainders
  double* fac = (double*)thi;   // epilogue: per qubit, factor of I, X, Z, Y (4 * 64W <= NE)
  int64_t* s_pre = (int64_t*)(tlo + NE);                               // [kBwdGroup + 1] group scan
  int64_t* s_off = s_pre + kBwdGroup + 1;                              // [kBwdGroup] first rows
  __shared__ double s_cmax[kBwdBlock / 64];
  __shared__ long long s_cnt[kBwdBlock / 64];
  __shared__ uint64_t scan_tmp[kBwdBlock / 64];
  __shared__ int s_bad;
  if (threadIdx.x == 0) s_bad = 0;
  __syncthreads();
  for (int i = threadIdx.x; i < NE; i += kBwdBlock) {
    const int k = i % kBwdStride;
    lut[i] = k < kLutEntries ? lut_g[i / kBwdStride * kLutEntries + k] : 0.0;
    thi[i] = tlo[i] = 0ull;
  }
  for (int q = threadIdx.x; q < nq; q += kBwdBlock)
    if (!(fabs(theta[q]) <= DBL_MAX && fabs(phi[q]) <= DBL_MAX)) s_bad = 1;
  const double scale = dE ? *dE : 1.0;
  bool ok = true;   // every coefficient finite and below 2^31 in magnitude
  double cmax = 0.0;
  long long nmine = 0;
  // Workgroup g takes the groups of G consecutive buckets g, g + grid, ...;
  // a group's rows are one flat range, one term per thread and pass, the next
  // pass's term loaded while this one is processed.
  const int64_t B = 1ll << *st.m;
  int64_t G = B / gridDim.x;
  G = G < 1 ? 1 : (G > kBwdGroup ? kBwdGroup : G);
  const int64_t ngroups = (B + G - 1) / G;
  for (int64_t grp = blockIdx.x; grp < ngroups; grp += gridDim.x) {
    const int64_t b = grp * G + threadIdx.x;
    const bool mine = threadIdx.x < G && b < B;
    const int64_t cnt = mine ? st.cnt[b] : 0;
    const int64_t off = mine ? st.off[b] : 0;
    uint64_t total;
    // (the scan's barriers also order the previous group's reads of s_pre)
    const uint64_t ex = block_exclusive_scan_n<kBwdBlock / 64>((uint64_t)cnt, scan_tmp, total);
    if (threadIdx.x < kBwdGroup) {
      s_pre[threadIdx.x] = (int64_t)ex;
      s_off[threadIdx.x] = off;
    }
    if (threadIdx.x == 0) s_pre[kBwdGroup] = (int64_t)total;
    __syncthreads();
    const int64_t n = (int64_t)total;
    auto row_of = [&](int64_t i) {
      int lo = 0;   // the last bucket of the group whose first row is <= i
#pragma unroll
      for (int step = kBwdGroup / 2; step; step >>= 1)
        if (s_pre[lo + step] <= i) lo += step;
      return s_off[lo] + (i - s_pre[lo]);
    };
    uint64_t cx[W], cz[W], nx[W], nz[W];
    double cc = 0.0, nc = 0.0;
    int64_t crow = 0, nrow = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) cx[w] = cz[w] = 0;
    if (threadIdx.x < n) {
      crow = row_of(threadIdx.x);
#pragma unroll
      for (int w = 0; w < W; ++w) {
        cx[w] = __builtin_nontemporal_load(&st.x[w * st.cap + crow]);
        cz[w] = __builtin_nontemporal_load(&st.z[w * st.cap + crow]);
      }
      cc = __builtin_nontemporal_load(&st.c[crow]);
    }
    for (int64_t i0 = 0; i0 < n; i0 += kBwdBlock) {
      const int64_t in = i0 + kBwdBlock + threadIdx.x;
#pragma unroll
      for (int w = 0; w < W; ++w) nx[w] = nz[w] = 0;
      nc = 0.0;
      if (in < n) {
        nrow = row_of(in);
#pragma unroll
        for (int w = 0; w < W; ++w) {
          nx[w] = __builtin_nontemporal_load(&st.x[w * st.cap + nrow]);
          nz[w] = __builtin_nontemporal_load(&st.z[w * st.cap + nrow]);
        }
        nc = __builtin_nontemporal_load(&st.c[nrow]);
      }
      if (i0 + threadIdx.x < n) {
        ++nmine;
        ok = ok && fabs(cc) < 0x1p31;
        cmax = fmax(cmax, fabs(cc));
        bwd_term<W>(lut, thi, tlo, cx, cz, cc, lam ? lam + crow : nullptr, scale);
      }
#pragma unroll
      for (int w = 0; w < W; ++w) { cx[w] = nx[w]; cz[w] = nz[w]; }
      cc = nc;
      crow = nrow;
    }
  }
  // bounds of the exact integer sums (see above), over the workgroup
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    cmax = fmax(cmax, __shfl_xor(cmax, d, 64));
    nmine += __shfl_xor(nmine, d, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    s_cmax[threadIdx.x >> 6] = cmax;
    s_cnt[threadIdx.x >> 6] = nmine;
  }
  if (!ok) s_bad = 1;
  __syncthreads();
  double cm = 0.0;
  long long nwg = 0;
  for (int k = 0; k < kBwdBlock / 64; ++k) {
    cm = fmax(cm, s_cmax[k]);
    nwg += s_cnt[k];
  }
  const bool in_range = s_bad == 0 && nwg < (1ll << 23) && cm * (double)nwg < 0x1p42;
  // the sums as doubles, over the energy table (no longer needed), then the
  // per-qubit factors over the first integer table
  for (int i = threadIdx.x; i < NE; i += kBwdBlock)
    lut[i] = (double)(long long)thi[i] * 0x1p-20 + (double)(long long)tlo[i] * 0x1p-60;
  __syncthreads();
  for (int q = threadIdx.x; q < 64 * W; q += kBwdBlock) {
    double st_ = 0, ct = 1, sp = 0, cp = 1;
    if (q < nq) {
      sincos(theta[q], &st_, &ct);
      sincos(phi[q], &sp, &cp);
    }
    for (int op = 0; op < 4; ++op) fac[4 * q + op] = bloch_factor(op, st_, ct, sp, cp);
  }
  __syncthreads();
  // S[q][sigma] from T: the codes of q's group with sigma at q's position,
  // each weighted by the product of the group's other factors of that code
  for (int k = threadIdx.x; k < 3 * nq; k += kBwdBlock) {
    const int q = k / 3, op = k % 3 + 1;   // op: 1 = X, 2 = Z, 3 = Y
    const int h = q >> 5, bit = q & 31;
    const int g = (int)div3_small((uint32_t)bit), r = bit - 3 * g;
    const double* tg = lut + h * NH + g * kBwdStride;
    double s = 0.0;
    for (int code = 1; code < kLutEntries; ++code) {
      if ((((code >> r) & 1) | (((code >> (3 + r)) & 1) << 1)) != op) continue;
      double other = 1.0;
      bool valid = true;
      for (int r2 = 0; r2 < 3; ++r2) {
        if (r2 == r) continue;
        const int o2 = ((code >> r2) & 1) | (((code >> (3 + r2)) & 1) << 1);
        if (3 * g + r2 >= 32) {   // position past the half word: no qubit
          valid = valid && o2 == 0;
          continue;
        }
        other *= fac[4 * (32 * h + 3 * g + r2) + o2];
      }
      if (valid) s += tg[code] * other;
    }
    acc_g[(int64_t)blockIdx.x * 3 * nq + k] = in_range ? s : __builtin_nan("");
  }
}

template <int W>
static void launch_bwd_w(int nq, const StoreDev& st, int grid, const double* theta,
                         const double* phi, const double* lut, const double* dE, double* lam,
                         double* acc, hipStream_t s) {
  const size_t lds = energy_bwd_lds_bytes(W);
  (void)hipFuncSetAttribute((const void*)k_energy_bwd<W>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)lds);
  hipLaunchKernelGGL(k_energy_bwd<W>, dim3(grid), dim3(kBwdBlock), lds, s, st, nq, theta, phi,
                     lut, dE, lam, acc);
}

void launch_energy_backward(int W, int nq, const StoreDev& st, int grid, const double* theta,
                            const double* phi, const double* lut, const double* dE, double* lam,
                            double* acc, hipStream_t s) {
  switch (W) {
    case 1: launch_bwd_w<1>(nq, st, grid, theta, phi, lut, dE, lam, acc, s); break;
    case 2: launch_bwd_w<2>(nq, st, grid, theta, phi, lut, dE, lam, acc, s); break;
    case 3: launch_bwd_w<3>(nq, st, grid, theta, phi, lut, dE, lam, acc, s); break;
    default: launch_bwd_w<4>(nq, st, grid, theta, phi, lut, dE, lam, acc, s); break;
  }
}

// One workgroup per qubit: S[q][sigma] summed over the per-workgroup
// partials in a fixed order, then the chain rule through the Bloch factors.
__global__ void k_backward_finalize(int nq, int grid, const double* acc, const double* theta,
                                    const double* phi, const double* dE, double* dtheta,
                                    double* dphi) {
  __shared__ double red[kWaves];
  const int q = blockIdx.x;
  double S[3];
  for (int k = 0; k < 3; ++k) {
    double v = 0.0;
    for (int g = threadIdx.x; g < grid; g += kBlock) v += acc[(int64_t)g * 3 * nq + 3 * q + k];
    S[k] = block_sum(v, red);   // valid in thread 0
  }
  if (threadIdx.x == 0) {
    double st, ct, sp, cp;
    sincos(theta[q], &st, &ct);
    sincos(phi[q], &sp, &cp);
    // sigma order X, Z, Y
    const double dt = S[0] * (ct * cp) + S[1] * (-st) + S[2] * (ct * sp);
    const double dp = S[0] * (-st * sp) + S[2] * (st * cp);
    const double sc = dE ? *dE : 1.0;
    dtheta[q] = sc * dt;
    dphi[q] = sc * dp;
  }
}

void launch_backward_finalize(int nq, int grid, const double* acc, const double* theta,
                              const double* phi, const double* dE, double* dtheta, double* dphi,
                              hipStream_t s) {
  if (nq <= 0) return;
  hipLaunchKernelGGL(k_backward_finalize, dim3(nq), dim3(kBlock), 0, s, nq, grid, acc, theta, phi,
                     dE, dtheta, dphi);
}

}  // namespace iqcc
