// QMF energy (Sec. II, Eq. 3; energy functional of App. A) and its gradient
// with respect to the Bloch angles.
//
// <K> of the product state is prod_j b_j(sigma_j) with b(I) = 1,
// b(X) = sin t cos f, b(Y) = sin t sin f, b(Z) = cos t.  Terms are streamed
// once; the product uses a table per group of 4 (or 3) qubits in LDS.  Partial
// sums are per workgroup and reduced in a fixed order.
#include <cfloat>

#include "iqcc_internal.h"
#include "work_split.h"

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

// ---------------------------------------------------------------------------
// Energy of a store in one launch.  Workgroup g takes the groups of G
// consecutive buckets g, g + grid, ... (G up to its threads, so that every workgroup
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
// the x bits low they were 16 entries apart and met in two banks).  Wider keys:
// 3-qubit groups, 22 per word and 64 entries each, because nibble tables would
// leave few waves per CU.
//
// The grid holds what the CUs keep resident (more workgroups would only build
// more tables), and of it as many workgroups take part ("active") as the rows
// and the buckets ask for (energy_buckets): with fewer rows a workgroup would
// spend its time on its table and its arrival, with more on another round of
// bucket searches and loads.
// The active workgroups leave their sums in the finish slot; the last of them
// to arrive adds them in a fixed order, so a call is one launch (two without a
// slot of the stream: 2 to 3 us more).
//
// Bound: HBM for large stores (40 bytes a two-word term), the chain of
// latencies (bucket table, rows, table build, arrival) for small ones.
// 1.6e7 two-word terms: 122 us, 5.2 TB/s (table, sums and reduction in three
// launches: 168 us); 361 terms: 6.6 us (23 us).
// ---------------------------------------------------------------------------
constexpr int kEItems = 4;
constexpr int kNibbleEntries = 256;
constexpr int kNibblesPerWord = 16;

template <int W>
struct EnergyTable {
  static constexpr bool kNibble = W <= 2;
  static constexpr int kEntries = kNibble ? W * kNibblesPerWord * kNibbleEntries : W * kGroupsPerWord * kLutEntries;
  // scratch of the build: the qubits' factors and, for nibbles, the products
  // of the two qubits of every even/odd pair
  static constexpr int kBuild = 64 * W * 4 + (kNibble ? 32 * W * 16 : 0);
};

// The qubits' factors [64 W][4] (I, X, Z, Y), 1.0 past the last qubit.  The
// workgroup's NT threads.
template <int W, int NT>
__device__ __forceinline__ void build_factors(double* fac, int nq, const double* theta, const double* phi) {
  for (int q = NT - 1 - (int)threadIdx.x; q < 64 * W; q += NT) {   // the last threads: the first ones have buckets
    double st = 0.0, ct = 1.0, sp = 0.0, cp = 1.0;
    const bool live = q < nq;
    if (live) {
      sincos(theta[q], &st, &ct);
      sincos(phi[q], &sp, &cp);
    }
#pragma unroll
    for (int op = 0; op < 4; ++op) fac[4 * q + op] = live ? bloch_factor(op, st, ct, sp, cp) : 1.0;
  }
}

// Builds the table from the factors in tmp (the whole workgroup; a barrier has
// to lie between the factors and this, and it ends with one).  Multiplying by
// the identity's factor 1.0 is exact.
template <int W, int NT>
__device__ void build_energy_table(double* lut, double* tmp) {
  const double* fac = tmp;
  if constexpr (EnergyTable<W>::kNibble) {
    double* pair = tmp + 64 * W * 4;   // [32 W][16]: z bits low, x bits high
    for (int e = threadIdx.x; e < 32 * W * 16; e += NT) {
      const int q = 2 * (e >> 4), z = e & 3, x = (e >> 2) & 3;
      pair[e] = fac[4 * q + ((x & 1) | ((z & 1) << 1))] * fac[4 * (q + 1) + ((x >> 1) | ((z >> 1) << 1))];
    }
    __syncthreads();
    for (int e = threadIdx.x; e < EnergyTable<W>::kEntries; e += NT) {
      const int z = e & 15, x = (e >> 4) & 15, gi = e >> 8;
      lut[e] = pair[(2 * gi) * 16 + ((z & 3) | ((x & 3) << 2))] * pair[(2 * gi + 1) * 16 + ((z >> 2) | ((x >> 2) << 2))];
    }
  } else {
    for (int e = threadIdx.x; e < EnergyTable<W>::kEntries; e += NT) {
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

template <int W, int NT>
size_t energy_lds_bytes() {
  // table, its build's scratch, first rows and row prefix sums of a group
  return (size_t)(EnergyTable<W>::kEntries + EnergyTable<W>::kBuild) * 8 + (size_t)NT * 8 +
         (size_t)(NT + 1) * 4;
}

template <int NT>
__device__ __forceinline__ BucketSplit energy_split(const StoreDev& st, unsigned grid) {
  return energy_buckets(*st.total, 1ll << *st.m, grid, NT);
}

// The workgroups' sums in a fixed order, valid in thread 0.
template <int NT>
__device__ __forceinline__ double energy_total(const double* slot, unsigned active, double* red) {
  double t = 0.0;
  for (unsigned k = threadIdx.x; k < active; k += NT) t += finish_get(slot, k);
  return block_sum_n<NT / 64>(t, red);
}

template <int W, int NT>
__global__ __launch_bounds__(NT) void k_energy(StoreDev st, int nq, const double* theta, const double* phi,
                                                     SumSlot sums, double* out) {
  extern __shared__ __align__(16) unsigned char smem_en[];
  double* lut = (double*)smem_en;
  double* tmp = lut + EnergyTable<W>::kEntries;                  // [kBuild]
  int64_t* s_off = (int64_t*)(tmp + EnergyTable<W>::kBuild);     // [NT]
  uint32_t* s_pre = (uint32_t*)(s_off + NT);               // [NT + 1]
  __shared__ double red[NT / 64];
  __shared__ uint64_t scan_tmp[NT / 64];
  __shared__ int s_last;
  const int B = 1 << *st.m;
  const BucketSplit split = energy_split<NT>(st, gridDim.x);
  const int G = split.G, ngroups = split.ngroups, active = split.active;
  if ((int)blockIdx.x >= active) return;
  // (the factors' chain of loads and sines beside that of the bucket table)
  build_factors<W, NT>(tmp, nq, theta, phi);
  bool table = false;
  double acc = 0.0;
  for (int grp = blockIdx.x; grp < ngroups; grp += active) {
    const int b = grp * G + (int)threadIdx.x;
    const bool mine = (int)threadIdx.x < G && b < B;
    const int64_t cnt = mine ? st.cnt[b] : 0;
    const int64_t off = mine ? st.off[b] : 0;
    uint64_t total;
    // (the scan's barriers also order the previous group's reads of s_pre)
    const uint64_t ex = block_exclusive_scan_n<NT / 64>((uint64_t)cnt, scan_tmp, total);
    s_pre[threadIdx.x] = (uint32_t)ex;
    s_off[threadIdx.x] = off;
    if (threadIdx.x == 0) s_pre[NT] = (uint32_t)total;
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
        const uint32_t i = i0 + r * NT + threadIdx.x;
        kc[r] = 0.0;
#pragma unroll
        for (int w = 0; w < W; ++w) kx[r][w] = kz[r][w] = 0;
        if (i < n) {
          int64_t row = base + i;
          if (!contig) {
            int lo = 0;   // the last bucket of the group whose first row is <= i
#pragma unroll
            for (int step = NT / 2; step; step >>= 1)
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
        build_energy_table<W, NT>(lut, tmp);
        table = true;
      }
#pragma unroll
      for (int r = 0; r < kEItems; ++r) acc += kc[r] * expect_table<W>(lut, kx[r], kz[r]);
      i0 += NT * kEItems;
    } while (i0 < n);
  }
  const double s = block_sum_n<NT / 64>(acc, red);
  if (!sums.single) {
    if (threadIdx.x == 0) finish_put(sums.slot, blockIdx.x, s);
    return;
  }
  if (active == 1) {
    if (threadIdx.x == 0) *out = s;
    return;
  }
  if (threadIdx.x < 64) {
    if (threadIdx.x == 0) finish_put(sums.slot, blockIdx.x, s);
    const bool last = finish_arrive(sums.slot, blockIdx.x, active);
    if (threadIdx.x == 0) s_last = last;
  }
  __syncthreads();
  if (s_last) {
    const double t = energy_total<NT>(sums.slot, active, red);
    if (threadIdx.x == 0) *out = t;
  }
}

// The second launch of a call without a slot of its stream.
template <int NT>
__global__ __launch_bounds__(NT) void k_energy_total(StoreDev st, unsigned grid, const double* slot, double* out) {
  __shared__ double red[NT / 64];
  const double t = energy_total<NT>(slot, (unsigned)energy_split<NT>(st, grid).active, red);
  if (threadIdx.x == 0) *out = t;
}

template <int W, int NT>
static void launch_energy_w(int nq, const StoreDev& st, int n_cu, int per_cu, size_t lds_per_cu, const double* theta,
                            const double* phi, const SumSlot& slot, double* out, hipStream_t s) {
  const size_t lds = energy_lds_bytes<W, NT>();
  // resident workgroups per CU: LDS (with the static part), 2048 threads
  int fit = (int)(lds_per_cu / (lds + 256));
  fit = fit < 1 ? 1 : (fit > 2048 / NT ? 2048 / NT : fit);
  int grid = n_cu * (per_cu < fit ? per_cu : fit);
  if (grid > kFinishWords) grid = kFinishWords;
  (void)hipFuncSetAttribute((const void*)k_energy<W, NT>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL((k_energy<W, NT>), dim3(grid), dim3(NT), lds, s, st, nq, theta, phi, slot, out);
  if (!slot.single)
    hipLaunchKernelGGL(k_energy_total<NT>, dim3(1), dim3(NT), 0, s, st, (unsigned)grid, slot.slot, out);
}

// A CU's LDS holds one table of two-word keys.  Where the rows of a store lie in
// bucket regions, each pass also searches its buckets, and the workgroup gets
// 1024 threads, the waves of two (5.4e7 terms 552 us with 512, 499 with 1024);
// loaded rows stream faster with 512 (1.6e7 terms 121 us, 125).
void launch_energy(int W, int nq, const StoreDev& st, bool regions, int n_cu, int per_cu, size_t lds_per_cu, const double* theta,
                   const double* phi, const SumSlot& slot, double* out, hipStream_t s) {
  switch (W) {
    case 1: launch_energy_w<1, 512>(nq, st, n_cu, per_cu, lds_per_cu, theta, phi, slot, out, s); break;
    case 2:
      if (regions) launch_energy_w<2, 1024>(nq, st, n_cu, per_cu, lds_per_cu, theta, phi, slot, out, s);
      else launch_energy_w<2, 512>(nq, st, n_cu, per_cu, lds_per_cu, theta, phi, slot, out, s);
      break;
    case 3: launch_energy_w<3, 512>(nq, st, n_cu, per_cu, lds_per_cu, theta, phi, slot, out, s); break;
    default: launch_energy_w<4, 512>(nq, st, n_cu, per_cu, lds_per_cu, theta, phi, slot, out, s); break;
  }
}

// ---------------------------------------------------------------------------
// Backward w.r.t. the Bloch angles (derivative of the Eq. 3 energy).
// dE/dtheta_q = sum_sigma S[q][sigma] db_sigma/dtheta (likewise phi), where
// S[q][sigma] adds, over the terms with sigma on qubit q, c times the product
// of the term's other factors.
//
// All terms of S[q][sigma] miss the same factor b = b_q(sigma), so
//   S[q][sigma] = (sum of v_k over the terms with sigma on q) / b,
//   v_k = c_k times the product of all of the term's factors,
// with one division at the end.  Factors that are zero or below 2^-100 ("null")
// are left out of v_k instead: a term with one null factor, on qubit q, counts
// only for q and its sigma there (undivided), a term with several counts
// nowhere -- what it would add holds a null factor and is below 2^-69.
//
// The sums are a contraction of the 0/1 matrix (x bits, z bits, x and z bits
// of the keys) with the v_k, and they are made exactly, so that they do not
// depend on the order of the rows: v_k is taken as a fixed-point number
// (resolution 2^-186, |v| < 2^31) of 32 digits of 7 bits, and the matrix cores
// add the digits of all terms per key bit (v_mfma_i32_32x32x32_i8: 32 qubits x
// 32 terms x 32 digits), exactly in 32-bit integers: every kCarryTerms terms the
// digits' carries move up one digit, so no sum passes 2^31; the top digit, which
// holds the signs and the carries out of the others, is below the number of
// terms.  Sums over exactly one of X, Z, Y are integer differences of
// those.  Per workgroup the 32 digit sums turn into one double, and the
// workgroups' doubles are added in a fixed order.  A workgroup that meets a
// non-finite coefficient or angle, |c| >= 2^31, or 2^31 terms writes NaN.
//
// Work split: a team of TW waves takes 64 TW terms at a time.  Each wave makes
// v and its digits, and writes the bytes of its 64 terms' keys to LDS by byte
// and term (the four bytes of a dword change places within four lanes first);
// after a barrier each wave multiplies the bits of "its" 32 qubits with the
// digits of the team's terms (of half of them for one-word keys).  A dword read
// back holds one byte of four terms' keys, so the lane of qubit q has its bit
// operand as (dword >> (q & 7)) & 0x01010101, and the eight lanes of a byte
// read the same address.  (With the keys transposed bit by bit in registers,
// 130 instructions per 64 terms against 40, 4e6 two-word terms took 108 us.)
//
// A workgroup holds three teams (one for wide keys), one wave of each per SIMD,
// and a team has a barrier of its own, so that one team's matrix products run
// beside another's vector work (4e6 two-word terms: four teams of 128 registers,
// some of them in memory, 109 us; three 94 us; a workgroup's barrier in place of
// the teams' and a workgroup per team were 4 % and 16 % slower).  A wave
// arrives at a barrier as soon as its part is done and waits only before it
// needs the others': it makes the next terms' products between the end of its
// matrix products and the wait for the team's, and loads terms between its
// writes and the wait for the team's (one wait at each arrival: 101 us).
//
// Bound: VALU issue (about 510 instructions per 64 two-word terms: 128 for the
// product, 100 for digits and bytes, 160 for the bit operands) and the waits of
// three waves per SIMD; 24 matrix products of 32 cycles run beside.  4e6
// two-word terms: 88 us; with every (term, group) value added to integer tables
// in LDS by two 64-bit atomics 203 us.  1.1e6 one-word terms: 26 us (67 us).
// acc layout: [3 * nq][workgroups] with sigma order X, Z, Y.
// ---------------------------------------------------------------------------
template <int W>
struct BwdGeom {
  static constexpr int kBlocks = 2 * W;                 // 32-qubit blocks
  static constexpr int kTeamWaves = W == 1 ? 4 : 2 * W;
  static constexpr int kTeams = W <= 2 ? 3 : 1;
  static constexpr int kThreads = 64 * kTeamWaves * kTeams;
  static constexpr int kSplit = kTeamWaves / kBlocks;   // waves that share a block's terms
};
constexpr int kDigits = 32;
constexpr int kDigitStride = 80;   // bytes per digit row of 64 terms (padded: 16-byte reads of 8 lanes hit all banks)
constexpr int kDigitBase = -186;   // log2 of the lowest digit's weight
// Terms of a workgroup after which its digit sums are carried: a sum stays below
// 127 x 2 kCarryTerms of new digits and what a carry leaves, 127 + 2 kCarryTerms in
// each wave.
constexpr uint32_t kCarryTerms = 1u << 22;

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

template <int W>
struct BwdShared {
  using T = EnergyTable<W>;
  using B = BwdGeom<W>;
  double lut[T::kEntries];                            // afterwards the digit sums
  double fac[64 * W * 4];
  alignas(16) uint8_t bytes[2][B::kTeams][B::kTeamWaves][8 * W * 64];   // x, z: byte of the key, term
  alignas(16) uint8_t dig[B::kTeams][B::kTeamWaves][kDigits * kDigitStride];
  int64_t s_off[kBwdGroup];
  uint32_t s_pre[kBwdGroup + 1];
  uint64_t null_mask[3][W];                           // qubits whose X, Z, Y factor is null
  uint64_t scan_tmp[B::kThreads / 64];
  unsigned arrived[B::kTeams];
  int bad;
  static_assert(sizeof(bytes) + sizeof(dig) >= sizeof(double) * T::kBuild, "the table is built there");
  static_assert(sizeof(lut) + sizeof(fac) + sizeof(bytes) + sizeof(dig) >= sizeof(int) * 96 * B::kBlocks * kDigits,
                "the digit sums fit");
};

// Bytes of dword d (4 rows of 64 bytes, one byte per term) of every lane's key:
// the 4 x 4 bytes of four lanes are transposed, and each lane writes the dword
// of its row.  sel1, sel2: the lane's byte selectors (see byte_selectors).
__device__ __forceinline__ void put_bytes(uint8_t* rows, int lane, uint32_t a, uint32_t sel1, uint32_t sel2) {
  uint32_t t = (uint32_t)__builtin_amdgcn_mov_dpp((int)a, 0xB1, 0xF, 0xF, false);   // quad_perm 1,0,3,2
  a = __builtin_amdgcn_perm(t, a, sel1);
  t = (uint32_t)__builtin_amdgcn_mov_dpp((int)a, 0x4E, 0xF, 0xF, false);            // quad_perm 2,3,0,1
  a = __builtin_amdgcn_perm(t, a, sel2);
  *reinterpret_cast<uint32_t*>(rows + (lane & 3) * 64 + (lane & ~3)) = a;
}

// Step 1 takes the even (odd) bytes of the even (odd) lane, step 2 the low
// (high) halves of the lanes with bit 1 clear (set).
__device__ __forceinline__ void byte_selectors(int lane, uint32_t& sel1, uint32_t& sel2) {
  sel1 = (lane & 1) ? 0x03070105u : 0x06020400u;
  sel2 = (lane & 2) ? 0x03020706u : 0x05040100u;
}

// Digits of v (|v| < 2^31) into the wave's digit rows, at this lane's term.
__device__ __forceinline__ void put_digits(uint8_t* dig, int lane, double v) {
  const v4i zero = {0, 0, 0, 0};
#pragma unroll
  for (int i = 0; i < 2; ++i) {   // 32 rows of 64 bytes
    const int k = lane + 64 * i;
    *reinterpret_cast<v4i*>(dig + (k >> 2) * kDigitStride + (k & 3) * 16) = zero;
  }
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const int e = (int)(u >> 52) & 0x7FF;
  uint64_t mant = (u & 0xFFFFFFFFFFFFFull) | (e ? 1ull << 52 : 0ull);
  int p = e - 1075 - kDigitBase;   // bit position of the lowest mantissa bit, at most 164
  if (p < 0) {
    mant = p > -64 ? mant >> -p : 0ull;
    p = 0;
  }
  const int d0 = (p * 293) >> 11;   // p / 7, at most 23
  int64_t m = (int64_t)(mant << (p - 7 * d0));
  m = (int64_t)u < 0 ? -m : m;      // two's complement: the last digit carries the sign
  uint8_t* at = dig + d0 * kDigitStride + lane;
  const uint32_t lo = (uint32_t)m, hi = (uint32_t)((uint64_t)m >> 32);
#pragma unroll
  for (int j = 0; j < 4; ++j) at[j * kDigitStride] = (uint8_t)__builtin_amdgcn_ubfe(lo, 7 * j, 7);
  at[4 * kDigitStride] = (uint8_t)(__builtin_amdgcn_alignbit(hi, lo, 28) & 127u);
#pragma unroll
  for (int j = 5; j < 8; ++j) at[j * kDigitStride] = (uint8_t)__builtin_amdgcn_ubfe(hi, 7 * j - 32, 7);
  at[8 * kDigitStride] = (uint8_t)(hi >> 24);
}

// Moves the carry of each digit sum to the next digit, in the next lane; the top
// digit keeps what it has.
__device__ __forceinline__ void carry_digits(v16i& s, int lane) {
  const int d = lane & (kDigits - 1);
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int c = d < kDigits - 1 ? s[i] >> 7 : 0;
    const int up = __shfl_up(c, 1, kDigits);
    s[i] += (d ? up : 0) - c * 128;
  }
}

// Barrier of one team's `waves` waves, in two halves, between which a wave does
// what needs no other wave: an arrival counter in LDS that only grows (`target`
// is the wave's own count of what it has to reach).  All waves of a workgroup
// are resident, and every wave of a team passes the same barriers in the same
// order, so each wait ends.
__device__ __forceinline__ void team_arrive(unsigned* arrived, unsigned& target, unsigned waves) {
  target += waves;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");   // this wave's LDS accesses are done
  if ((threadIdx.x & 63) == 0) __hip_atomic_fetch_add(arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ void team_wait(const unsigned* arrived, unsigned target) {
  while ((int)(target - __hip_atomic_load(arrived, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) > 0)
    __builtin_amdgcn_s_sleep(1);
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

template <int W>
__global__ __launch_bounds__(BwdGeom<W>::kThreads) void k_energy_bwd(StoreDev st, int nq, const double* theta,
                                                                     const double* phi, const double* dE,
                                                                     double* lam, double* acc_g) {
  using BG = BwdGeom<W>;
  constexpr int NT = BG::kThreads, NB = BG::kBlocks, TW = BG::kTeamWaves;
  extern __shared__ __align__(16) unsigned char smem_bwd[];
  BwdShared<W>& sh = *reinterpret_cast<BwdShared<W>*>(smem_bwd);
  const int B = 1 << *st.m;
  const BucketSplit split = gradient_buckets(*st.total, B, gridDim.x, NT);
  const int active = split.active, G = split.G, ngroups = split.ngroups;
  if ((int)blockIdx.x >= active) return;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int team = wave / TW, tw = wave % TW, block = tw % NB, part = tw / NB;
  // factors, their null masks, and the table of the factors without the null ones
  double* tmp = reinterpret_cast<double*>(sh.bytes);
  if (threadIdx.x == 0) sh.bad = 0;
  if (threadIdx.x < BG::kTeams) sh.arrived[threadIdx.x] = 0u;
  unsigned target = 0;
  for (int i = threadIdx.x; i < 3 * W; i += NT) (&sh.null_mask[0][0])[i] = 0ull;
  build_factors<W, NT>(sh.fac, nq, theta, phi);
  __syncthreads();
  bool null_here = false;
  for (int i = threadIdx.x; i < 64 * W * 4; i += NT) {
    const int q = i >> 2, op = i & 3;
    const double f = sh.fac[i];
    const bool null = fabs(f) < 0x1p-100;
    if (null) {
      atomicOr((unsigned long long*)&sh.null_mask[op == 1 ? 0 : op == 2 ? 1 : 2][q >> 6], 1ull << (q & 63));
      null_here = true;
    }
    tmp[i] = null ? 1.0 : f;
    if (op == 0 && q < nq && !(fabs(theta[q]) <= DBL_MAX && fabs(phi[q]) <= DBL_MAX)) sh.bad = 1;
  }
  const bool any_null = __syncthreads_or(null_here) != 0;
  build_energy_table<W, NT>(sh.lut, tmp);
  uint32_t sel1, sel2;
  byte_selectors(lane, sel1, sel2);
  const double scale = dE ? *dE : 1.0;
  bool ok = true;   // every coefficient finite and below 2^31 in magnitude, below 2^31 terms
  uint32_t nwg = 0;   // terms of the workgroup
  v16i sx, sz, sy;
#pragma unroll
  for (int i = 0; i < 16; ++i) sx[i] = sz[i] = sy[i] = 0;
  // Workgroup g takes the groups of G consecutive buckets g, g + active, ...;
  // a group's rows are one flat range, one term per thread and pass, the next
  // pass's term loaded while this one's bits are multiplied.
  // A group of more than kCarryTerms rows is walked in parts, i_first the first row.
  uint32_t i_first = 0;
  for (int grp = blockIdx.x; grp < ngroups;) {
    const int b = grp * G + (int)threadIdx.x;
    const bool mine = (int)threadIdx.x < G && b < B;
    const int64_t cnt = mine ? st.cnt[b] : 0;
    const int64_t off = mine ? st.off[b] : 0;
    uint64_t total;
    // (the scan's barriers also order the previous group's reads of s_pre)
    const uint64_t ex = block_exclusive_scan_n<NT / 64>((uint64_t)cnt, sh.scan_tmp, total);
    if (threadIdx.x < kBwdGroup) {
      sh.s_pre[threadIdx.x] = (uint32_t)ex;
      sh.s_off[threadIdx.x] = off;
    }
    if (threadIdx.x == 0) sh.s_pre[kBwdGroup] = (uint32_t)total;
    __syncthreads();
    const int64_t base = sh.s_off[0];   // one range of rows, as in the energy
    const bool contig = __syncthreads_and(!mine || off - (int64_t)ex == base) != 0;
    constexpr uint32_t kPart = kCarryTerms / NT * NT;
    const uint32_t n = (uint32_t)total - i_first < kPart ? (uint32_t)total : i_first + kPart;
    uint64_t kx[W], kz[W];
    double c;
    int64_t row;
    auto load = [&](uint32_t i) {
      c = 0.0;
      row = 0;
#pragma unroll
      for (int w = 0; w < W; ++w) kx[w] = kz[w] = 0;
      if (i < n) {
        row = base + i;
        if (!contig) {
          int lo = 0;   // the last bucket of the group whose first row is <= i
#pragma unroll
          for (int step = kBwdGroup / 2; step; step >>= 1)
            if (sh.s_pre[lo + step] <= i) lo += step;
          row = sh.s_off[lo] + (i - sh.s_pre[lo]);
        }
#pragma unroll
        for (int w = 0; w < W; ++w) {
          kx[w] = __builtin_nontemporal_load(&st.x[w * st.cap + row]);
          kz[w] = __builtin_nontemporal_load(&st.z[w * st.cap + row]);
        }
        c = __builtin_nontemporal_load(&st.c[row]);
      }
    };
    load(i_first + threadIdx.x);
    for (uint32_t i0 = i_first; i0 < n; i0 += NT) {
      const bool live = i0 + threadIdx.x < n;
      const bool has_terms = i0 + 64 * wave < n;   // of the wave
      double v = 0.0, all = 1.0;
      if (has_terms) {
        all = expect_table<W>(sh.lut, kx, kz);
        v = c * all;
        if (any_null) {
          uint64_t nm[W];
          int nn = 0;
#pragma unroll
          for (int w = 0; w < W; ++w) {
            nm[w] = (kx[w] & ~kz[w] & sh.null_mask[0][w]) | (kz[w] & ~kx[w] & sh.null_mask[1][w]) |
                    (kx[w] & kz[w] & sh.null_mask[2][w]);
            nn += __popcll(nm[w]);
          }
          if (nn) {
#pragma unroll
            for (int w = 0; w < W; ++w) {
              for (uint64_t t = nm[w]; t; t &= t - 1) {
                const int q = __builtin_ctzll(t);
                all *= sh.fac[4 * (64 * w + q) + ((int)((kx[w] >> q) & 1) | ((int)((kz[w] >> q) & 1) << 1))];
              }
            }
#pragma unroll
            for (int w = 0; w < W; ++w) { kx[w] &= nm[w]; kz[w] &= nm[w]; }
            if (nn > 1) v = 0.0;
          }
        }
        ok = ok && fabs(c) < 0x1p31;
        if (lam && live) lam[row] = scale * all;
      }
      team_wait(&sh.arrived[team], target);   // the team has read the last pass's digits
      if (has_terms) {
        put_digits(sh.dig[team][tw], lane, fabs(v) < 0x1p31 ? v : 0.0);   // (c = 0 past the last row)
#pragma unroll
        for (int w = 0; w < W; ++w) {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            put_bytes(sh.bytes[0][team][tw] + (2 * w + h) * 256, lane, (uint32_t)(kx[w] >> (32 * h)), sel1, sel2);
            put_bytes(sh.bytes[1][team][tw] + (2 * w + h) * 256, lane, (uint32_t)(kz[w] >> (32 * h)), sel1, sel2);
          }
        }
      }
      team_arrive(&sh.arrived[team], target, TW);
      load(i0 + NT + threadIdx.x);
      team_wait(&sh.arrived[team], target);
#pragma unroll 1
      for (int p = part; p < TW; p += BG::kSplit) {
        if (i0 + 64 * (team * TW + p) >= n) break;
        const int at = (4 * block + ((lane >> 3) & 3)) * 64 + (lane >> 5) * 16;
        const uint8_t* dg = sh.dig[team][p] + (lane & 31) * kDigitStride + (lane >> 5) * 16;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
          const v4i bx = *reinterpret_cast<const v4i*>(sh.bytes[0][team][p] + at + 32 * kb);
          const v4i bz = *reinterpret_cast<const v4i*>(sh.bytes[1][team][p] + at + 32 * kb);
          const v4i bd = *reinterpret_cast<const v4i*>(dg + 32 * kb);
          v4i ax, az, ay;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            ax[i] = (int)(((uint32_t)bx[i] >> (lane & 7)) & 0x01010101u);
            az[i] = (int)(((uint32_t)bz[i] >> (lane & 7)) & 0x01010101u);
            ay[i] = ax[i] & az[i];
          }
          sx = __builtin_amdgcn_mfma_i32_32x32x32_i8(ax, bd, sx, 0, 0, 0);
          sz = __builtin_amdgcn_mfma_i32_32x32x32_i8(az, bd, sz, 0, 0, 0);
          sy = __builtin_amdgcn_mfma_i32_32x32x32_i8(ay, bd, sy, 0, 0, 0);
        }
      }
      team_arrive(&sh.arrived[team], target, TW);
    }
    const uint32_t done = nwg + (n - i_first);
    if ((done ^ nwg) / kCarryTerms) {
      carry_digits(sx, lane);
      carry_digits(sz, lane);
      carry_digits(sy, lane);
    }
    nwg = done;
    ok = ok && nwg < 1u << 31;
    i_first = n < (uint32_t)total ? n : 0u;
    if (i_first == 0) grp += active;
  }
  if (!ok) sh.bad = 1;
  __syncthreads();
  const bool in_range = sh.bad == 0;
  // digit sums of all waves (x or z alone: less the sums over both), over the
  // table and what follows it; then one double per (qubit, sigma).  Column d of
  // row r sits at d ^ (r mod 32): both the adds (one row, all columns) and the
  // reads (one column, all rows) touch every bank once.
  int* sums = reinterpret_cast<int*>(sh.lut);   // [3][32 NB][kDigits]
  for (int i = threadIdx.x; i < 3 * 32 * NB * kDigits; i += NT) sums[i] = 0;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int r = 32 * block + 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3);
    const int at = r * kDigits + ((lane & 31) ^ (r & 31));
    atomicAdd(&sums[at], sx[i] - sy[i]);
    atomicAdd(&sums[32 * NB * kDigits + at], sz[i] - sy[i]);
    atomicAdd(&sums[64 * NB * kDigits + at], sy[i]);
  }
  __syncthreads();
  for (int k = threadIdx.x; k < 3 * 32 * NB; k += NT) {
    const int sg = k / (32 * NB), q = k % (32 * NB);
    if (q >= nq) continue;
    int dg[kDigits];
#pragma unroll
    for (int d = 0; d < kDigits; ++d) dg[d] = sums[k * kDigits + (d ^ (k & 31))];
    // carries moved up, then the digits from the top (a negative sum has a
    // negative carry out of the top digit)
    int carry = 0;
#pragma unroll
    for (int d = 0; d < kDigits; ++d) {
      const int t = dg[d] + carry;   // below 2^31
      dg[d] = t & 127;
      carry = t >> 7;
    }
    double s = (double)carry;
#pragma unroll
    for (int d = kDigits - 1; d >= 0; --d) s = s * 128.0 + (double)dg[d];
    acc_g[(int64_t)(3 * q + sg) * gridDim.x + blockIdx.x] = in_range ? s * 0x1p-186 : __builtin_nan("");
  }
}

template <int W>
static int launch_bwd_w(int nq, const StoreDev& st, int grid, const double* theta, const double* phi,
                        const double* dE, double* lam, double* acc, hipStream_t s) {
  const size_t lds = sizeof(BwdShared<W>);
  (void)hipFuncSetAttribute((const void*)k_energy_bwd<W>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL(k_energy_bwd<W>, dim3(grid), dim3(BwdGeom<W>::kThreads), lds, s, st, nq, theta, phi, dE, lam,
                     acc);
  return BwdGeom<W>::kThreads;
}

// One workgroup per qubit: S[q][sigma] summed over the workgroups in a fixed
// order and divided by the factor it misses, then the chain rule through the
// Bloch factors.
__global__ __launch_bounds__(kBlock) void k_backward_finalize(StoreDev st, int threads, int grid, const double* acc,
                                                              const double* theta, const double* phi,
                                                              const double* dE, double* dtheta, double* dphi) {
  __shared__ double red[kWaves];
  const int q = blockIdx.x;
  const int active = (int)gradient_buckets(*st.total, 1ll << *st.m, grid, threads).active;
  double S[3] = {0.0, 0.0, 0.0};
  for (int g = threadIdx.x; g < active; g += kBlock) {
#pragma unroll
    for (int k = 0; k < 3; ++k) S[k] += acc[(int64_t)(3 * q + k) * grid + g];
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) S[k] = block_sum(S[k], red);   // valid in thread 0
  if (threadIdx.x == 0) {
    double sn, ct, sp, cp;
    sincos(theta[q], &sn, &ct);
    sincos(phi[q], &sp, &cp);
    // sigma order X, Z, Y
    const int ops[3] = {1, 2, 3};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const double b = bloch_factor(ops[k], sn, ct, sp, cp);
      if (!(fabs(b) < 0x1p-100)) S[k] /= b;
    }
    const double dt = S[0] * (ct * cp) + S[1] * (-sn) + S[2] * (ct * sp);
    const double dp = S[0] * (-sn * sp) + S[2] * (sn * cp);
    const double sc = dE ? *dE : 1.0;
    dtheta[q] = sc * dt;
    dphi[q] = sc * dp;
  }
}

void launch_energy_backward(int W, int nq, const StoreDev& st, int grid, const double* theta, const double* phi,
                            const double* dE, double* lam, double* acc, double* dtheta, double* dphi, hipStream_t s) {
  if (nq <= 0) return;
  int threads = 0;
  switch (W) {
    case 1: threads = launch_bwd_w<1>(nq, st, grid, theta, phi, dE, lam, acc, s); break;
    case 2: threads = launch_bwd_w<2>(nq, st, grid, theta, phi, dE, lam, acc, s); break;
    case 3: threads = launch_bwd_w<3>(nq, st, grid, theta, phi, dE, lam, acc, s); break;
    default: threads = launch_bwd_w<4>(nq, st, grid, theta, phi, dE, lam, acc, s); break;
  }
  hipLaunchKernelGGL(k_backward_finalize, dim3(nq), dim3(kBlock), 0, s, st, threads, grid, acc, theta, phi, dE,
                     dtheta, dphi);
}

}  // namespace iqcc
