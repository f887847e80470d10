// Algorithm 2 ("Given projection, computing hashcode"; App A.3, hashing
// kernel) with the projections on the matrix cores and every sign certified
// against the fixed-order fp64 arithmetic of bpc_hash_keys.
//
// The iterative residual r_{i+1} = r_i - u_i P_i makes bit i depend on the
// signs before it only through the Gram matrix of P:
//
//     a_i = r_i . P_i = k . P_i - sum_{t<i} u_t (P_t . P_i),
//
// so the N x L products k . P_i are one dense contraction (K times P^T), and
// what stays sequential per key is an L x L triangle of corrections.  The
// contraction runs as bf16 MFMA: a bf16 key times fp32 P is exact once P is
// cut into three bf16 parts (hi + mid + lo, by truncation, exactly P), and
// the products accumulate in fp32.  The corrections run in fp32 on the
// vector units with the Gram matrix (fp64, rounded to fp32) as wavefront-
// uniform operands; at L >= 64 the corrections by earlier 16-bit blocks are
// one more bf16 contraction (signs +-1 times the Gram entries cut like P,
// the hi products in a chain of their own) and only each block's own
// triangle stays on the vector units.
//
// The fp32 value a^ differs from the value a the fixed-order fp64 reference
// computes (canonical residual, four-block dot) by at most
//
//   E_i = 136 u S + (i + 2) u (|a^| + 2.01 C_i) + (36 + i) 2^-53 (S + Q_i)
//         + |k| 2^-100 + 2^-110,                     u = 2^-24,
//
// S = |k| |P_i| >= sum_d |k_d P_id| (Cauchy-Schwarz), C_i = sum_{t<i}
// |P_t . P_i| (inflated for the Gram matrix's own fp64 error), Q_i =
// sum_d (sum_t |P_td|) |P_id|.  The first term is fp32 accumulation inside
// the MFMA chains (each of the four 32-coordinate hi-part steps adds at most
// 32 roundings of the running sum; the mid and lo parts, 2^-8 and 2^-16 of
// the size, are accumulated apart and added once), the second the
// corrections and the Gram matrix's rounding to fp32, the third the
// reference's own rounding (i rounded subtractions per coordinate and the
// 34 roundings of a four-block dot), the last two underflow of bf16 parts
// and products.  With the corrections on the matrix cores the bound takes
// 138 u S, (i + 4) in place of (i + 2) before 2.01 C_i, and 2^-109: the
// mid/lo chain gains at most 32 roundings per earlier block of sums below
// 2^-7 (S + C_i), the hi chain at most 16 T roundings of sums below C_i, and
// one addition joins it.  The evaluation of E_i in fp32 is covered by a factor
// 1 + 2^-8.  When |a^| > E_i + 1.01e-6 the reference's sign is that of a^,
// and |fp32(a)| >= 1e-6, so the decision is not fragile.  Otherwise (a few
// keys in ten thousand, and every decision near zero), the wavefront
// recomputes that one decision in the reference arithmetic: the residual
// rebuilt from the bf16 key with one rounded subtraction per earlier bit, in
// order, and the four-block dot; the fragile test is then the reference's.
// Non-finite values make every comparison fail and take the same route.

//
// Where more than kHmMany of a tile's 64 keys are uncertain in one block of
// bits (rank-deficient keys, a P that fits them exactly) the whole tile is
// decided in the reference arithmetic, four lanes per key; rows of P that are
// zero, and the first other row for keys that are zero, need neither.
//
// What bounds it: vector issue and LDS reads (each block's triangle of
// corrections, its operands read uniformly from LDS), at two wavefronts per
// SIMD.  Batch 16 x 8 heads x 131072 keys, L = 64: 1.90 ms (2.67 before the
// parts of P were cut once per workgroup, the certificate was folded into one
// multiply-add per bit, the next tile's keys were loaded during the last block's
// decisions and the set-up moved to the fp64 matrix cores; of these 0.5 came when
// 20 registers were no longer spilled); 8 x 1048576 keys, L = 128: 4.4 ms (5.40);
// 8 x 8192 keys, L = 64, mostly set-up: 32 us (64).

#include "bpc_internal.h"
#include "mfma_split.h"

namespace bpc {

// 64 keys per wavefront per iteration; eight wavefronts per workgroup at
// L >= 64, where one workgroup takes most of a CU's LDS, else four
template <int L>
constexpr int hm_threads() { return L >= 64 ? 512 : 256; }
// Up to L = 64 the bf16 parts of P (and of the Gram entries the matrix-core
// corrections read) are kept in LDS in operand order beside the fp32 P, cut
// once per workgroup; at L = 128 they do not fit and every wavefront cuts them
// again for each 64 keys.  Cutting them each time was 1200 of 4300 vector
// instructions per 64 keys at L = 64.
template <int L>
constexpr bool hm_parts() { return L <= 64; }
constexpr int kHmPsStride = 132;     // fp32 P row stride in LDS (floats)
constexpr int kHmXsStride = 20;      // transpose buffer row stride (floats)

// Decision `bit` of one key in the reference arithmetic, computed by the
// whole wavefront: lane l carries coordinates l and l + 64 of the residual,
// rebuilt from the bf16 key with one rounded subtraction per earlier bit in
// ascending order; the products are rounded, then each block of 32
// coordinates is summed in ascending order from +0 and the blocks combined
// as ((b0 + b1) + (b2 + b3)).  krow and u0..u3 (the key's code words so far)
// are the same in every lane; fb is the wavefront's scratch of 128 doubles.
__device__ __forceinline__ double hm_reference_decision(const uint16_t* krow, const float* Ps, int bit, uint32_t u0,
                                                     uint32_t u1, uint32_t u2, uint32_t u3, double* fb) {
  const int l = threadIdx.x & 63;
  double r0 = bf16_to_f64(krow[l]), r1 = bf16_to_f64(krow[l + 64]);
  for (int t = 0; t < bit; ++t) {
    const int q = t >> 5;
    const uint32_t word = q == 0 ? u0 : q == 1 ? u1 : q == 2 ? u2 : u3;
    const bool ut = (word >> (t & 31)) & 1u;
    const double p0 = (double)Ps[t * kHmPsStride + l], p1 = (double)Ps[t * kHmPsStride + l + 64];
    r0 = ut ? r0 - p0 : r0 + p0;
    r1 = ut ? r1 - p1 : r1 + p1;
  }
  fb[l] = dmul(r0, (double)Ps[bit * kHmPsStride + l]);
  fb[64 + l] = dmul(r1, (double)Ps[bit * kHmPsStride + l + 64]);
  wave_lds_sync();
  double s = 0.0;
  if (l < 4) {
#pragma unroll 8
    for (int e = 0; e < 32; ++e) s = dadd(s, fb[32 * l + e]);
  }
  const double s0 = readlane_f64(s, 0), s1 = readlane_f64(s, 1), s2 = readlane_f64(s, 2), s3 = readlane_f64(s, 3);
  wave_lds_sync();  // fb is rewritten by the next call only after these reads
  return dadd(dadd(s0, s1), dadd(s2, s3));
}

// The Gram matrix by rows, each row t holding the 16-wide column blocks from
// t's own block on: G[t][i] (t < i) at hm_gram_row<L>(t) + i - 16 (t / 16).
template <int L>
__device__ __forceinline__ int hm_gram_row(int t) {
  constexpr int nb = L / 16;
  const int a = t >> 4, r = t & 15;
  return 16 * (16 * (nb * a - a * (a - 1) / 2) + r * (nb - a));
}
template <int L>
constexpr int hm_gram_size() { return 256 * (L / 16) * (L / 16 + 1) / 2; }

// At L >= 64 the corrections by earlier blocks run on the matrix cores (see
// the main loop), and the Gram matrix (the same size) is kept as the 16 x 16
// diagonal blocks (row t, column i % 16 at 256 (t / 16) + 16 (t % 16) +
// i % 16), then, for every bit i of block T >= 1, the 16 T entries G[t][i],
// t < 16 T, contiguous (the matrix-core operand reads 8 consecutive t).
template <int L>
constexpr bool hm_mm_corr() { return L >= 64; }
template <int L>
__device__ __forceinline__ int hm_gram_col(int i) {  // the entries G[t][i], t < 16 (i / 16)
  constexpr int nb = L / 16;
  const int T = i >> 4;
  return 256 * nb + 256 * (T * (T - 1) / 2) + 16 * T * (i & 15);
}
// the index of G[t][i], t < i
template <int L>
__device__ __forceinline__ int hm_gram_at(int t, int i) {
  if constexpr (hm_mm_corr<L>()) {
    if ((t >> 4) == (i >> 4)) return 256 * (t >> 4) + 16 * (t & 15) + (i & 15);
    return hm_gram_col<L>(i) + t;
  } else {
    return hm_gram_row<L>(t) + i - 16 * (t >> 4);
  }
}
// G[t][16 (t / 16) .. + 15], the row of t inside its own column block
template <int L>
__device__ __forceinline__ int hm_gram_diag(int t) {
  if constexpr (hm_mm_corr<L>()) return 256 * (t >> 4) + 16 * (t & 15);
  else return hm_gram_row<L>(t);
}

// Eight bf16 operands +-1 from the bits of `byte` (bit set: -1), low half of
// each word first; all zero when !on
__device__ __forceinline__ uint4 sign_operand(uint32_t byte, bool on) {
  uint32_t w[4];
#pragma unroll
  for (int k = 0; k < 4; ++k)
    w[k] = on ? (0x3F803F80u | (((byte >> (2 * k)) & 1u) << 15) | (((byte >> (2 * k + 1)) & 1u) << 31)) : 0u;
  return make_uint4(w[0], w[1], w[2], w[3]);
}

// All decisions of 64 keys in the reference arithmetic, for tiles in which many
// are uncertain: four lanes per key, lane q of a quad holding the fp64
// residual of coordinates [32 q, 32 q + 32), 16 keys at a time.  Writes the
// code words and returns the lane's count of fragile decisions.
template <int L>
__device__ __forceinline__ unsigned int hm_reference_tile(const uint16_t* Kb, int64_t sK_n, int base, int key_end,
                                                          const float* Ps, uint32_t* Cb) {
  constexpr int W = L / 32;
  const int lane = threadIdx.x & 63, qd = lane & 3;
  unsigned int nfrag = 0;
#pragma unroll 1
  for (int pass = 0; pass < 4; ++pass) {
    const int key = base + 16 * pass + (lane >> 2);
    const bool valid = key < key_end;
    const uint16_t* row = Kb + (int64_t)(valid ? key : base) * sK_n + 32 * qd;
    double r[32];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint4 v = *reinterpret_cast<const uint4*>(row + 8 * q);
      const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int e = 0; e < 8; ++e)
        r[8 * q + e] = bf16_to_f64((uint16_t)((e & 1) ? (w[e >> 1] >> 16) : (w[e >> 1] & 0xFFFFu)));
    }
    uint32_t word = 0u;
#pragma unroll 1
    for (int i = 0; i < L; ++i) {
      const float* p = Ps + i * kHmPsStride + 32 * qd;
      double acc = 0.0;
#pragma unroll
      for (int e = 0; e < 32; ++e) acc = dadd(acc, dmul(r[e], (double)p[e]));
      const double s01 = dadd(acc, __shfl_xor(acc, 1, 64));
      const double a = dadd(s01, __shfl_xor(s01, 2, 64));
      const bool u = a >= 0.0;
      if (qd == 0 && valid && fragile_decision(a)) ++nfrag;
      if ((i >> 5) == qd && u) word |= 1u << (i & 31);
      const double sg = u ? -1.0 : 1.0;
#pragma unroll
      for (int e = 0; e < 32; ++e) r[e] = __builtin_fma(sg, (double)p[e], r[e]);
    }
    if (valid && qd < W) Cb[(int64_t)key * W + qd] = word;
  }
  return nfrag;
}
// uncertain keys in one block of 16 bits above which the tile is done so
constexpr int kHmMany = 24;

typedef double f64x4_t __attribute__((ext_vector_type(4)));

template <int L>
struct HmShared {
  float Ps[L * kHmPsStride];              // P of this (b, h), fp32
  float Gs[hm_gram_size<L>()];            // fp32(P_t . P_i) for t < i, at hm_gram_at(t, i)
  float2 cst[L];                          // per bit: e1, e3 of the bound |k| e1 + e3 on |a^|
  uint32_t emax[2];                       // their maxima, as bits
  uint4 Pp[hm_parts<L>() ? (L / 16) * 4 * 3 * 64 : 1];   // parts of P: ((T 4 + m) 3 + part) 64 + lane
  uint4 Gp[L == 64 ? 4 * 3 * 64 : 1];     // parts of G: ((T T / 4 + st) 3 + part) 64 + lane
  float Xs[hm_threads<L>() / 64][64 * kHmXsStride];  // per wavefront: MFMA tile -> one key per lane (also setup scratch)
  double fb[hm_threads<L>() / 64][kHeadDim];  // per wavefront: the products of one reference decision
  unsigned int nzero;                     // zero rows of P
  unsigned int first;                     // the first row that is not zero (L: none)
  unsigned int nfrag, nfall;
};

template <int L>
__global__ __launch_bounds__(hm_threads<L>(), 2) void hash_mm_kernel(const uint16_t* __restrict__ K, int64_t sK_b,
                                                             int64_t sK_h, int64_t sK_n, int Hkv, int N,
                                                             const float* __restrict__ P, int64_t sP_b, int64_t sP_h,
                                                             uint32_t* __restrict__ codes, int64_t sC_b,
                                                             int64_t sC_h, unsigned long long* __restrict__ fragile,
                                                             unsigned long long* __restrict__ fallbacks,
                                                             int keys_per_wg) {
  constexpr int W = L / 32;
  constexpr int kHmThreads = hm_threads<L>();
  constexpr int NWV = kHmThreads / 64;
  __shared__ __align__(16) HmShared<L> sh;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int bh = blockIdx.y;
  const int b = bh / Hkv, h = bh % Hkv;
  const float* Pb = P + b * sP_b + h * sP_h;
  const uint16_t* Kb = K + b * sK_b + h * sK_h;

  // ---- set-up: P, its Gram matrix and the per-bit bound constants ----------
  for (int e = tid; e < L * 32; e += kHmThreads) {
    const int i = e >> 5, c = e & 31;
    *reinterpret_cast<float4*>(&sh.Ps[i * kHmPsStride + 4 * c]) = reinterpret_cast<const float4*>(Pb)[e];
  }
  if (tid == 0) sh.nfrag = 0, sh.nfall = 0, sh.nzero = 0, sh.first = L, sh.emax[0] = 0u, sh.emax[1] = 0u;
  __syncthreads();
  double* Ad = reinterpret_cast<double*>(&sh.Xs[0][0]);  // sum_t |P_td|, [128]
  double* nP = Ad + kHeadDim;                             // |P_t| in fp64, [L]
  {
    // The Gram matrix on the fp64 matrix cores: one 16 x 16 block (a, b), a <= b,
    // per wavefront and turn; lane l supplies row l % 16 and coordinate 4 k +
    // l / 16 of either operand and holds rows 4 j + l / 16 of column l % 16.
    constexpr int nb = L / 16;
    const int r16 = lane & 15, k4 = lane >> 4;
    for (int pr = wave; pr < nb * (nb + 1) / 2; pr += NWV) {
      int ba = 0, off = pr;
      while (off >= nb - ba) off -= nb - ba, ++ba;
      const int bb = ba + off;
      const float* pa = &sh.Ps[(16 * ba + r16) * kHmPsStride + k4];
      const float* pb = &sh.Ps[(16 * bb + r16) * kHmPsStride + k4];
      f64x4_t g = (f64x4_t){0.0, 0.0, 0.0, 0.0};
#pragma unroll 8
      for (int k = 0; k < kHeadDim; k += 4)
        g = __builtin_amdgcn_mfma_f64_16x16x4f64((double)pa[k], (double)pb[k], g, 0, 0, 0);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int t = 16 * ba + 4 * j + k4, i = 16 * bb + r16;
        if (t < i) sh.Gs[hm_gram_at<L>(t, i)] = (float)g[j];
      }
    }
  }
  // sum_t |P_td| and |P_t|: several lanes of a wavefront each
  {
    constexpr int S = kHmThreads / kHeadDim;
    const int d = tid / S, s = tid % S;
    double a = 0.0;
#pragma unroll 4
    for (int t = s; t < L; t += S) a += fabs((double)sh.Ps[t * kHmPsStride + d]);
#pragma unroll
    for (int o = 1; o < S; o <<= 1) a += __shfl_xor(a, o, 64);
    if (s == 0) Ad[d] = a;
  }
  constexpr int SB = kHmThreads / L;  // lanes per bit
  {
    const int t = tid / SB, s = tid % SB;
    double a = 0.0;
#pragma unroll 4
    for (int d = s; d < kHeadDim; d += SB) {
      const double x = (double)sh.Ps[t * kHmPsStride + d];
      a = fma(x, x, a);
    }
#pragma unroll
    for (int o = 1; o < SB; o <<= 1) a += __shfl_xor(a, o, 64);
    if (s == 0) nP[t] = sqrt(a) * (1.0 + 0x1p-40);
  }
  __syncthreads();
  const int cbit = tid / SB, csub = tid % SB;
  double cabs = 0.0, q = 0.0;
  for (int t = csub; t < cbit; t += SB)
    cabs += fabs((double)sh.Gs[hm_gram_at<L>(t, cbit)]) + 0x1p-20 * nP[t] * nP[cbit];
#pragma unroll 4
  for (int d = csub; d < kHeadDim; d += SB) q += Ad[d] * fabs((double)sh.Ps[cbit * kHmPsStride + d]);
#pragma unroll
  for (int o = 1; o < SB; o <<= 1) cabs += __shfl_xor(cabs, o, 64), q += __shfl_xor(q, o, 64);
  if (csub == 0) {
    const int i = cbit;
    const double up = 1.0 + 0x1p-20;
    // with the corrections on the matrix cores: two more roundings of
    // 2^-7-sized sums per earlier bit in the mid/lo chain (+2 u S, +2 u C_i)
    constexpr bool mm = hm_mm_corr<L>();
    const double c1 = ((mm ? 138.0 : 136.0) * 0x1p-24 + (36.0 + i) * 0x1p-53) * up;
    const double c2 = (i + 2.0) * 0x1p-24;
    const double c3 = ((i + (mm ? 4.0 : 2.0)) * 0x1p-24 * 2.01 * cabs + q * (36.0 + i) * 0x1p-53 +
                       (mm ? 0x1p-109 : 0x1p-110) + 1.01e-6) *
                      up;
    // |a^| > (|k| (|P_i| c1 + 2^-100) + c2 |a^| + c3) (1 + 2^-8), solved for |a^|
    const double f = (1.0 + 0x1p-8) / (1.0 - c2 * (1.0 + 0x1p-8)) * up;
    const float e1 = (float)((nP[i] * up * c1 + 0x1p-100) * f * up), e3 = (float)(c3 * f * up);
    sh.cst[i] = make_float2(e1, e3);
    // A zero row of P gives a = +0 for every finite key: u = +1 and fragile,
    // counted per key below.  A bound below zero lets it pass as certain (and
    // not when |k| is infinite or NaN).
    if (nP[i] == 0.0) {
      sh.cst[i] = make_float2(0.f, -3e38f);
      atomicAdd(&sh.nzero, 1u);
    } else {
      atomicMin(&sh.first, (unsigned int)i);
      // (infinite and NaN bounds have the largest bits)
      atomicMax(&sh.emax[0], __float_as_uint(e1) & 0x7FFFFFFFu);
      atomicMax(&sh.emax[1], __float_as_uint(e3) & 0x7FFFFFFFu);
    }
  }
  if constexpr (hm_parts<L>()) {
    for (int e = tid; e < (L / 16) * 4 * 64; e += kHmThreads) {
      const int l = e & 63, m = (e >> 6) & 3, T = e >> 8;
      const float* prow = &sh.Ps[(16 * T + (l & 15)) * kHmPsStride + 32 * m + 8 * (l >> 4)];
      uint4* o = &sh.Pp[(T * 4 + m) * 3 * 64 + l];
      split3(*reinterpret_cast<const float4*>(prow), *reinterpret_cast<const float4*>(prow + 4), o[0], o[64], o[128]);
    }
  }
  if constexpr (L == 64) {
    for (int e = tid; e < 4 * 64; e += kHmThreads) {
      const int l = e & 63, s = e >> 6, T = s < 2 ? s + 1 : 3, st = s == 3 ? 1 : 0;
      const int t0 = 32 * st + 8 * (l >> 4);
      float4 x = make_float4(0.f, 0.f, 0.f, 0.f), y = x;
      if (t0 < 16 * T) {
        const float* gp = &sh.Gs[hm_gram_col<L>(16 * T + (l & 15)) + t0];
        x = *reinterpret_cast<const float4*>(gp), y = *reinterpret_cast<const float4*>(gp + 4);
      }
      uint4* o = &sh.Gp[s * 3 * 64 + l];
      split3(x, y, o[0], o[64], o[128]);
    }
  }
  __syncthreads();
  const float e1max = __uint_as_float(sh.emax[0]), e3max = __uint_as_float(sh.emax[1]);

  // ---- main loop: 64 keys per wavefront per iteration --------------------
  const int c16 = lane & 15, g4 = lane >> 4;
  float* Xs = sh.Xs[wave];
  double* fb = sh.fb[wave];
  const int key_begin = blockIdx.x * keys_per_wg;
  const int key_end = min(N, key_begin + keys_per_wg);
  unsigned int nfrag = 0, nfall = 0;
  // B operands of a tile: lane i holds key base + 16 tau + i % 16, coordinates
  // 32 m + 8 (i / 16) .. + 7
  uint4 kv[4][4];
  auto load_keys = [&](int base) {
#pragma unroll
    for (int tau = 0; tau < 4; ++tau) {
      const int key = base + 16 * tau + c16;
      const uint16_t* row = Kb + (int64_t)min(key, key_end - 1) * sK_n + 8 * g4;
#pragma unroll
      for (int m = 0; m < 4; ++m) kv[tau][m] = *reinterpret_cast<const uint4*>(row + 32 * m);
    }
  };
  if (hm_parts<L>() && key_begin + wave * 64 < key_end) load_keys(key_begin + wave * 64);
  for (int base = key_begin + wave * 64; base < key_end; base += NWV * 64) {
    if constexpr (!hm_parts<L>()) load_keys(base);
    float ss[4];
#pragma unroll
    for (int tau = 0; tau < 4; ++tau) {
      ss[tau] = 0.f;
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const uint32_t wv[4] = {kv[tau][m].x, kv[tau][m].y, kv[tau][m].z, kv[tau][m].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float lo = bf16_to_f32(wv[e] & 0xFFFFu), hi = bf16_to_f32(wv[e] >> 16);
          ss[tau] = fmaf(lo, lo, ss[tau]);
          ss[tau] = fmaf(hi, hi, ss[tau]);
        }
      }
      ss[tau] += __shfl_xor(ss[tau], 16, 64);
      ss[tau] += __shfl_xor(ss[tau], 32, 64);
    }
    // from here on lane l owns key base + l (its norm sits in ss[l / 16])
    const float ssq = g4 == 0 ? ss[0] : g4 == 1 ? ss[1] : g4 == 2 ? ss[2] : ss[3];
    const float nk = sqrtf(ssq * (1.f + 0x1p-14f)) * (1.f + 0x1p-20f);
    // bounds that reach 1e30 (or are not numbers) certify nothing
    const float nkb = fmaf(nk, e1max, e3max) < 1e30f ? nk : __builtin_inff();
    const bool valid = base + lane < key_end;
    const uint16_t* my_row = Kb + (int64_t)(base + lane) * sK_n;
    // Zero keys (padding): up to the first row of P that is not zero the residual
    // is zero and a = +0, so that bit is u = +1 and fragile without recomputing;
    // a^ is +0 there too.  Half of 8 x 131072 keys zero: 108, 169, 465 us at
    // L = 32, 64, 128, as without zero keys (437, 900, 1845 with their tiles in
    // the reference arithmetic).  Found from the operands in registers; at L = 128
    // that costs all keys 3 %, and uncertain keys are looked at again instead.
    uint32_t zbit = 0xFFFFu;
    if (hm_parts<L>() && __ballot(ssq == 0.f)) {  // (squares below 2^-149 vanish: the keys themselves decide)
      uint32_t mine = 0u;
#pragma unroll
      for (int tau = 0; tau < 4; ++tau) {
        uint32_t any = 0u;
#pragma unroll
        for (int m = 0; m < 4; ++m) any |= (kv[tau][m].x | kv[tau][m].y) | (kv[tau][m].z | kv[tau][m].w);
        any |= (uint32_t)__shfl_xor((int)any, 16, 64);
        any |= (uint32_t)__shfl_xor((int)any, 32, 64);
        mine = g4 == tau ? any & 0x7FFF7FFFu : mine;
      }
      if (valid && mine == 0u && nkb < 3.4e38f) zbit = sh.first;
    }
    uint32_t cw[W];
#pragma unroll
    for (int w = 0; w < W; ++w) cw[w] = 0u;
    // (the zero rows, where they pass as certain: recomputed ones count themselves)
    unsigned int tfrag = valid && nkb < 3.4e38f ? sh.nzero : 0u, tfall = 0;
    if (zbit < (uint32_t)L) ++tfrag;
    bool many = false;
#pragma unroll
    for (int T = 0; T < L / 16; ++T) {
      if (many) break;
      // projections of bits 16 T .. 16 T + 15 of the 64 keys
      // (up to L = 64 two halves of the tile in turn, to halve the accumulators;
      // at L = 128 that would cut P and G twice)
      constexpr int HT = hm_parts<L>() ? 2 : 4;
#pragma unroll
      for (int hf = 0; hf < 4; hf += HT) {
        f32x4_t ah[HT], as[HT], ch[HT];
#pragma unroll
        for (int x = 0; x < HT; ++x) ah[x] = as[x] = ch[x] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          uint4 phi, pmid, plo;
          if constexpr (hm_parts<L>()) {
            const uint4* pp = &sh.Pp[(T * 4 + m) * 3 * 64 + lane];
            phi = pp[0], pmid = pp[64], plo = pp[128];
          } else {
            const float* prow = &sh.Ps[(16 * T + c16) * kHmPsStride + 32 * m + 8 * g4];
            split3(*reinterpret_cast<const float4*>(prow), *reinterpret_cast<const float4*>(prow + 4), phi, pmid, plo);
          }
#pragma unroll
          for (int x = 0; x < HT; ++x) {
            as[x] = mfma32(plo, kv[hf + x][m], as[x]);
            as[x] = mfma32(pmid, kv[hf + x][m], as[x]);
            ah[x] = mfma32(phi, kv[hf + x][m], ah[x]);
          }
        }
        if constexpr (hm_mm_corr<L>()) {
          // The corrections by earlier blocks as one more contraction: D[j][key]
          // = sum_{t < 16 T} fp32(G[t][16 T + j]) s_t(key), s_t = -1 where bit t
          // of the key is set, else +1 (exact in bf16).  Gram entries are cut
          // into hi + mid + lo like P; the hi products go to their own chain
          // ch (sums of size C_i), mid and lo to the small chain as.
#pragma unroll
          for (int st = 0; st < (T + 1) / 2; ++st) {
            const uint32_t cws = cw[st];
            // lane (g4, c16): A = G[32 st + 8 g4 .. + 7][16 T + c16], B = signs of
            // the same 8 bits of key 16 tau + c16 (none past 16 T)
            const bool on = 32 * st + 8 * g4 < 16 * T;
            uint4 ghi = make_uint4(0u, 0u, 0u, 0u), gmid = ghi, glo = ghi;
            if constexpr (L == 64) {
              const uint4* gp = &sh.Gp[(T * T / 4 + st) * 3 * 64 + lane];
              ghi = gp[0], gmid = gp[64], glo = gp[128];
            } else if (on) {
              const float* gp = &sh.Gs[hm_gram_col<L>(16 * T + c16) + 32 * st + 8 * g4];
              split3(*reinterpret_cast<const float4*>(gp), *reinterpret_cast<const float4*>(gp + 4), ghi, gmid, glo);
            }
#pragma unroll
            for (int x = 0; x < HT; ++x) {
              const uint32_t word = (uint32_t)__shfl((int)cws, 16 * (hf + x) + c16, 64);
              const uint4 sb = sign_operand((word >> (8 * g4)) & 0xFFu, on);
              ch[x] = mfma32(ghi, sb, ch[x]);
              as[x] = mfma32(gmid, sb, as[x]);
              as[x] = mfma32(glo, sb, as[x]);
            }
          }
        }
#pragma unroll
        for (int x = 0; x < HT; ++x)
          *reinterpret_cast<float4*>(&Xs[(16 * (hf + x) + c16) * kHmXsStride + 4 * g4]) =
              make_float4((ah[x][0] + as[x][0]) + ch[x][0], (ah[x][1] + as[x][1]) + ch[x][1],
                          (ah[x][2] + as[x][2]) + ch[x][2], (ah[x][3] + as[x][3]) + ch[x][3]);
      }
      // the next tile's keys are on their way while the last block is decided
      if (hm_parts<L>() && T == L / 16 - 1 && base + NWV * 64 < key_end) load_keys(base + NWV * 64);
      wave_lds_sync();
      float y[16];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float4 v = *reinterpret_cast<const float4*>(&Xs[lane * kHmXsStride + 4 * q]);
        y[4 * q] = v.x, y[4 * q + 1] = v.y, y[4 * q + 2] = v.z, y[4 * q + 3] = v.w;
      }
      // corrections by the bits of earlier blocks: y_j -= u_t Gr[t][j]
      // (on the vector units at L = 32)
#pragma unroll
      for (int w = 0; w < W; ++w) {
        if (hm_mm_corr<L>() || 32 * w >= 16 * T) break;
        const int nb = min(32, 16 * T - 32 * w);
        const uint32_t word = cw[w];
#pragma unroll 4
        for (int tt = 0; tt < nb; ++tt) {
          const float sg = ((word >> tt) & 1u) ? -1.f : 1.f;
          const int t = 32 * w + tt;
          const float4* gr = reinterpret_cast<const float4*>(&sh.Gs[hm_gram_at<L>(t, 16 * T)]);
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const float4 g = gr[q];
            y[4 * q] = fmaf(sg, g.x, y[4 * q]);
            y[4 * q + 1] = fmaf(sg, g.y, y[4 * q + 1]);
            y[4 * q + 2] = fmaf(sg, g.z, y[4 * q + 2]);
            y[4 * q + 3] = fmaf(sg, g.w, y[4 * q + 3]);
          }
        }
      }
      // The block's own bits, in order.  An uncertain decision takes the sign
      // of a^ for now and is recorded; the recorded ones are then decided in
      // the reference arithmetic, lowest bit first, and kept as overrides.
      // Where a speculated sign was wrong, the block's later bits of that key
      // rested on it, and the block is run again with the overrides.
      // (Its start is the lane's row of Xs, written back where the corrections
      // of earlier blocks were added above.)
      if (!hm_mm_corr<L>() && T > 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *reinterpret_cast<float4*>(&Xs[lane * kHmXsStride + 4 * q]) =
              make_float4(y[4 * q], y[4 * q + 1], y[4 * q + 2], y[4 * q + 3]);
      }
      // First with every sign taken from a^ (its sign bit: a certain a^ is not
      // zero, and a^ of a zero row is +0), the uncertain ones collected beside.
      uint32_t neg = 0u, unc = 0u;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int bit = 16 * T + i;
        const float2 cb = sh.cst[bit];
        const float a = y[i];
        neg = __builtin_amdgcn_alignbit(neg, __float_as_uint(a), 31);
        unc = unc + unc + (fabsf(a) > fmaf(nkb, cb.x, cb.y) ? 0u : 1u);
        if (i < 15) {
          const float s = __uint_as_float((__float_as_uint(a) & 0x80000000u) | 0x3F800000u);
          const float4* gr = reinterpret_cast<const float4*>(&sh.Gs[hm_gram_diag<L>(bit)]);
#pragma unroll
          for (int q = (i + 1) / 4; q < 4; ++q) {
            const float4 g = gr[q];
            const float gv[4] = {g.x, g.y, g.z, g.w};
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (4 * q + e > i) y[4 * q + e] = fmaf(-s, gv[e], y[4 * q + e]);
          }
        }
      }
      uint32_t ub = __brev(~neg) >> 16;
      const uint32_t zm = (zbit >> 4) == (uint32_t)T ? 1u << (zbit & 15u) : 0u;
      unc = valid ? (__brev(unc) >> 16) & ~zm : 0u;
      uint32_t ovm = 0u, ovv = 0u;
      while (true) {
        unsigned long long todo = __ballot(unc != 0u);
        if (!todo) break;
        if (!hm_parts<L>() && (int)(sh.first >> 4) == T) {
          const uint32_t zm = 1u << (sh.first & 15u);
          const bool may = (unc & zm) && nkb == 0.f;
          if (__ballot(may)) {
            uint32_t any = 0u;
            if (may)
              for (int q = 0; q < kHeadDim / 8; ++q) {
                const uint4 v = reinterpret_cast<const uint4*>(my_row)[q];
                any |= (v.x | v.y) | (v.z | v.w);
              }
            if (may && (any & 0x7FFF7FFFu) == 0u) unc &= ~zm, ovm |= zm, ovv |= zm, ++tfrag;
            todo = __ballot(unc != 0u);
            if (!todo) break;
          }
        }
        many = __popcll(todo) > kHmMany;
        if (many) break;
        bool rerun = false;
        while (todo) {
          const int j = __ffsll((long long)todo) - 1;
          todo &= todo - 1;
          uint32_t uj = __builtin_amdgcn_readlane(unc, j);
          const uint32_t ubj = __builtin_amdgcn_readlane(ub, j);
          uint32_t uw[4] = {0u, 0u, 0u, 0u};
#pragma unroll
          for (int w = 0; w < W; ++w) uw[w] = __builtin_amdgcn_readlane(cw[w], j);
          uw[(16 * T) >> 5] |= ubj << ((16 * T) & 31);
          // (the read-lane builtin returns a signed int: widen through uint32_t)
          const uint64_t rp = (uint64_t)(uintptr_t)my_row;
          const uint32_t rlo = (uint32_t)__builtin_amdgcn_readlane((uint32_t)rp, j);
          const uint32_t rhi = (uint32_t)__builtin_amdgcn_readlane((uint32_t)(rp >> 32), j);
          const uint16_t* krow = reinterpret_cast<const uint16_t*>((uintptr_t)(((uint64_t)rhi << 32) | rlo));
          while (uj) {
            const int i0 = __ffs(uj) - 1;
            uj &= uj - 1;
            const double ae = hm_reference_decision(krow, sh.Ps, 16 * T + i0, uw[0], uw[1], uw[2], uw[3], fb);
            const bool uref = ae >= 0.0;
            ++tfall;
            if (lane == j) {
              ovm |= 1u << i0;
              ovv |= (uref ? 1u : 0u) << i0;
              tfrag += fragile_decision(ae) ? 1u : 0u;
            }
            if (uref != (((ubj >> i0) & 1u) != 0u)) {
              rerun = true;  // this key's later bits of the block rested on the wrong sign
              break;
            }
          }
        }
        if (!rerun) break;
        unc = 0u, ub = 0u;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float4 v = *reinterpret_cast<const float4*>(&Xs[lane * kHmXsStride + 4 * q]);
          y[4 * q] = v.x, y[4 * q + 1] = v.y, y[4 * q + 2] = v.z, y[4 * q + 3] = v.w;
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int bit = 16 * T + i;
          const float2 cb = sh.cst[bit];
          const float a = y[i];
          const bool sure = !valid || fabsf(a) > fmaf(nkb, cb.x, cb.y);
          bool u = a >= 0.f;
          if ((ovm >> i) & 1u) u = (ovv >> i) & 1u;
          else if (!sure) unc |= (1u << i) & ~zm;
          ub |= (u ? 1u : 0u) << i;
          if (i < 15) {
            const float sg = u ? -1.f : 1.f;
            const float* gr = &sh.Gs[hm_gram_diag<L>(bit)];
#pragma unroll
            for (int e = i + 1; e < 16; ++e) y[e] = fmaf(sg, gr[e], y[e]);
          }
        }
      }
      cw[(16 * T) >> 5] |= ub << ((16 * T) & 31);
      wave_lds_sync();  // Xs is rewritten by the next block only after these reads
    }
    if (many) {
      nfrag += hm_reference_tile<L>(Kb, sK_n, base, key_end, sh.Ps, codes + b * sC_b + h * sC_h);
      nfall += (unsigned int)min(64, key_end - base) * L;
      // (the loop over the blocks may have been left before it loaded these)
      if constexpr (hm_parts<L>())
        if (base + NWV * 64 < key_end) load_keys(base + NWV * 64);
      continue;
    }
    nfrag += tfrag, nfall += tfall;
    if (valid) {
      uint32_t* cp = codes + b * sC_b + h * sC_h + (int64_t)(base + lane) * W;
      if constexpr (W == 1) cp[0] = cw[0];
      else if constexpr (W == 2) *reinterpret_cast<uint2*>(cp) = make_uint2(cw[0], cw[1]);
      else *reinterpret_cast<uint4*>(cp) = make_uint4(cw[0], cw[1], cw[2], cw[3]);
    }
  }
  // nfall is counted once per recomputed decision by every lane of the wavefront
  unsigned int wf = nfrag;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) wf += __shfl_xor(wf, o, 64);
  if (lane == 0) {
    if (wf) atomicAdd(&sh.nfrag, wf);
    if (nfall) atomicAdd(&sh.nfall, nfall);
  }
  __syncthreads();
  if (tid == 0) {
    if (fragile && sh.nfrag) atomicAdd(fragile, (unsigned long long)sh.nfrag);
    if (fallbacks && sh.nfall) atomicAdd(fallbacks, (unsigned long long)sh.nfall);
  }
}

template <int L>
static hipError_t launch_hash_mm_L(const uint16_t* K, int64_t sK_b, int64_t sK_h, int64_t sK_n, int B, int Hkv,
                                   int N, const float* P, int64_t sP_b, int64_t sP_h, uint32_t* codes, int64_t sC_b,
                                   int64_t sC_h, unsigned long long* fragile, unsigned long long* fallbacks,
                                   hipStream_t stream) {
  static_assert(sizeof(HmShared<L>) <= 160 * 1024, "LDS budget");
  constexpr int kHmThreads = hm_threads<L>();
  // about 2048 workgroups of four wavefronts, 1024 of eight, each over whole
  // wavefront iterations
  const long long total = (long long)B * Hkv * N;
  constexpr long long kWgs = 2048 * 256 / kHmThreads;
  long long per = (total + kWgs - 1) / kWgs;
  per = (per + kHmThreads - 1) / kHmThreads * kHmThreads;
  per = per < kHmThreads ? kHmThreads : per > 64 * kHmThreads ? 64 * kHmThreads : per;
  const int keys_per_wg = (int)per;
  const dim3 grid((unsigned)((N + keys_per_wg - 1) / keys_per_wg), (unsigned)(B * Hkv));
  hash_mm_kernel<L><<<grid, kHmThreads, 0, stream>>>(K, sK_b, sK_h, sK_n, Hkv, N, P, sP_b, sP_h, codes, sC_b,
                                                        sC_h, fragile, fallbacks, keys_per_wg);
  return hipGetLastError();
}

hipError_t launch_hash_mm(const uint16_t* K, int64_t sK_b, int64_t sK_h, int64_t sK_n, int B, int Hkv, int N, int L,
                          const float* P, int64_t sP_b, int64_t sP_h, uint32_t* codes, int64_t sC_b, int64_t sC_h,
                          unsigned long long* fragile, unsigned long long* fallbacks, hipStream_t stream) {
  switch (L) {
    case 32:
      return launch_hash_mm_L<32>(K, sK_b, sK_h, sK_n, B, Hkv, N, P, sP_b, sP_h, codes, sC_b, sC_h, fragile,
                                  fallbacks, stream);
    case 64:
      return launch_hash_mm_L<64>(K, sK_b, sK_h, sK_n, B, Hkv, N, P, sP_b, sP_h, codes, sC_b, sC_h, fragile,
                                  fallbacks, stream);
    default:
      return launch_hash_mm_L<128>(K, sK_b, sK_h, sK_n, B, Hkv, N, P, sP_b, sP_h, codes, sC_b, sC_h, fragile,
                                   fallbacks, stream);
  }
}

}  // namespace bpc
