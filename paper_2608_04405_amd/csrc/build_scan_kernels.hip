// Algorithm 1 ("Constructing hash codes and corresponding hashing
// projection", Sec. 3.2) without the residuals: the results of the
// fixed-order fp64 build, bit for bit, from one read of the bf16 keys per bit.
//
// With R_j = k_j - sum_{t<i} u_jt P_t, both things bit i needs unroll:
//
//   a_j = R_j . g_i = k_j . g_i - sum_{t<i} u_jt (P_t . g_i)
//   s   = sum_j u_ji R_j = sum_j u_ji k_j - sum_{t<i} n_it P_t,
//         n_it = sum_j u_ji u_jt = N - 2 popcount(column i ^ column t),
//
// so a pass reads each key once (256 bytes) plus its code words, and the
// L x D fused subtractions per key of a rebuilt residual (or its 1 KiB of
// fp64 checkpoint) never happen.  Neither value is the fixed-order one, so
// both are certified:
//
// Signs, in three tiers.  (1) k_j . g_i on the matrix cores (bf16 keys times
// g cut exactly into three bf16 parts, fp32 accumulation), the corrections
// from fp32 tables of the partial sums over each code byte.  The distance to
// the fixed-order value is at most |k| alpha1 + beta1 (build_solve_kernel).
// (2) A decision inside that bound (about one in a thousand) is taken again in
// fp64, with the bound |k| alpha2 + beta2; both betas hold the threshold of a
// fragile decision.  (3) What is still inside (the fragile decisions and a few
// more) is decided in the reference arithmetic itself.
//
// P: |s - (the pairwise-tree sum)| <= B per coordinate, from the energy of
// the residual, E_d = sum_j R_jd^2, which is known without the residual
// (E' = E - 2 p s + N p^2) and bounds sum_j |R_jd| by sqrt(N E_d).  When
// (float)((s - B) / N) and (float)((s + B) / N) are the same bits, that is
// P[i][d]; otherwise (about one (b, h) and bit in several hundred) the
// column's tree is summed in the reference order.  Columns whose sums are exact
// certify with B = 0.  Columns with a non-finite key, zero columns with a -0 in
// them and vanished columns whose sum may be -0 always take the exact route.
//
// A (b, h) in which that happens often (non-finite keys, few different keys,
// sums that fit the signs exactly) would have one workgroup sum column after
// column, or decide every sign three times, on every bit: at 8 x 16384 keys and
// L = 64 a NaN in one head made a build of 1.2 ms one of 767.  It leaves the
// scan for good: from the bit in question on its workgroups rebuild the
// residuals and form the tree of every column (dense_pass), as the rebuilding
// passes do and at 0.7 to 1.1 times their speed (those 767 ms become 2.8; 16
// different keys, repeated, 52 -> 3.6; 3.2 by the rebuilding passes).  That bit is repeated in the next launch, so such
// a (b, h) runs one bit behind the others and the build ends with one more pair
// of launches, in which they do nothing.

#pragma clang fp contract(off)

#include "bpc_internal.h"
#include "build_tree.h"
#include "mfma_split.h"

namespace bpc {

constexpr int kScanThreads = 256;
constexpr double kEps = 0x1p-53;

typedef uint16_t u16x2_t __attribute__((ext_vector_type(2)));

// One reduce-scatter level over the 16 lanes of a row: lane l and its partner
// (CTRL: row mirror, half mirror, or a quad permutation) add their halves of
// the 2 * HALF values they carry; the lane with bit BIT set keeps the upper half.
template <int CTRL, int BIT, int HALF>
__device__ __forceinline__ void row_reduce_level(double (&v)[32], int lane) {
  const bool upper = (lane >> BIT) & 1;
#pragma unroll
  for (int e = 0; e < HALF; ++e) {
    const double send = upper ? v[e] : v[HALF + e];
    const double keep = upper ? v[HALF + e] : v[e];
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(send), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(send), CTRL, 0xF, 0xF, false);
    v[e] = keep + __hiloint2double(hi, lo);
  }
}
// the sums over the row of 32 values per lane: afterwards v[0] and v[1] of lane
// l are those of the values row_reduce_index(l) and the next
__device__ __forceinline__ void row_reduce(double (&v)[32], int lane) {
  row_reduce_level<0x140, 3, 16>(v, lane);  // row_mirror: l and 15 - l
  row_reduce_level<0x141, 2, 8>(v, lane);   // row_half_mirror
  row_reduce_level<0x4E, 1, 4>(v, lane);    // quad_perm [2, 3, 0, 1]
  row_reduce_level<0xB1, 0, 2>(v, lane);    // quad_perm [1, 0, 3, 2]
}
__device__ __forceinline__ int row_reduce_index(int lane) { return 2 * (lane & 15); }

// A 64-key tile of a wavefront in matrix-core operand order: lane (c16, g4)
// holds, of key base + 16 tau + c16, the coordinates 32 m + 8 g4 .. + 7 in
// kv[tau][m]; keys past N are zero.  row_bytes < 2^25, so that an offset within
// the tile fits 32 bits.
__device__ __forceinline__ void load_tile(const uint16_t* Kb, uint32_t row_bytes, int base, int N, int c16, int g4,
                                          uint4 (&kv)[4][4]) {
  const char* tile = reinterpret_cast<const char*>(Kb) + (uint64_t)base * row_bytes;  // the same in every lane
#pragma unroll
  for (int tau = 0; tau < 4; ++tau) {
    const uint32_t off = (uint32_t)min(16 * tau + c16, N - 1 - base) * row_bytes + 16u * g4;
#pragma unroll
    for (int m = 0; m < 4; ++m) kv[tau][m] = *reinterpret_cast<const uint4*>(tile + (off + 64u * m));
  }
  if (base + 64 > N) {
#pragma unroll
    for (int tau = 0; tau < 4; ++tau)
#pragma unroll
      for (int m = 0; m < 4; ++m)
        if (base + 16 * tau + c16 >= N) kv[tau][m] = make_uint4(0u, 0u, 0u, 0u);
  }
}

// ---------------------------------------------------------------------------
// Per (b, h) and coordinate: sum k^2 (psum), the largest and smallest nonzero
// magnitude (pext: max in the low half, min in the high half; bit 15 of the
// low half: a sign bit was seen, in an all-zero column a negative zero); per key an upper bound of |k| as bf16.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kScanThreads, 2) void build_stat_kernel(const uint16_t* __restrict__ K, int64_t sK_b,
                                                                     int64_t sK_h, int64_t sK_n, int Hkv, int N,
                                                                     int blocks_per_wg, double* __restrict__ psum,
                                                                     uint32_t* __restrict__ pext,
                                                                     uint16_t* __restrict__ knorm, int nblk) {
  __shared__ double red[4][kHeadDim];
  __shared__ uint32_t ext[kHeadDim][3];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c16 = lane & 15, g4 = lane >> 4;
  const int bh = blockIdx.y, b = bh / Hkv, h = bh % Hkv;
  const uint16_t* Kb = K + b * sK_b + h * sK_h;
  const uint32_t row_bytes = (uint32_t)sK_n * 2u;
  for (int e = tid; e < kHeadDim; e += kScanThreads) ext[e][0] = 0u, ext[e][1] = 0x7FFFu, ext[e][2] = 0u;
  __syncthreads();
  // two coordinates per word: the largest magnitude, the smallest magnitude
  // minus one (so that zeros count as the largest), the bits seen
  double acc[32];
  u16x2_t mx[16], mn[16];
  uint32_t seen[16];
#pragma unroll
  for (int e = 0; e < 32; ++e) acc[e] = 0.0;
#pragma unroll
  for (int e = 0; e < 16; ++e) mx[e] = (u16x2_t){0, 0}, mn[e] = (u16x2_t){0xFFFF, 0xFFFF}, seen[e] = 0u;
  const int blk_end = min((int)(blockIdx.x + 1) * blocks_per_wg, nblk);
  for (int blk = blockIdx.x * blocks_per_wg + wave; blk < blk_end; blk += 4) {
    uint4 kv[4][4];
    load_tile(Kb, row_bytes, __builtin_amdgcn_readfirstlane(blk * 64), N, c16, g4, kv);
    float ss[4];
#pragma unroll
    for (int tau = 0; tau < 4; ++tau) {
      ss[tau] = 0.f;
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const uint32_t wd[4] = {kv[tau][m].x, kv[tau][m].y, kv[tau][m].z, kv[tau][m].w};
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const float f0 = __uint_as_float(wd[w] << 16), f1 = __uint_as_float(wd[w] & 0xFFFF0000u);
          acc[8 * m + 2 * w] = __builtin_fma((double)f0, (double)f0, acc[8 * m + 2 * w]);
          acc[8 * m + 2 * w + 1] = __builtin_fma((double)f1, (double)f1, acc[8 * m + 2 * w + 1]);
          ss[tau] = fmaf(f1, f1, fmaf(f0, f0, ss[tau]));
          const u16x2_t mag = __builtin_bit_cast(u16x2_t, wd[w] & 0x7FFF7FFFu);
          mx[4 * m + w] = __builtin_elementwise_max(mx[4 * m + w], mag);
          mn[4 * m + w] = __builtin_elementwise_min(mn[4 * m + w], (u16x2_t)(mag - (u16x2_t){1, 1}));
          seen[4 * m + w] |= wd[w];
        }
      }
      ss[tau] += __shfl_xor(ss[tau], 16, 64);
      ss[tau] += __shfl_xor(ss[tau], 32, 64);
    }
    // lane l: the key base + l; rounded up (the sum's own roundings, squares
    // below 2^-126, the cut to bf16)
    const float s = g4 == 0 ? ss[0] : g4 == 1 ? ss[1] : g4 == 2 ? ss[2] : ss[3];
    const float nk = sqrtf(s * (1.f + 0x1p-14f)) * (1.f + 0x1p-20f) + 0x1p-55f;
    const uint32_t nb = __float_as_uint(nk);
    // (infinity and NaN keep their class: the cut below adds no carry into them)
    const uint32_t up = nk < 3e38f ? (nb + 0xFFFFu) >> 16 : (nk == nk ? 0x7F80u : 0x7FC0u);
    if (blk * 64 + lane < N) knorm[(size_t)bh * N + blk * 64 + lane] = (uint16_t)up;
  }
#pragma unroll
  for (int e = 0; e < 32; ++e) {
    const int d = 32 * (e >> 3) + 8 * g4 + (e & 7);
    atomicMax(&ext[d][0], (uint32_t)mx[e >> 1][e & 1]);
    atomicMin(&ext[d][1], min((uint32_t)(uint16_t)mn[e >> 1][e & 1] + 1u, 0x7FFFu));
    if ((seen[e >> 1] >> (16 * (e & 1))) & 0x8000u) atomicOr(&ext[d][2], 1u);
  }
  row_reduce(acc, lane);
  const int e0 = row_reduce_index(lane);
#pragma unroll
  for (int x = 0; x < 2; ++x) red[wave][32 * (e0 >> 3) + 8 * g4 + (e0 & 7) + x] = acc[x];
  __syncthreads();
  if (tid < kHeadDim) {
    const size_t at = ((size_t)bh * gridDim.x + blockIdx.x) * kHeadDim + tid;
    psum[at] = (red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid]);
    pext[at] = (ext[tid][0] | (ext[tid][2] << 15)) | (ext[tid][1] << 16);
  }
}

// ---------------------------------------------------------------------------
// Decision `bit` of one key in the reference arithmetic, by the whole
// wavefront: lane l rebuilds coordinates l and l + 64 with one rounded
// subtraction per earlier bit, the products are rounded, each block of 32
// coordinates is summed in ascending order from +0 and the blocks combined as
// ((b0 + b1) + (b2 + b3)).
// ---------------------------------------------------------------------------
template <int W>
__device__ __forceinline__ double reference_decision(const uint16_t* krow, const float* Pb, const float* g, int bit,
                                                     const uint32_t (&cw)[W], double* fb) {
  const int l = threadIdx.x & 63;
  double r0 = bf16_to_f64(krow[l]), r1 = bf16_to_f64(krow[l + 64]);
#pragma unroll
  for (int w = 0; w < W; ++w) {
    for (int t = 32 * w; t < min(bit, 32 * w + 32); ++t) {
      const double p0 = (double)Pb[t * kHeadDim + l], p1 = (double)Pb[t * kHeadDim + l + 64];
      const double sg = ((cw[w] >> (t & 31)) & 1u) ? -1.0 : 1.0;
      r0 = __builtin_fma(sg, p0, r0);
      r1 = __builtin_fma(sg, p1, r1);
    }
  }
  fb[l] = dmul(r0, (double)g[l]);
  fb[64 + l] = dmul(r1, (double)g[l + 64]);
  wave_lds_sync();
  double s = 0.0;
  if (l < 4)
    for (int e = 0; e < 32; ++e) s = dadd(s, fb[32 * l + e]);
  const double s0 = readlane_f64(s, 0), s1 = readlane_f64(s, 1), s2 = readlane_f64(s, 2), s3 = readlane_f64(s, 3);
  wave_lds_sync();  // fb is rewritten by the next call only after these reads
  return dadd(dadd(s0, s1), dadd(s2, s3));
}

// The same decisions for all 64 keys of a tile at once, one key per lane (each
// lane reads its own row; g, P and the corrections are the same in every lane):
// first in fp64 without the residual, then, where `todo` asks for it, in the
// reference arithmetic.
template <int W>
__device__ __forceinline__ double lane_decision(const uint16_t* row, const double* cb, const float* g, int bit,
                                                const uint32_t* cw) {
  double a = 0.0;
#pragma unroll 1
  for (int q = 0; q < kHeadDim / 8; ++q) {
    const uint4 v = reinterpret_cast<const uint4*>(row)[q];
    const uint32_t wd[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int e = 0; e < 8; ++e)
      a = __builtin_fma(bf16_to_f64((uint16_t)((e & 1) ? (wd[e >> 1] >> 16) : (wd[e >> 1] & 0xFFFFu))),
                        (double)g[8 * q + e], a);
  }
#pragma unroll
  for (int w = 0; w < W; ++w)
    for (int t = 32 * w; t < min(bit, 32 * w + 32); ++t) a += ((cw[w] >> (t & 31)) & 1u) ? -cb[t] : cb[t];
  return a;
}
template <int W>
__device__ __forceinline__ double lane_reference_decision(const uint16_t* row, const float* Pb, const float* g, int bit,
                                                          const uint32_t* cw) {
  double blk[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    double s = 0.0;
#pragma unroll 1
    for (int q = 0; q < 4; ++q) {
      const int d0 = 32 * c + 8 * q;
      const uint4 v = *reinterpret_cast<const uint4*>(row + d0);
      const uint32_t wd[4] = {v.x, v.y, v.z, v.w};
      double r[8];
#pragma unroll
      for (int e = 0; e < 8; ++e)
        r[e] = bf16_to_f64((uint16_t)((e & 1) ? (wd[e >> 1] >> 16) : (wd[e >> 1] & 0xFFFFu)));
#pragma unroll
      for (int w = 0; w < W; ++w)
        for (int t = 32 * w; t < min(bit, 32 * w + 32); ++t) {
          const double sg = ((cw[w] >> (t & 31)) & 1u) ? -1.0 : 1.0;
#pragma unroll
          for (int e = 0; e < 8; ++e) r[e] = __builtin_fma(sg, (double)Pb[t * kHeadDim + d0 + e], r[e]);
        }
#pragma unroll
      for (int e = 0; e < 8; ++e) s = dadd(s, dmul(r[e], (double)g[d0 + e]));
    }
    blk[c] = s;
  }
  return dadd(dadd(blk[0], blk[1]), dadd(blk[2], blk[3]));
}
// uncertain keys of a tile above which all its keys are decided at once
constexpr int kScanMany = 16;

// ---------------------------------------------------------------------------
// What a (b, h) does (x of `mode`), the columns redone so far (y) and the tiles
// of 64 keys whose signs went to the reference arithmetic (z).  The sign pass
// reads the state from its bounds, which it needs anyway: alpha1 = -state.
// ---------------------------------------------------------------------------
constexpr int kScanning = 0, kDenseFirst = 1, kDense = 2;  // kDenseFirst: the bit's fragile decisions are counted already
// Columns over the whole build beyond which the scan is left.  Of random keys a
// (b, h) redoes less than one in a build; each holds up the pass by up to 7 ms (a
// million keys).
constexpr int kDenseColumns = 8;
__device__ __forceinline__ bool leave_scan(int columns, int tiles, int nblk) {
  return columns > kDenseColumns || tiles > 2 * nblk;  // two whole bits of uncertain signs
}

__device__ __forceinline__ void load_row(double (&p)[16], const_ptr<double> src) {
#pragma unroll
  for (int e = 0; e < 16; ++e) p[e] = src[e];
}
// Uses the values, so that scalar loads issued after this point are not waited
// for with them (these return in no order and are waited for all together).
__device__ __forceinline__ void wait_row(double (&p)[16]) {
#pragma unroll
  for (int e = 0; e < 16; e += 8)
    asm volatile("" ::"s"(p[e]), "s"(p[e + 1]), "s"(p[e + 2]), "s"(p[e + 3]), "s"(p[e + 4]), "s"(p[e + 5]),
                 "s"(p[e + 6]), "s"(p[e + 7]));
}

// One bit of a (b, h) that has left the scan, for chunks [begin, end): signs,
// bit planes and the tree sum of every column over each chunk, all in the
// reference arithmetic.  Wavefront c owns coordinates [32 c, 32 c + 32); a lane
// takes two keys at a time, one of each half of the chunk, so that every scalar
// load of P serves both, and half a row of P is loaded ahead.  Bound by the fp64
// subtractions and the tree; 8 x 131072 keys, L = 64, all heads: 20 ms a build
// (25 with one key per lane, 27 with two and no load ahead; the rebuilding passes,
// which keep more wavefronts in flight, 15).
template <int W>
__device__ __forceinline__ void dense_pass(const uint16_t* Kb, int64_t sK_n, int N, int bit, int begin, int end,
                                           const float* g, const double* P64b, uint64_t* planes, double* part,
                                           double (*xch)[4][64], double (*groot)[kHeadDim],
                                           unsigned long long* fragile) {
  constexpr int NP = W == 4 ? 2 : 1;
  static_assert(kBuildGroups == 2, "two keys per lane, one tree level across them");
  const int lane = threadIdx.x & 63;
  const int c = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const const_ptr<double> prow = uniform_ptr(P64b + 32 * c);
  const const_ptr<float> gp = uniform_ptr(g + 32 * c);
  int nfrag = 0;
  for (int chunk = begin; chunk < end; ++chunk) {
    double r[2][32];
    uint32_t cw[2][2 * NP];
    uint64_t* pl = planes + (size_t)chunk * 2 * (32 * W);
    const int key0 = chunk * kBuildChunk + lane;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const bool live = chunk * kBuildChunk + 64 * q < N;
#pragma unroll
      for (int x = 0; x < NP; ++x) {
        const uint64_t col = live && lane + 64 * x < bit ? pl[32 * W * q + lane + 64 * x] : 0ull;
        cw[q][2 * x] = (uint32_t)col, cw[q][2 * x + 1] = (uint32_t)(col >> 32);
        if (bit > 64 * x) transpose64(cw[q][2 * x], cw[q][2 * x + 1]);
      }
      if (key0 + 64 * q < N) {
        load_block(Kb + (int64_t)(key0 + 64 * q) * sK_n + 32 * c, r[q]);
      } else {
#pragma unroll
        for (int e = 0; e < 32; ++e) r[q][e] = 0.0;
      }
    }
    // half a row of P in use, the other half on its way
    double pa[16], pb[16];
    const_ptr<double> next = prow;
    load_row(pa, next);
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const int nb = min(32, bit - 32 * w);
      for (int ib = 0; ib < nb; ++ib) {
        const double s0 = ((cw[0][w] >> ib) & 1u) ? -1.0 : 1.0, s1 = ((cw[1][w] >> ib) & 1u) ? -1.0 : 1.0;
        wait_row(pa);
        load_row(pb, next + 16);
        if (32 * w + ib + 1 < bit) next += kHeadDim;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          r[0][e] = __builtin_fma(s0, pa[e], r[0][e]);
          r[1][e] = __builtin_fma(s1, pa[e], r[1][e]);
        }
        wait_row(pb);
        load_row(pa, next);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          r[0][16 + e] = __builtin_fma(s0, pb[e], r[0][16 + e]);
          r[1][16 + e] = __builtin_fma(s1, pb[e], r[1][16 + e]);
        }
      }
    }
    double acc0 = 0.0, acc1 = 0.0;
#pragma unroll
    for (int e = 0; e < 32; ++e) {
      acc0 = dadd(acc0, dmul(r[0][e], (double)gp[e]));
      acc1 = dadd(acc1, dmul(r[1][e], (double)gp[e]));
    }
    xch[0][c][lane] = acc0, xch[1][c][lane] = acc1;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const double a = dadd(dadd(xch[q][0][lane], xch[q][1][lane]), dadd(xch[q][2][lane], xch[q][3][lane]));
      const bool u = a >= 0.0, valid = key0 + 64 * q < N;
      if (c == 0) {
        const unsigned long long M = __ballot(valid && u);
        nfrag += __popcll(__ballot(valid && fragile_decision(a)));
        if (lane == 0 && chunk * kBuildChunk + 64 * q < N) pl[32 * W * q + bit] = M;
      }
      const double s = group_tree(r[q], valid, u, lane);
      if (lane < 32) groot[q][32 * c + group_tree_index(lane)] = s;
    }
    __syncthreads();
    if (threadIdx.x < kHeadDim)
      part[(size_t)chunk * kHeadDim + threadIdx.x] = dadd(groot[0][threadIdx.x], groot[1][threadIdx.x]);
  }
  if (fragile && threadIdx.x == 0 && nfrag) atomicAdd(fragile, (unsigned long long)nfrag);
}

// The sum of every column from its chunks' tree sums, by the whole workgroup:
// blocks of kDenseFold folded from one array into the other.  Thread d < 128 returns
// column d's.
template <int NTH>
__device__ __forceinline__ double dense_sum(double* part, double* fold, int nchunks) {
  const int d = threadIdx.x & (kHeadDim - 1);
  double* src = part;
  double* dst = fold;
  for (int cnt = nchunks; cnt > 1;) {
    const int nb = (cnt + kDenseFold - 1) / kDenseFold;
    for (int x = threadIdx.x / kHeadDim; x < nb; x += NTH / kHeadDim)
      dst[(size_t)x * kHeadDim + d] =
          fold_sums<kDenseFold>(src + (size_t)x * kDenseFold * kHeadDim + d, min(kDenseFold, cnt - x * kDenseFold));
    __syncthreads();
    double* t = src;
    src = dst, dst = t, cnt = nb;
  }
  return src[d];
}

// ---------------------------------------------------------------------------
// One bit: sign and bit plane of every key, and per workgroup
// sum_j u_j k_j (fp64) and the popcounts against the earlier bit planes.
// Bound by the read of the keys; per 64 keys a wavefront issues about 460
// vector instructions, 384 of them the fp64 sum (widen, convert, fused add).
// (The launch after the last bit is for the (b, h) that have left the scan.)
// ---------------------------------------------------------------------------
template <int W>
__global__ __launch_bounds__(kScanThreads, 2) void build_sign_kernel(
    const uint16_t* __restrict__ K, int64_t sK_b, int64_t sK_h, int64_t sK_n, int Hkv, int N, int bit,
    int blocks_per_wg, int nblk, const float* __restrict__ G, const float* __restrict__ P,
    const uint16_t* __restrict__ knorm, const float* __restrict__ tab, const double* __restrict__ corr, const float4* __restrict__ bound,
    uint64_t* __restrict__ planes, double* __restrict__ psum, uint32_t* __restrict__ pcnt,
    const double* __restrict__ P64, double* __restrict__ part, int4* __restrict__ mode,
    unsigned long long* __restrict__ fragile) {
  constexpr int L = 32 * W;
  constexpr int NP = W == 4 ? 2 : 1;  // bit planes per lane
  __shared__ __align__(16) float tab_s[4 * W][256];
  __shared__ double red[4][kHeadDim];
  __shared__ uint32_t cnt_s[4][L];
  __shared__ uint4 ga_s[4][64];
  __shared__ int frag;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c16 = lane & 15, g4 = lane >> 4;
  const int bh = blockIdx.y, b = bh / Hkv, h = bh % Hkv;
  const uint16_t* Kb = K + b * sK_b + h * sK_h;
  const uint32_t row_bytes = (uint32_t)sK_n * 2u;
  const float* Pb = P + (size_t)bh * L * kHeadDim;
  const float* g = G + (size_t)min(bit, L - 1) * kHeadDim;
  const double* cb = corr + (size_t)bh * L;
  const int nbytes = (bit + 7) >> 3;  // code bytes that hold earlier bits
  const int blk_begin = blockIdx.x * blocks_per_wg + wave;
  const int blk_end = min((int)(blockIdx.x + 1) * blocks_per_wg, nblk);
  if (tid == 0) frag = 0;
  {
    const float4* src = reinterpret_cast<const float4*>(tab + (size_t)bh * (4 * W) * 256);
    for (int e = tid; e < nbytes * 64; e += kScanThreads) reinterpret_cast<float4*>(&tab_s[0][0])[e] = src[e];
  }
  // A operand: row c16 holds part c16 % 4 of g (hi, mid, lo, nothing), so that
  // every lane group g4 finds its key's three products in its own D rows
  {
    const int m = wave;
    const float4* gp = reinterpret_cast<const float4*>(g + 32 * m + 8 * g4);
    uint4 hi, mid, lo;
    split3(gp[0], gp[1], hi, mid, lo);
    const int part = c16 & 3;
    ga_s[m][lane] = part == 0 ? hi : part == 1 ? mid : part == 2 ? lo : make_uint4(0u, 0u, 0u, 0u);
  }
  const float4 bd = bound[bh];  // alpha1, beta1, alpha2, beta2
  __syncthreads();
  if (bd.x < 0.f) {
    const int chunk0 = (int)blockIdx.x * blocks_per_wg / kBuildGroups;
    dense_pass<W>(Kb, sK_n, N, bit - 1, chunk0,
                  min(chunk0 + blocks_per_wg / kBuildGroups, (nblk + kBuildGroups - 1) / kBuildGroups),
                  G + (size_t)(bit - 1) * kHeadDim, P64 + (size_t)bh * L * kHeadDim, planes + (size_t)bh * nblk * L,
                  part + (size_t)bh * ((nblk + kBuildGroups - 1) / kBuildGroups) * kHeadDim,
                  reinterpret_cast<double(*)[4][64]>(&tab_s[0][0]), red,
                  bd.x == -(float)kDense ? fragile : nullptr);
    return;
  }
  if (bit >= L) return;

  double acc[32];
#pragma unroll
  for (int e = 0; e < 32; ++e) acc[e] = 0.0;
  uint32_t cnt[NP];
#pragma unroll
  for (int x = 0; x < NP; ++x) cnt[x] = 0u;
  int nfrag = 0;
  double* fb = red[wave];
  for (int blk = blk_begin; blk < blk_end; blk += 4) {
    const int base = blk * 64;
    const bool valid = base + lane < N;
    const float nk = bf16_to_f32(knorm[(size_t)bh * N + min(base + lane, N - 1)]);
    // lane t: column t (and t + 64) of the 64 keys' code bits; transposed, lane
    // j: the code words of key j so far
    uint64_t* pl = planes + ((size_t)bh * nblk + blk) * L;
    uint64_t col[NP];
    uint32_t cw[2 * NP];
#pragma unroll
    for (int x = 0; x < NP; ++x) {
      col[x] = lane + 64 * x < bit ? pl[lane + 64 * x] : 0ull;
    }
    uint4 kv[4][4];
    load_tile(Kb, row_bytes, base, N, c16, g4, kv);
#pragma unroll
    for (int x = 0; x < NP; ++x) {
      cw[2 * x] = (uint32_t)col[x], cw[2 * x + 1] = (uint32_t)(col[x] >> 32);
      if (bit > 64 * x) transpose64(cw[2 * x], cw[2 * x + 1]);
    }

    float y = 0.f;
    {
      f32x4_t d[4];
#pragma unroll
      for (int tau = 0; tau < 4; ++tau) d[tau] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const uint4 ga = ga_s[m][lane];
#pragma unroll
        for (int tau = 0; tau < 4; ++tau) d[tau] = mfma32(ga, kv[tau][m], d[tau]);
      }
#pragma unroll
      for (int tau = 0; tau < 4; ++tau) {
        const float s = d[tau][0] + (d[tau][1] + d[tau][2]);
        y = g4 == tau ? s : y;
      }
    }
    // lane l from here on: key base + l
#pragma unroll
    for (int w = 0; w < W; ++w)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (4 * w + q < nbytes) y -= tab_s[4 * w + q][(cw[w] >> (8 * q)) & 0xFFu];
    const float t1 = fmaf(nk, bd.x, bd.y);
    const bool sure = !valid || (fabsf(y) > t1 && t1 < 1e30f);
    bool u = y >= 0.f;
    unsigned long long todo = __ballot(!sure);
    if (__popcll(todo) > kScanMany) {
      const uint16_t* row = Kb + (int64_t)min(base + lane, N - 1) * sK_n;
      const double a = lane_decision<W>(row, cb, g, bit, cw);
      const double t2 = __builtin_fma((double)nk, (double)bd.z, (double)bd.w);
      const bool sure2 = sure || (fabs(a) > t2 && t2 < 1e290);
      if (!sure) u = a >= 0.0;
      todo = __ballot(!sure2);
      if (__popcll(todo) > kScanMany) {
        const double ar = lane_reference_decision<W>(row, Pb, g, bit, cw);
        if (lane == 0) atomicAdd(&mode[bh].z, 1);
        if (!sure2) {
          u = ar >= 0.0;
          nfrag += fragile_decision(ar) ? 1 : 0;
        }
        todo = 0ull;
      }
    }
    while (todo) {
      const int j = __ffsll((long long)todo) - 1;
      todo &= todo - 1;
      const uint16_t* krow = Kb + (int64_t)(base + j) * sK_n;
      uint32_t cj[W];
#pragma unroll
      for (int w = 0; w < W; ++w) cj[w] = __builtin_amdgcn_readlane(cw[w], j);
      const double nj = (double)__uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(nk), j));
      const uint32_t kk = reinterpret_cast<const uint32_t*>(krow)[lane];
      const float2 gg = reinterpret_cast<const float2*>(g)[lane];
      double a = __builtin_fma(bf16_to_f64((uint16_t)(kk >> 16)), (double)gg.y,
                               bf16_to_f64((uint16_t)(kk & 0xFFFFu)) * (double)gg.x);
#pragma unroll
      for (int x = 0; x < NP; ++x) {
        const int t = lane + 64 * x;
        uint32_t wd = cj[0];
#pragma unroll
        for (int w = 1; w < W; ++w) wd = (t >> 5) == w ? cj[w] : wd;
        if (t < bit) a += ((wd >> (t & 31)) & 1u) ? -cb[t] : cb[t];
      }
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) a += __shfl_xor(a, o, 64);
      const double t2 = __builtin_fma(nj, (double)bd.z, (double)bd.w);
      if (!(fabs(a) > t2 && t2 < 1e290)) {
        a = reference_decision<W>(krow, Pb, g, bit, cj, fb);
        if (lane == j) nfrag += fragile_decision(a) ? 1 : 0;
      }
      if (lane == j) u = a >= 0.0;
    }
    const unsigned long long M = __ballot(valid && u);
    if (lane == 0) pl[bit] = M;
#pragma unroll
    for (int x = 0; x < NP; ++x)
      if (lane + 64 * x <= bit) cnt[x] += __popcll(col[x] ^ M);  // lane `bit`: the keys with u = +1
#pragma unroll
    for (int tau = 0; tau < 4; ++tau) {
      const uint32_t half = (uint32_t)(M >> (32 * (tau >> 1)));
      const uint32_t on = (half >> (16 * (tau & 1) + c16)) & 1u;
      const double sg = __hiloint2double((int)(0xBFF00000u ^ (on << 31)), 0);
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const uint32_t wd[4] = {kv[tau][m].x, kv[tau][m].y, kv[tau][m].z, kv[tau][m].w};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float f = __uint_as_float((e & 1) ? (wd[e >> 1] & 0xFFFF0000u) : (wd[e >> 1] << 16));
          acc[8 * m + e] = __builtin_fma(sg, (double)f, acc[8 * m + e]);
        }
      }
    }
  }
  row_reduce(acc, lane);
  const int e0 = row_reduce_index(lane);
#pragma unroll
  for (int x = 0; x < 2; ++x) red[wave][32 * (e0 >> 3) + 8 * g4 + (e0 & 7) + x] = acc[x];
#pragma unroll
  for (int x = 0; x < NP; ++x)
    if (lane + 64 * x < L) cnt_s[wave][lane + 64 * x] = cnt[x];
  if (fragile && nfrag) atomicAdd(&frag, nfrag);
  __syncthreads();
  const size_t wg = (size_t)bh * gridDim.x + blockIdx.x;
  if (tid < kHeadDim) psum[wg * kHeadDim + tid] = (red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid]);
  if (tid <= bit) pcnt[wg * L + tid] = (cnt_s[0][tid] + cnt_s[1][tid]) + (cnt_s[2][tid] + cnt_s[3][tid]);
  if (fragile && tid == 0 && frag) atomicAdd(fragile, (unsigned long long)frag);
}

// ---------------------------------------------------------------------------
// a + b = s + e exactly
__device__ __forceinline__ void two_sum(double a, double b, double& s, double& e) {
  s = a + b;
  const double bb = s - a;
  e = (a - (s - bb)) + (b - bb);
}

// The pairwise tree (adjacent pairs; +0 past N inside a chunk of 128 rows, the
// odd chunk carried above) of u_j R_jd for one coordinate, in the reference
// arithmetic, by the whole workgroup.  planes: the (b, h)'s bit planes, bits
// 0 .. bit of 64 keys at a stride of L words; pcol: P[t][d] for t < bit; node: global
// scratch of two doubles per chunk.
//
// A wavefront takes eight blocks of 64 keys at a time, one key of each per lane
// (eight independent chains), whose signs it gets by transposing the bit planes
// as the sign pass does.  Bound by vector issue (four instructions per key and
// bit) on one compute unit.  A column of a million keys at L = 128: 4 to 7 ms (8
// to 15 with a chunk per lane, each reading its bytes of every plane); the whole
// build of 8 x 1048576 keys 105 -> 82 ms.  A function of its own, so that the solves
// that do not need it (all but a few) keep their code short: 8 x 8192 keys, L = 64,
// 1062 -> 1036 us.
template <int W, int NTH>
__device__ __noinline__ double reference_column(const uint16_t* Kd, int64_t sK_n, const uint64_t* planes, int N, int bit,
                                   const double* pcol, double* node) {
  constexpr int NP = W == 4 ? 2 : 1;
  constexpr int Q = 8;  // blocks per turn
  const int lane = threadIdx.x & 63;
  const int nblk = (N + 63) / 64, nch = (N + kBuildChunk - 1) / kBuildChunk;
  for (int b0 = Q * (threadIdx.x >> 6); b0 < nblk; b0 += Q * (NTH / 64)) {
    double v[Q];
    uint32_t cw[Q][2 * NP];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int blk = min(b0 + q, nblk - 1);
      v[q] = bf16_to_f64(Kd[(int64_t)min(blk * 64 + lane, N - 1) * sK_n]);
#pragma unroll
      for (int x = 0; x < NP; ++x) {
        const uint64_t col = lane + 64 * x <= bit ? planes[(size_t)blk * (32 * W) + lane + 64 * x] : 0ull;
        cw[q][2 * x] = (uint32_t)col, cw[q][2 * x + 1] = (uint32_t)(col >> 32);
      }
    }
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
      for (int x = 0; x < NP; ++x) transpose64(cw[q][2 * x], cw[q][2 * x + 1]);
    bool u[Q];
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const int nb = min(32, bit - 32 * w);
#pragma unroll 2
      for (int t = 0; t < nb; ++t) {
        const double p = pcol[32 * w + t];
#pragma unroll
        for (int q = 0; q < Q; ++q)
          v[q] = __builtin_fma(__hiloint2double((int)(0x3FF00000u | ((cw[q][w] >> t) << 31)), 0), p, v[q]);
      }
      if (w == bit >> 5) {
#pragma unroll
        for (int q = 0; q < Q; ++q) u[q] = (cw[q][w] >> (bit & 31)) & 1u;
      }
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      v[q] = (b0 + q) * 64 + lane >= N ? 0.0 : u[q] ? v[q] : -v[q];
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) v[q] = v[q] + __shfl_xor(v[q], o, 64);
    }
#pragma unroll
    for (int q = 0; q < Q; q += 2)
      if (lane == 0 && (b0 + q) / 2 < nch) node[(b0 + q) / 2] = v[q] + v[q + 1];
  }
  double* src = node;
  double* dst = node + nch;
  int cnt = nch;
  while (cnt > 1) {
    __syncthreads();
    const int half = (cnt + 1) >> 1;
    for (int i = threadIdx.x; i < half; i += NTH) dst[i] = 2 * i + 1 < cnt ? src[2 * i] + src[2 * i + 1] : src[2 * i];
    double* x = src;
    src = dst, dst = x, cnt = half;
  }
  __syncthreads();
  const double r = src[0];
  __syncthreads();
  return r;
}

constexpr int kSolveThreads = 512;
constexpr int kSolveSlices = kSolveThreads / kHeadDim;  // threads per coordinate

// One workgroup per (b, h): P[bit] from the pass's sums, certified or summed
// again in the reference order, then what the next pass needs: the
// corrections c_t = P_t . g (fp64, and fp32 tables per code byte) and the
// bounds.  With bit < 0 the first call of a build: the key statistics.
//
// |s - reference| <= 2^-53 1.02 (sum_x sqrt(N E_x) [the roundings of the
// residual's subtraction x = 1 .. bit] + levels sqrt(N E) [of the tree] + chain
// sqrt(N E_0) [of this side's sum of keys]) + 2^-51 |s|; the energies carry
// 2^-36 E_0 of slack for their own roundings.  Most of these sums are exact and
// then count nothing: the keys and the P[t][d] removed from them are multiples
// of a common power of two q (of their smallest ulp), every residual is below
// M = max |k| + sum_t |P_td|, and an addition whose result is a multiple of q
// below 2^53 q does not round.  So the residual is exact while M < 2^53 q, the
// tree up to the level l with 2^l M < 2^53 q, and the sum of keys when
// N max |k| < 2^53 q.
template <int W>
__global__ __launch_bounds__(kSolveThreads) void build_solve_kernel(
    const uint16_t* __restrict__ K, int64_t sK_b, int64_t sK_h, int64_t sK_n, int Hkv, int N, int bit, int nwg,
    int chain, const float* __restrict__ G, const uint64_t* __restrict__ planes,
    const double* __restrict__ psum, const uint32_t* __restrict__ pcnt, const uint32_t* __restrict__ pext,
    double* __restrict__ node, float* __restrict__ P, double* __restrict__ P64, double* __restrict__ stat,
    double* __restrict__ cmat, double* __restrict__ corr, float* __restrict__ tab, float4* __restrict__ bound,
    double* __restrict__ part, double* __restrict__ fold, int4* __restrict__ mode) {
  constexpr int L = 32 * W;
  constexpr int NS = kSolveSlices;
  constexpr int NX = (8 * L + kSolveThreads - 1) / kSolveThreads;  // rounds of eight lanes per later bit
  __shared__ double sh[NS][kHeadDim], sl[NS][kHeadDim];
  __shared__ double p_s[kHeadDim], a_s[kHeadDim], col_s[L], c_s[L];
  __shared__ int n_s[L];
  __shared__ int redo[kHeadDim], nredo;
  const int tid = threadIdx.x, d = tid & (kHeadDim - 1), sl8 = tid >> 7;
  const int bh = blockIdx.x, b = bh / Hkv, h = bh % Hkv;
  // per coordinate: energies of the keys and of the residual, its sum of
  // roundings, the chain coefficient, sum_t |P_td|, max |k| and the quantum q
  double* E0 = stat + (size_t)bh * kScanStats * kHeadDim;
  double* E = E0 + kHeadDim;
  double* Rs = E + kHeadDim;
  double* ch = Rs + kHeadDim;
  double* Aa = ch + kHeadDim;
  double* Kx = Aa + kHeadDim;
  double* Qu = Kx + kHeadDim;
  const double dN = (double)N;
  // Every load this call will need is issued here: what follows is a chain of
  // short steps between barriers, bound by their latency.
  const int next = bit + 1;
  const int eighth = tid & 7;
  const int4 md = mode[bh];
  double pv[L / NS];
#pragma unroll
  for (int x = 0; x < L / NS; ++x)
    pv[x] = sl8 + NS * x < bit ? P64[((size_t)bh * L + sl8 + NS * x) * kHeadDim + d] : 0.0;
  double v_e0 = 0.0, v_e = 0.0, v_rs = 0.0, v_ch = 0.0, v_aa = 0.0, v_kx = 0.0, v_qu = 0.0;
  if (bit >= 0 && tid < kHeadDim)
    v_e0 = E0[d], v_e = E[d], v_rs = Rs[d], v_ch = ch[d], v_aa = Aa[d], v_kx = Kx[d], v_qu = Qu[d];
  float4 gs[NX][4];
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    const int sx = min((tid >> 3) + r * (kSolveThreads / 8), L - 1);
#pragma unroll
    for (int x = 0; x < 4; ++x) gs[r][x] = reinterpret_cast<const float4*>(G + (size_t)sx * kHeadDim + 16 * eighth)[x];
  }
  const double c_old = tid < bit && next < L ? cmat[((size_t)bh * L + next) * L + tid] : 0.0;
  float g0 = 0.f, g1 = 0.f;
  if (tid < 64 && next < L) g0 = G[(size_t)next * kHeadDim + tid], g1 = G[(size_t)next * kHeadDim + 64 + tid];
  // the pass's sums of keys (thread (sl8, d)) and its popcounts against the
  // earlier bit planes (thread (sl8, t)), eight workgroups' worth per round
  double s = 0.0;
  int cn = 0;
  for (int w0 = sl8; w0 < nwg; w0 += 8 * NS) {
    double x[8];
    int c[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const size_t w = (size_t)bh * nwg + min(w0 + NS * e, nwg - 1);
      x[e] = psum[w * kHeadDim + d];
      c[e] = (int)pcnt[w * L + min(d, L - 1)];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (w0 + NS * e >= nwg) x[e] = 0.0, c[e] = 0;
    s += ((x[0] + x[1]) + (x[2] + x[3])) + ((x[4] + x[5]) + (x[6] + x[7]));
    cn += ((c[0] + c[1]) + (c[2] + c[3])) + ((c[4] + c[5]) + (c[6] + c[7]));
  }
  const int nch = (N + kBuildChunk - 1) / kBuildChunk;
  if (bit >= 0 && md.x != kScanning) {
    const double T = dense_sum<kSolveThreads>(part + (size_t)bh * nch * kHeadDim,
                                              fold + (size_t)bh * ((nch + kDenseFold - 1) / kDenseFold) * kHeadDim, nch);
    if (tid < kHeadDim) {
      const size_t at = ((size_t)bh * L + bit - 1) * kHeadDim + d;
      const float p = (float)(T / dN);
      P[at] = p;
      P64[at] = (double)p;
    }
    if (tid == 0) bound[bh].x = -(float)kDense;
    return;
  }
  if (bit >= L) return;
  if (tid < L) n_s[tid] = 0;
  if (tid == 0) nredo = 0;
  __syncthreads();
  if (d <= bit) atomicAdd(&n_s[d], cn);

  if (bit < 0) {
    if (tid == 0) mode[bh] = make_int4(kScanning, 0, 0, 0);
    uint32_t mx = 0u, mn = 0x7FFFu, nz = 0u;
    for (int w = sl8; w < nwg; w += NS) {
      const uint32_t x = pext[((size_t)bh * nwg + w) * kHeadDim + d];
      mx = max(mx, x & 0x7FFFu), mn = min(mn, x >> 16), nz |= x & 0x8000u;
    }
    sh[sl8][d] = s;
    sl[sl8][d] = __longlong_as_double((long long)(((uint64_t)(nz | mx) << 32) | mn));
    __syncthreads();
    if (tid < kHeadDim) {
      double e = 0.0;
      mx = 0u, mn = 0x7FFFu, nz = 0u;
#pragma unroll
      for (int x = 0; x < NS; ++x) {
        e += sh[x][d];
        const uint64_t w = (uint64_t)__double_as_longlong(sl[x][d]);
        mx = max(mx, (uint32_t)(w >> 32) & 0x7FFFu), mn = min(mn, (uint32_t)w), nz |= (uint32_t)(w >> 32) & 0x8000u;
      }
      // the keys' common quantum: 2^-7 of the smallest magnitude's power of
      // two (2^-133 for denormals); every sum of them is a multiple of it
      const double quantum = ldexp(1.0, max((int)(mn >> 7), 1) - 127 - 7);
      const bool exact = dN * bf16_to_f64((uint16_t)mx) < 0x1p53 * quantum;
      e *= 1.0 + 0x1p-34;
      E0[d] = e;
      E[d] = e;
      Rs[d] = 0.0;
      // an all-zero column with a negative zero in it: its sums' zero signs
      // follow the reference order only (NaN never certifies)
      ch[d] = (mx == 0u && nz) ? __builtin_nan("") : exact ? 0.0 : (double)chain;
      Aa[d] = 0.0;
      Kx[d] = bf16_to_f64((uint16_t)mx);
      Qu[d] = quantum;
      a_s[d] = 0.0;
    }
    __syncthreads();
  } else {
    __syncthreads();
    // sum_t n_t P_td, each product and sum with its rounding error kept
    double hi = 0.0, lo = 0.0;
#pragma unroll
    for (int x = 0; x < L / NS; ++x) {
      if (sl8 + NS * x >= bit) break;
      const double n = dN - 2.0 * (double)n_s[sl8 + NS * x];
      const double p = pv[x];
      const double q = n * p, qe = __builtin_fma(n, p, -q);
      double e;
      two_sum(hi, q, hi, e);
      lo += e + qe;
    }
    double e;
    two_sum(s, -hi, sh[sl8][d], e);
    sl[sl8][d] = e - lo;
    __syncthreads();
    double S = 0.0, lo2 = 0.0;
    if (tid < kHeadDim) {
#pragma unroll
      for (int x = 0; x < NS; ++x) {
        two_sum(S, sh[x][d], S, e);
        lo2 += e + sl[x][d];
      }
      two_sum(S, lo2, S, e);
      const double NE = sqrt(dN * (v_e + 0x1p-36 * v_e0));
      // levels of the tree (one spare) above those whose sums are exact
      const double M = (v_kx + v_aa) * (1.0 + 0x1p-20), top = 0x1p53 * v_qu;
      int levels = 34 - __clz(N);
      for (double x = M; levels > 0 && 2.0 * x < top; x *= 2.0) --levels;
      // Where nothing rounds at all both sides hold the same number, which over
      // short columns often lies halfway between two floats.
      const bool exact = levels == 0 && v_rs == 0.0 && v_ch == 0.0 && e == 0.0;
      const double B =
          exact ? 0.0 : kEps * 1.02 * (v_rs + levels * NE + v_ch * sqrt(dN * v_e0)) + 0x1p-51 * fabs(S);
      const float pl = (float)((S - B) / dN), ph = (float)((S + B) / dN);
      p_s[d] = (double)pl;
      // The residuals of an all-zero column are all +0, and those of another
      // column may have become so exactly: their sum is +0 unless every term is
      // -0, that is no key has u = +1 and the last chunk no padding.
      const bool all_negative = n_s[bit] == 0 && N % kBuildChunk == 0;
      if (!(__float_as_uint(pl) == __float_as_uint(ph) && fabsf(pl) < 3e38f) ||
          (all_negative && pl == 0.f && v_e0 != 0.0))
        redo[atomicAdd(&nredo, 1)] = d;
      else if (all_negative && v_e0 == 0.0) p_s[d] = -0.0;
    }
    __syncthreads();
    const int nr = nredo;
    const int nblk = (N + 63) / 64;
    if (leave_scan(md.y + nr, md.z, nblk)) {  // this bit again, by dense_pass
      if (tid == 0) mode[bh].x = kDense, bound[bh].x = -(float)kDenseFirst;
      return;
    }
    if (nr && tid == 0) mode[bh].y = md.y + nr;
    for (int r = 0; r < nr; ++r) {
      const int dd = redo[r];
      if (tid < bit) col_s[tid] = P64[((size_t)bh * L + tid) * kHeadDim + dd];
      __syncthreads();
      const double T = reference_column<W, kSolveThreads>(K + b * sK_b + h * sK_h + dd, sK_n,
                                                         planes + (size_t)bh * nblk * L, N, bit, col_s,
                                                         node + (size_t)bh * 2 * nch);
      if (tid == 0) p_s[dd] = (double)(float)(T / dN);
    }
    __syncthreads();
    if (tid < kHeadDim) {
      const double p = p_s[d];
      P[((size_t)bh * L + bit) * kHeadDim + d] = (float)p;
      P64[((size_t)bh * L + bit) * kHeadDim + d] = p;
      double En = v_e - 2.0 * p * S + dN * p * p;
      En = En < 0.0 ? 0.0 : En;
      E[d] = En;
      const double A = v_aa + fabs(p);
      Aa[d] = A;
      // p is a multiple of its fp32 ulp
      const uint32_t pe = (__float_as_uint((float)p) >> 23) & 0xFFu;
      const double q = p == 0.0 ? v_qu : fmin(v_qu, ldexp(1.0, max((int)pe, 1) - 127 - 23));
      Qu[d] = q;
      if (!((v_kx + A) * (1.0 + 0x1p-20) < 0x1p53 * q)) Rs[d] = v_rs + sqrt(dN * (En + 0x1p-36 * v_e0));
      a_s[d] = A;
    }
    __syncthreads();
    // c[s][bit] = P[bit] . g_s for the bits s to come: eight lanes per s
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      const int sx = (tid >> 3) + r * (kSolveThreads / 8);
      if (sx <= bit || sx >= L) continue;
      double c = 0.0;
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const double* pp = p_s + 16 * eighth + 4 * x;
        c = __builtin_fma(pp[0], (double)gs[r][x].x, c);
        c = __builtin_fma(pp[1], (double)gs[r][x].y, c);
        c = __builtin_fma(pp[2], (double)gs[r][x].z, c);
        c = __builtin_fma(pp[3], (double)gs[r][x].w, c);
      }
      c += __shfl_xor(c, 1, 64);
      c += __shfl_xor(c, 2, 64);
      c += __shfl_xor(c, 4, 64);
      if (eighth == 0) {
        cmat[((size_t)bh * L + sx) * L + bit] = c;
        if (sx == next) c_s[bit] = c;
      }
    }
  }
  if (next >= L) return;
  if (tid < L && tid != bit) c_s[tid] = c_old;
  __syncthreads();
  if (tid < next) corr[(size_t)bh * L + tid] = c_s[tid];
  const int nbytes = (next + 7) >> 3;
  for (int e = tid; e < nbytes * 256; e += kSolveThreads) {
    const int q = e >> 8;
    double v = 0.0;
#pragma unroll
    for (int x = 0; x < 8; ++x) v += ((e >> x) & 1) ? c_s[8 * q + x] : -c_s[8 * q + x];
    tab[(size_t)bh * (4 * W) * 256 + e] = (float)v;
  }
  // |g|, sum_t |c_t| and Q = sum_d (sum_t |P_td|) |g_d| of the next bit
  if (tid < 64) {
    double n2 = (double)g0 * g0 + (double)g1 * g1, c = 0.0;
    double q = a_s[tid] * fabs((double)g0) + a_s[tid + 64] * fabs((double)g1);
    for (int t = tid; t < next; t += 64) c += fabs(c_s[t]);
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) n2 += __shfl_xor(n2, o, 64), q += __shfl_xor(q, o, 64), c += __shfl_xor(c, o, 64);
    if (tid == 0) {
      // Tier 2: the reference's (36 + i) and this side's (at most 130 + 130 +
      // 140) roundings of sums below |k| |g| + Q, and the fragile threshold.
      // Tier 1: the matrix-core chains (138 u |k| |g|), up to 19 fp32 additions
      // of table entries (u (|k| |g| + C) each), u = 2^-24; underflow of bf16
      // parts, products and keys.
      const double gl = sqrt(n2) * (1.0 + 0x1p-20) + 0x1p-500;
      const double a2 = 0x1p-43 * gl, b2 = 0x1p-43 * q + 1.01e-6;
      const double a1 = 160.0 * 0x1p-24 * gl + 0x1p-100 + a2;
      const double b1 = 24.0 * 0x1p-24 * c + b2 + 0x1p-109 * (1.0 + gl);
      const double up = 1.0 + 0x1p-8;
      bound[bh] = make_float4((float)(a1 * up), (float)(b1 * up), (float)(a2 * up), (float)(b2 * up));
    }
  }
}

// The code words of every key from the bit planes: one wavefront per 64 keys.
template <int W>
__global__ __launch_bounds__(kScanThreads) void build_codes_kernel(const uint64_t* __restrict__ planes, int Hkv, int N,
                                                                   int nblk, uint32_t* __restrict__ codes,
                                                                   int64_t sC_b, int64_t sC_h) {
  constexpr int L = 32 * W;
  constexpr int NP = W == 4 ? 2 : 1;
  const int lane = threadIdx.x & 63, blk = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int bh = blockIdx.y, b = bh / Hkv, h = bh % Hkv;
  if (blk >= nblk) return;
  const uint64_t* pl = planes + ((size_t)bh * nblk + blk) * L;
  uint32_t cw[2 * NP];
#pragma unroll
  for (int x = 0; x < NP; ++x) {
    const uint64_t col = lane + 64 * x < L ? pl[lane + 64 * x] : 0ull;
    cw[2 * x] = (uint32_t)col, cw[2 * x + 1] = (uint32_t)(col >> 32);
    transpose64(cw[2 * x], cw[2 * x + 1]);
  }
  const int key = blk * 64 + lane;
  if (key >= N) return;
  uint32_t* cp = codes + b * sC_b + h * sC_h + (int64_t)key * W;
  if constexpr (W == 1) cp[0] = cw[0];
  else if constexpr (W == 2) *reinterpret_cast<uint2*>(cp) = make_uint2(cw[0], cw[1]);
  else *reinterpret_cast<uint4*>(cp) = make_uint4(cw[0], cw[1], cw[2], cw[3]);
}

template <int W>
static void launch_build_scan_W(const BuildArgs& a, const BuildLayout& lay) {
  constexpr int L = 32 * W;
  const int BH = a.B * a.Hkv;
  char* ws = a.ws;
  double* psum = reinterpret_cast<double*>(ws + lay.off_psum);
  uint32_t* pcnt = reinterpret_cast<uint32_t*>(ws + lay.off_pcnt);
  uint64_t* planes = reinterpret_cast<uint64_t*>(ws + lay.off_planes);
  uint16_t* knorm = reinterpret_cast<uint16_t*>(ws + lay.off_knorm);
  double* node = reinterpret_cast<double*>(ws + lay.off_node);
  double* P64 = reinterpret_cast<double*>(ws + lay.off_p64);
  double* stat = reinterpret_cast<double*>(ws + lay.off_stat);
  double* cmat = reinterpret_cast<double*>(ws + lay.off_cmat);
  double* corr = reinterpret_cast<double*>(ws + lay.off_corr);
  float* tab = reinterpret_cast<float*>(ws + lay.off_tab);
  float4* bound = reinterpret_cast<float4*>(ws + lay.off_bound);
  double* part = reinterpret_cast<double*>(ws + lay.off_part);
  double* fold = reinterpret_cast<double*>(ws + lay.off_sfold);
  int4* mode = reinterpret_cast<int4*>(ws + lay.off_mode);
  const dim3 grid(lay.scan_wgs, BH);
  const int bpw = lay.scan_blocks, nblk = (a.N + 63) / 64;
  // additions one key passes through on this side: a lane's own chain, the
  // row, wavefront and workgroup levels
  const int chain = bpw + lay.scan_wgs / 4 + 32;
  build_stat_kernel<<<grid, kScanThreads, 0, a.stream>>>(a.K, a.sK_b, a.sK_h, a.sK_n, a.Hkv, a.N, bpw, psum, pcnt,
                                                         knorm, nblk);
  for (int bit = -1; bit <= L; ++bit) {
    if (bit >= 0)
      build_sign_kernel<W><<<grid, kScanThreads, 0, a.stream>>>(a.K, a.sK_b, a.sK_h, a.sK_n, a.Hkv, a.N, bit, bpw, nblk,
                                                                a.G, a.P, knorm, tab, corr, bound, planes, psum, pcnt,
                                                                P64, part, mode, a.fragile);
    build_solve_kernel<W><<<BH, kSolveThreads, 0, a.stream>>>(a.K, a.sK_b, a.sK_h, a.sK_n, a.Hkv, a.N, bit,
                                                              lay.scan_wgs, chain, a.G, planes, psum, pcnt, pcnt, node,
                                                              a.P, P64, stat, cmat, corr, tab, bound, part, fold, mode);
  }
  build_codes_kernel<W><<<dim3((nblk + 3) / 4, BH), kScanThreads, 0, a.stream>>>(planes, a.Hkv, a.N, nblk, a.codes,
                                                                                 a.sC_b, a.sC_h);
}

void launch_build_scan(const BuildArgs& a, const BuildLayout& lay) {
  switch (a.L) {
    case 32: launch_build_scan_W<1>(a, lay); break;
    case 64: launch_build_scan_W<2>(a, lay); break;
    default: launch_build_scan_W<4>(a, lay); break;
  }
}

}  // namespace bpc
