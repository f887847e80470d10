// Device helpers of Algorithm 1 in its own arithmetic: a block of 32 coordinates
// of one key per lane, and the pairwise tree over keys and chunks of keys.
#pragma once

#include "bpc_internal.h"

namespace bpc {

// the partner lane's value at lane ^ M (quad permutes for 1 and 2)
template <int M>
__device__ __forceinline__ double xor_lane(double x) {
  if constexpr (M == 1 || M == 2) {
    constexpr int ctrl = (M == 1) ? 0xB1 : 0x4E;  // quad_perm [1,0,3,2] / [2,3,0,1]
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), ctrl, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), ctrl, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
  } else {
    return __shfl_xor(x, M, 64);
  }
}

// A wavefront-uniform address of data that no kernel writes while this one
// runs, in the constant address space so that loads through it are scalar.
template <typename T>
using const_ptr = const __attribute__((address_space(4))) T*;

template <typename T>
__device__ __forceinline__ const_ptr<T> uniform_ptr(const T* p) {
  const uint64_t a = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
  return (const_ptr<T>)(((uint64_t)hi << 32) | lo);
}

// one reduce-scatter level: lanes l and l ^ (1 << K) add their halves of the
// 2 * HALF coordinates they carry; the lane with bit K clear keeps the lower half
template <int K, int HALF>
__device__ __forceinline__ void rs_level(double (&v)[32], int lane) {
  const bool upper = (lane >> K) & 1;
#pragma unroll
  for (int e = 0; e < HALF; ++e) {
    const double send = upper ? v[e] : v[HALF + e];
    const double keep = upper ? v[HALF + e] : v[e];
    v[e] = dadd(keep, xor_lane<1 << K>(send));
  }
}

// 32 coordinates of one key
__device__ __forceinline__ void load_block(const uint16_t* krow, double (&r)[32]) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint4 v = *reinterpret_cast<const uint4*>(krow + 8 * q);
    const uint32_t wd[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int e = 0; e < 8; ++e)
      r[8 * q + e] = bf16_to_f64((uint16_t)((e & 1) ? (wd[e >> 1] >> 16) : (wd[e >> 1] & 0xFFFFu)));
  }
}

// bits from .. bit - 1, whose signs are in cw, removed from the residual; prow:
// this block's coordinates of P
template <int W>
__device__ __forceinline__ void remove_bits(double (&r)[32], const uint32_t* cw, int from, int bit,
                                            const_ptr<double> prow) {
#pragma unroll
  for (int w = 0; w < W; ++w) {
    const int nb = min(32, bit - 32 * w);
    const uint32_t word = cw[w];
    for (int ib = max(0, from - 32 * w); ib < nb; ++ib) {
      const double sg = ((word >> ib) & 1u) ? -1.0 : 1.0;
      const_ptr<double> p = prow + (size_t)(32 * w + ib) * kHeadDim;
#pragma unroll
      for (int e = 0; e < 32; ++e) r[e] = __builtin_fma(sg, p[e], r[e]);
    }
  }
}

// u_j R_j (exact), keys past N padded with +0, and the tree over the
// wavefront's 64 keys: after the five reduce-scatter levels lane l carries the
// coordinate whose index is l's low five bits reversed, summed over its half of
// the keys; the xor-32 step adds the two halves
__device__ __forceinline__ double group_tree(const double (&r)[32], bool valid, bool u, int lane) {
  double v[32];
#pragma unroll
  for (int e = 0; e < 32; ++e) v[e] = valid ? (u ? r[e] : -r[e]) : 0.0;
  rs_level<0, 16>(v, lane);
  rs_level<1, 8>(v, lane);
  rs_level<2, 4>(v, lane);
  rs_level<3, 2>(v, lane);
  rs_level<4, 1>(v, lane);
  return dadd(v[0], xor_lane<32>(v[0]));
}
__device__ __forceinline__ int group_tree_index(int lane) { return (int)(__brev((uint32_t)lane) >> 27); }

// The pairwise tree over c <= F sums of one coordinate, rows of kHeadDim apart,
// level by level with the odd one carried
template <int F>
__device__ __forceinline__ double fold_sums(const double* src, int c) {
  double v[F];
#pragma unroll
  for (int e = 0; e < F; ++e) v[e] = (e < c) ? src[(size_t)e * kHeadDim] : 0.0;
#pragma unroll
  for (int w = F / 2; w >= 1; w >>= 1) {
#pragma unroll
    for (int i = 0; i < w; ++i) v[i] = (2 * i + 1 < c) ? dadd(v[2 * i], v[2 * i + 1]) : v[2 * i];
    c = (c + 1) >> 1;
  }
  return v[0];
}

}  // namespace bpc
