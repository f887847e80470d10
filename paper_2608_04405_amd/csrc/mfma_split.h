// Device helpers shared by the kernels that project bf16 keys on the matrix
// cores with an fp32 operand cut exactly into three bf16 parts.
#pragma once

#include "bpc_internal.h"

namespace bpc {

typedef short bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// D += A B for one 16 x 16 x 32 bf16 tile (fp32 accumulation).  Lane i
// supplies A[i % 16][8 (i / 16) + j] and B[8 (i / 16) + j][i % 16] for
// j = 0..7 (two bf16 per word, low half first) and holds D[4 (i / 16) + j]
// [i % 16] for j = 0..3.  The order of the coordinates inside a lane only has
// to agree between A and B.
__device__ __forceinline__ f32x4_t mfma32(const uint4 a, const uint4 b, f32x4_t d) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b),
                                                 d, 0, 0, 0);
}

// Eight fp32 values cut exactly into three bf16 parts: hi keeps the top 8
// significant bits, mid the next 8, lo the rest (at most 8 significant bits
// remain once hi and mid are subtracted; both subtractions are exact).
__device__ __forceinline__ void split3(const float4 p0, const float4 p1, uint4& hi, uint4& mid, uint4& lo) {
  const float v[8] = {p0.x, p0.y, p0.z, p0.w, p1.x, p1.y, p1.z, p1.w};
  uint32_t h[8], m[8], l[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const uint32_t bh = __float_as_uint(v[e]) & 0xFFFF0000u;
    const float r1 = v[e] - __uint_as_float(bh);
    const uint32_t bm = __float_as_uint(r1) & 0xFFFF0000u;
    const float r2 = r1 - __uint_as_float(bm);
    h[e] = bh, m[e] = bm, l[e] = __float_as_uint(r2);
  }
  hi = make_uint4(__builtin_amdgcn_perm(h[1], h[0], 0x07060302u), __builtin_amdgcn_perm(h[3], h[2], 0x07060302u),
                  __builtin_amdgcn_perm(h[5], h[4], 0x07060302u), __builtin_amdgcn_perm(h[7], h[6], 0x07060302u));
  mid = make_uint4(__builtin_amdgcn_perm(m[1], m[0], 0x07060302u), __builtin_amdgcn_perm(m[3], m[2], 0x07060302u),
                   __builtin_amdgcn_perm(m[5], m[4], 0x07060302u), __builtin_amdgcn_perm(m[7], m[6], 0x07060302u));
  lo = make_uint4(__builtin_amdgcn_perm(l[1], l[0], 0x07060302u), __builtin_amdgcn_perm(l[3], l[2], 0x07060302u),
                  __builtin_amdgcn_perm(l[5], l[4], 0x07060302u), __builtin_amdgcn_perm(l[7], l[6], 0x07060302u));
}

__device__ __forceinline__ void wave_lds_sync() {
  // LDS operations of one wavefront complete in order; the fences keep the
  // compiler from moving LDS accesses across this point
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ double readlane_f64(double x, int lane) {
  const uint64_t b = __double_as_longlong(x);
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)b, lane);
  const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(b >> 32), lane);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// A 64 x 64 bit matrix transposed across a wavefront: lane t gives column t
// (bit j of hi:lo), lane j receives row j (bit t of hi:lo).  Six exchanges of
// halves with lane ^ 32, 16, 8, 4, 2, 1.
__device__ __forceinline__ void transpose64(uint32_t& lo, uint32_t& hi) {
  const int lane = threadIdx.x & 63;
  {
    const auto r = __builtin_amdgcn_permlane32_swap(lo, hi, false, false);
    lo = r[0], hi = r[1];
  }
  const uint32_t sel16 = (lane & 16) ? 0x07060302u : 0x05040100u;
  const uint32_t sel8 = (lane & 8) ? 0x03070105u : 0x06020400u;
  uint32_t w[2] = {lo, hi};
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    uint32_t x = w[i];
    // (even rows: own, partner; odd rows: partner, own)
    const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    x = __builtin_amdgcn_perm(r[1], r[0], sel16);
    uint32_t p = (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x128, 0xF, 0xF, false);  // row_ror:8
    x = __builtin_amdgcn_perm(p, x, sel8);
    // xor 4: half mirror, then the quads reversed
    p = (uint32_t)__builtin_amdgcn_mov_dpp(__builtin_amdgcn_mov_dpp((int)x, 0x141, 0xF, 0xF, false), 0x1B, 0xF, 0xF,
                                           false);
    p = __builtin_amdgcn_alignbit(p, p, (lane & 4) ? 4 : 28);
    uint32_t m = (lane & 4) ? 0xF0F0F0F0u : 0x0F0F0F0Fu;
    x = (x & m) | (p & ~m);
    p = (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x4E, 0xF, 0xF, false);  // quad_perm [2, 3, 0, 1]
    p = __builtin_amdgcn_alignbit(p, p, (lane & 2) ? 2 : 30);
    m = (lane & 2) ? 0xCCCCCCCCu : 0x33333333u;
    x = (x & m) | (p & ~m);
    p = (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xB1, 0xF, 0xF, false);  // quad_perm [1, 0, 3, 2]
    p = __builtin_amdgcn_alignbit(p, p, (lane & 1) ? 1 : 31);
    m = (lane & 1) ? 0xAAAAAAAAu : 0x55555555u;
    w[i] = (x & m) | (p & ~m);
  }
  lo = w[0], hi = w[1];
}

}  // namespace bpc
