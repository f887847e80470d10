// Prefill kernels: binary principal components (Algorithm "Constructing
// hash codes and corresponding hashing projection", Sec. 3.2) and hashing
// of keys against a given projection (Algorithm "Given projection,
// computing hashcode", Sec. 3.2).
//
// Both decide code bits from fp64 dot products in the fixed order of
// include/bpc.h, so the codes are reproducible bit for bit.

#pragma clang fp contract(off)

#include <type_traits>

#include "bpc_internal.h"
#include "build_tree.h"
#include "mfma_split.h"

namespace bpc {

// ============================================================================
// Algorithm 1 in its own arithmetic, for few keys (build_path), for workspaces
// too small for the scanning build (build_scan_kernels.hip, which needs some L / 8
// + 2 bytes per key more, and rows below 32 MiB apart), and for the residual norms
// after either.  Each bit is one pass over the keys of every (sequence,
// KV head) plus one reduction per (b, h):
//   build_bit_kernel    one workgroup per chunk of kBuildChunk keys, in groups
//                       of 64 (one key per lane); the four wavefronts of a
//                       group own the coordinate blocks [32 c, 32 c + 32), so
//                       every lane of a wavefront needs the same element of P
//                       and G at the same time and reads it as a scalar
//                       operand.  The fp64 residual of the lane's key is
//                       recomputed from the bf16 key, the key's code bits
//                       decided so far and the stored rows of P,
//                       R = (((k - u_0 P_0) - u_1 P_1) - ...), one rounded
//                       subtraction per bit (fma(-u, p, r) with u = +-1 is that
//                       subtraction: the product is exact), exactly as an
//                       in-place update would compute it.  Then a_j = R_j . g_i
//                       (fixed order), u_j and code bit i, and the chunk's
//                       pairwise tree of u_j R_j: a full binary tree over its
//                       rows, +0 past N, formed across lanes by a reduce-scatter
//                       butterfly (each level halves the coordinates a lane
//                       carries) and across the key groups in LDS.
//   build_fold_kernel   (more than 8 x 32 chunks per (b, h)) the subtrees over
//                       aligned blocks of 32 chunk sums, many workgroups
//   build_finish_kernel pairwise tree over the chunk sums (or those subtrees),
//                       v = s / N,
//                       P[i] = (float)v (and its fp64 widening for the next
//                       passes).
// Without a checkpoint nothing of size N x D is stored: the pass reads the keys
// again, trading fp64 arithmetic (about L^2 D / 2 fused subtractions per key over
// the whole build) for memory traffic.  With one (1 KiB per key of workspace), the
// pass at every multiple m T of kBuildCkptPeriod also stores R after m T bits, in
// place, and the passes up to (m + 1) T start from it: at most T subtractions per
// pass, for a 1 KiB read instead of the 256-byte key.
// ============================================================================

__global__ void build_prep_kernel(const float* __restrict__ G, double* __restrict__ G64, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) G64[i] = (double)G[i];
}

template <int W>
__global__ __launch_bounds__(kBuildThreads) void build_bit_kernel(
    const uint16_t* __restrict__ K, int64_t sK_b, int64_t sK_h, int64_t sK_n, int Hkv, int N, int L, int bit,
    const double* __restrict__ G64, const double* __restrict__ P64, uint32_t* __restrict__ codes, int64_t sC_b,
    int64_t sC_h, double* __restrict__ part, int nchunks, unsigned long long* __restrict__ fragile,
    double* __restrict__ ck, int ck_from, int ck_store) {
  __shared__ double xch[kBuildGroups][4][64];         // per-block partial dots of each key
  __shared__ double groot[kBuildGroups][kHeadDim];    // tree root of each key group
  __shared__ int frag;
  const int bh = blockIdx.y;
  const int b = bh / Hkv, h = bh % Hkv;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = wv & 3, grp = wv >> 2;
  if (threadIdx.x == 0) frag = 0;

  const int key = blockIdx.x * kBuildChunk + grp * 64 + lane;
  const bool valid = key < N;
  double r[32];
  uint32_t cw[W];
#pragma unroll
  for (int w = 0; w < W; ++w) cw[w] = 0u;
  uint32_t* crow = codes + b * sC_b + h * sC_h + (int64_t)(valid ? key : 0) * W;
  // this lane's 32 coordinates in the checkpoint: element e of the block at
  // ckrow[(e / 2) * 64 + lane], so that each load covers 1 KiB of the
  // wavefront's keys
  typedef double f64x2 __attribute__((ext_vector_type(2)));
  f64x2* ckrow = ck ? reinterpret_cast<f64x2*>(ck + ((((size_t)bh * nchunks + blockIdx.x) * kBuildGroups + grp) * 4 +
                                                     c) * (32 * 64)) + lane
                    : nullptr;
  if (valid) {
    if (ck_from > 0) {
#pragma unroll
      for (int e2 = 0; e2 < 16; ++e2) {
        const f64x2 x = __builtin_nontemporal_load(ckrow + 64 * e2);
        r[2 * e2] = x.x;
        r[2 * e2 + 1] = x.y;
      }
    } else {
      load_block(K + b * sK_b + h * sK_h + (int64_t)key * sK_n + 32 * c, r);
    }
#pragma unroll
    for (int w = 0; w < W; ++w)
      if (32 * w < bit) cw[w] = crow[w];
  } else {
#pragma unroll
    for (int e = 0; e < 32; ++e) r[e] = 0.0;  // never contributes: padded below
  }
  // the residual after bits 0 .. bit - 1: bits ck_from .. bit - 1 removed from
  // the checkpoint (or all of them from the key)
  remove_bits<W>(r, cw, ck_from, bit, uniform_ptr(P64 + (size_t)bh * L * kHeadDim + 32 * c));
  if (ck_store && valid) {
#pragma unroll
    for (int e2 = 0; e2 < 16; ++e2) {
      const f64x2 x = {r[2 * e2], r[2 * e2 + 1]};
      __builtin_nontemporal_store(x, ckrow + 64 * e2);
    }
  }
  // a_j = R_j . g (four blocks of 32, ascending, combined ((b0 + b1) + (b2 + b3)))
  const_ptr<double> g = uniform_ptr(G64 + (size_t)bit * kHeadDim + 32 * c);
  double acc = 0.0;
#pragma unroll
  for (int e = 0; e < 32; ++e) acc = dadd(acc, dmul(r[e], g[e]));
  xch[grp][c][lane] = acc;
  __syncthreads();
  const double a =
      dadd(dadd(xch[grp][0][lane], xch[grp][1][lane]), dadd(xch[grp][2][lane], xch[grp][3][lane]));
  const bool u = a >= 0.0;
  if (c == 0) {
    if (valid) crow[bit >> 5] = ((bit & 31) ? cw[bit >> 5] : 0u) | ((u ? 1u : 0u) << (bit & 31));
    if (fragile) {
      const unsigned long long m = __ballot(valid && fragile_decision(a));
      if (lane == 0 && m) atomicAdd(&frag, __popcll(m));
    }
  }
  const double s = group_tree(r, valid, u, lane);
  if (lane < 32) {
    groot[grp][32 * c + group_tree_index(lane)] = s;
  }
  __syncthreads();
  static_assert(kBuildGroups == 2, "one tree level across the key groups");
  if (threadIdx.x < kHeadDim)
    part[((size_t)bh * nchunks + blockIdx.x) * kHeadDim + threadIdx.x] =
        dadd(groot[0][threadIdx.x], groot[1][threadIdx.x]);
  if (fragile && threadIdx.x == 0 && frag) atomicAdd(fragile, (unsigned long long)frag);
}

// Thread d of workgroup (x, bh) folds the aligned block of chunk sums
// [x kBuildFold, (x + 1) kBuildFold) of coordinate d, level by level with the
// odd one carried (the last block may be short): the subtree of the pairwise
// tree over those chunks.
__global__ __launch_bounds__(kHeadDim) void build_fold_kernel(const double* __restrict__ part, int nchunks,
                                                              double* __restrict__ fold, int nfold) {
  const int bh = blockIdx.y, x = blockIdx.x, d = threadIdx.x;
  const int begin = x * kBuildFold;
  fold[((size_t)bh * nfold + x) * kHeadDim + d] =
      fold_sums<kBuildFold>(part + ((size_t)bh * nchunks + begin) * kHeadDim + d, min(kBuildFold, nchunks - begin));
}

// One workgroup per (b, h): thread (blk, d) folds an aligned block of S
// chunk sums of coordinate d (S a power of two, 8 blocks cover all chunks) as
// a binary counter, and the block roots are then paired level by level in LDS
// with the odd one carried.  Both are the pairwise tree with the odd element
// carried: a binary counter's final right fold equals level-wise pairing, and
// level-wise pairing of the leaves splits at every aligned power of two.
constexpr int kFinishBlocks = 8;

__global__ __launch_bounds__(kFinishBlocks* kHeadDim) void build_finish_kernel(int N, int L, int bit, int nchunks,
                                                                               const double* __restrict__ part,
                                                                               float* __restrict__ P,
                                                                               double* __restrict__ P64) {
  __shared__ double node[kFinishBlocks][kHeadDim];
  const int bh = blockIdx.x;
  const int d = threadIdx.x & (kHeadDim - 1), blk = threadIdx.x >> 7;
  int S = 1;
  while (S * kFinishBlocks < nchunks) S <<= 1;
  const int begin = blk * S, end = min(begin + S, nchunks);
  const double* src = part + (size_t)bh * nchunks * kHeadDim + d;
  double stack_v[32];
  int stack_l[32];
  int top = 0;
  for (int c0 = begin; c0 < end; c0 += 8) {
    double x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = (c0 + e < end) ? src[(size_t)(c0 + e) * kHeadDim] : 0.0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if (c0 + e >= end) break;
      double y = x[e];
      int lvl = 0;
      while (top > 0 && stack_l[top - 1] == lvl) {
        y = dadd(stack_v[top - 1], y);
        --top;
        ++lvl;
      }
      stack_v[top] = y;
      stack_l[top] = lvl;
      ++top;
    }
  }
  if (top > 0) {
    double y = stack_v[top - 1];
    for (int t = top - 2; t >= 0; --t) y = dadd(stack_v[t], y);
    node[blk][d] = y;
  }
  int cnt = (nchunks + S - 1) / S;
  while (cnt > 1) {
    __syncthreads();
    const int half = (cnt + 1) >> 1;
    double y = 0.0;
    if (blk < half) y = (2 * blk + 1 < cnt) ? dadd(node[2 * blk][d], node[2 * blk + 1][d]) : node[2 * blk][d];
    __syncthreads();
    if (blk < half) node[blk][d] = y;
    cnt = half;
  }
  if (blk == 0) {
    const double v = node[0][d] / (double)N;
    const float pf = (float)v;
    P[((size_t)bh * L + bit) * kHeadDim + d] = pf;
    P64[((size_t)bh * L + bit) * kHeadDim + d] = (double)pf;
  }
}

template <int W>
static void launch_rebuild(const BuildArgs& a, const BuildLayout& lay, bool checkpoint) {
  double* part = reinterpret_cast<double*>(a.ws + lay.off_part);
  double* fold = reinterpret_cast<double*>(a.ws + lay.off_fold);
  double* P64 = reinterpret_cast<double*>(a.ws + lay.off_p64);
  double* G64 = reinterpret_cast<double*>(a.ws + lay.off_g64);
  const int BH = a.B * a.Hkv;
  const dim3 grid(lay.nchunks, BH);
  double* ck = checkpoint ? reinterpret_cast<double*>(a.ws + lay.off_ck) : nullptr;
  const int ng = a.L * kHeadDim;
  build_prep_kernel<<<(ng + 255) / 256, 256, 0, a.stream>>>(a.G, G64, ng);
  for (int bit = 0; bit < a.L; ++bit) {
    // With a checkpoint the pass at bit m T stores R after m T bits, and the
    // passes up to the next one start from it.
    const int past = bit % kBuildCkptPeriod;
    const int from = ck ? max(bit - (past ? past : kBuildCkptPeriod), 0) : 0;
    const int store = ck && bit > 0 && past == 0;
    build_bit_kernel<W><<<grid, kBuildThreads, 0, a.stream>>>(a.K, a.sK_b, a.sK_h, a.sK_n, a.Hkv, a.N, a.L, bit, G64,
                                                             P64, a.codes, a.sC_b, a.sC_h, part, lay.nchunks,
                                                             a.fragile, ck, from, store);
    if (lay.nfold) {
      build_fold_kernel<<<dim3(lay.nfold, BH), kHeadDim, 0, a.stream>>>(part, lay.nchunks, fold, lay.nfold);
      build_finish_kernel<<<BH, kFinishBlocks * kHeadDim, 0, a.stream>>>(a.N, a.L, bit, lay.nfold, fold, a.P, P64);
    } else {
      build_finish_kernel<<<BH, kFinishBlocks * kHeadDim, 0, a.stream>>>(a.N, a.L, bit, lay.nchunks, part, a.P, P64);
    }
  }
}

// Scan (S), rebuilding passes (R) or those with a checkpoint (C), by the time of
// the whole build.  The rebuilding passes hold one 128-key chunk per compute unit
// up to 256 chunks and take little more for 256 than for one, but reduce the
// chunks of a (b, h) in one workgroup (up to 256 of them; beyond, folded first);
// the scan has two launches per bit of some 10 us, handles 256 keys of a (b, h)
// per workgroup, and over no more keys than bits leaves itself for dense_pass.
// Measured ratios:
//   S / R up to 256 chunks: L = 32, one head of 4096, 8192 and 32768 keys 1.04,
//     0.88, 0.49, 2 x 4096 and 6144 1.04, 0.92, 8 x 4096 1.05; L = 64, one of 2048
//     and 4096 1.03, 0.98, 8 x 2048 and 3072 1.00, 0.95, 32 x 1024 1.04; L = 128
//     0.85 to 1.0 beyond 128 keys, 2 to 3.2 up to 128.
//   S / R beyond: 0.25 to 0.94; but L = 32, one head of 65536, 98304, 131072 keys
//     1.24, 1.08, 1.01, and up to 128 keys per head 1.05 to 1.25 at L = 32 (0.8 to 0.9
//     at L = 64, 2 to 3.7 at 128).
//   S / C up to 256 chunks: one head of 8192 and 12288 keys 0.96, 0.76 (L = 32), 1.00,
//     0.82 (64), 1.22, 0.98 (128), 2 x 6144 0.99, 1.05, 1.27; 8 x 4096 1.07, 1.11, 1.42.
//   S / C beyond: up to 128 keys per head 1.3 to 3.7; one head of 49152, 98304, 131072
//     1.05, 1.07, 0.99 (32), 1.04, 0.99, 0.91 (64), 1.28, 1.18, 0.96 (128); L = 64, 128
//     heads, 49152 and 65536 keys in all 1.04, 0.96, 8 heads 0.81, 0.73; L = 128, 16 heads, 65536
//     and 98304 1.13, 0.87, 8 heads, 49152 and 65536 1.01, 0.91, 512 heads x 256 1.25.
BuildPath build_path(int B, int Hkv, int N, int L, bool checkpoint) {
  const int64_t BH = (int64_t)B * Hkv, keys = BH * N;
  const int64_t chunks = BH * ((N + kBuildChunk - 1) / kBuildChunk);
  const bool few = chunks <= 256;
  bool scan;
  if (!checkpoint) {
    if (N <= kBuildChunk) scan = L == 64 && !few;
    else if (few) scan = (int64_t)N * L >= 6144 * 32;
    else scan = !(L == 32 && BH == 1 && N < 196608);
    return scan ? kBuildScan : kBuildPlain;
  }
  if (few) scan = N >= (L == 32 ? 6144 : L == 64 ? 8192 : 12288);
  else if (N <= kBuildChunk) scan = false;
  else if (BH == 1) scan = N >= (L == 64 ? 98304 : 131072);
  else if (L == 32) scan = true;
  else if (L == 64) scan = BH <= 64 || keys >= 65536;
  else scan = (N >= 12288 && N <= 32768) || (N > 256 && keys >= (BH <= 8 ? 65536 : 98304));
  return scan ? kBuildScan : kBuildCheckpoint;
}

hipError_t launch_build(const BuildArgs& a, size_t ws_bytes) {
  const BuildLayout lay = build_layout(a.B, a.Hkv, a.N, a.L);
  const bool room = ws_bytes >= lay.total_ck;
  BuildPath path = build_path(a.B, a.Hkv, a.N, a.L, room);
  // (the scan's tiles of 64 rows are addressed by 32-bit offsets)
  if (path == kBuildScan && (ws_bytes < lay.total || a.sK_n >= (1 << 24)))
    path = room ? kBuildCheckpoint : kBuildPlain;
  if (path == kBuildScan) {
    launch_build_scan(a, lay);
  } else {
    switch (a.L) {
      case 32: launch_rebuild<1>(a, lay, path == kBuildCheckpoint); break;
      case 64: launch_rebuild<2>(a, lay, path == kBuildCheckpoint); break;
      default: launch_rebuild<4>(a, lay, path == kBuildCheckpoint); break;
    }
  }
  if (a.err)
    return launch_norm(a.K, a.sK_b, a.sK_h, a.sK_n, a.B, a.Hkv, a.N, a.L, a.P, (int64_t)a.Hkv * a.L * kHeadDim,
                       (int64_t)a.L * kHeadDim, a.codes, a.sC_b, a.sC_h, a.err, a.stream);
  return hipGetLastError();
}

// ============================================================================
// Residual norms ||k - h P|| of hashed keys, in the reference arithmetic: each
// coordinate's residual by one rounded subtraction per bit (a fused one, the
// product with u = +-1 being exact), the squares summed in four blocks of 32.
//
// Bound by the L x 128 fp64 subtractions per key (4 cycles each per
// wavefront).  A wavefront owns one block of 32 coordinates of 256 keys, four
// keys per lane, and takes it in two halves of 16 so that the 64 residuals fit
// registers; the rows of P are staged in LDS already widened, 32 at a time, and
// each entry read there serves four subtractions.  3.2 M keys at L = 64 (a
// batch of 4 x 8 heads x 100003): 1.05 ms, of which the subtractions and squares
// are 0.9 at the rate they issue; reading P as scalars and widening it in every
// wavefront took 1.35 ms, and the kernel that decided the signs in the same
// arithmetic 4.34.
// ============================================================================
constexpr int kNormKeys = 256;  // keys per workgroup: four per lane of each of four wavefronts

template <int W>
__global__ __launch_bounds__(256, 2) void norm_kernel(const uint16_t* __restrict__ K, int64_t sK_b, int64_t sK_h,
                                                      int64_t sK_n, int Hkv, int N, const float* __restrict__ P,
                                                      int64_t sP_b, int64_t sP_h,
                                                      const uint32_t* __restrict__ codes, int64_t sC_b, int64_t sC_h,
                                                      float* __restrict__ err) {
  __shared__ double xch[4][kNormKeys];
  __shared__ __align__(16) double ps[32][64];  // 32 rows of P, one half of every block, widened
  const int bh = blockIdx.y, b = bh / Hkv, h = bh % Hkv;
  const int lane = threadIdx.x & 63;
  const int c = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint16_t* Kb = K + b * sK_b + h * sK_h + 32 * c;
  const uint32_t* Cb = codes + b * sC_b + h * sC_h;
  const float* Pb = P + b * sP_b + h * sP_h;
  const int key0 = blockIdx.x * kNormKeys + lane;
  uint32_t cw[4][W];
#pragma unroll
  for (int x = 0; x < 4; ++x)
#pragma unroll
    for (int w = 0; w < W; ++w) cw[x][w] = Cb[(int64_t)min(key0 + 64 * x, N - 1) * W + w];
  double sq[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
  for (int half = 0; half < 2; ++half) {
    double r[4][16];
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const uint4* row = reinterpret_cast<const uint4*>(Kb + (int64_t)min(key0 + 64 * x, N - 1) * sK_n + 16 * half);
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const uint4 v = row[q];
        const uint32_t wd[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int e = 0; e < 8; ++e)
          r[x][8 * q + e] = bf16_to_f64((uint16_t)((e & 1) ? (wd[e >> 1] >> 16) : (wd[e >> 1] & 0xFFFFu)));
      }
    }
#pragma unroll
    for (int w = 0; w < W; ++w) {
      __syncthreads();
      for (int e = threadIdx.x; e < 32 * 16; e += 256) {
        const int t = e >> 4, q = e & 15;  // four floats: block q / 4, part q % 4 of its half
        const float4 v = *reinterpret_cast<const float4*>(Pb + (size_t)(32 * w + t) * kHeadDim + 32 * (q >> 2) +
                                                          16 * half + 4 * (q & 3));
        double* o = &ps[t][4 * q];
        o[0] = v.x, o[1] = v.y, o[2] = v.z, o[3] = v.w;
      }
      __syncthreads();
#pragma unroll 2
      for (int t = 0; t < 32; ++t) {
        const double* p = &ps[t][16 * c];
        double sg[4];
#pragma unroll
        for (int x = 0; x < 4; ++x)
          sg[x] = __hiloint2double((int)(0x3FF00000u | ((cw[x][w] >> t) << 31)), 0);  // -u
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const double pv = p[e];
#pragma unroll
          for (int x = 0; x < 4; ++x) r[x][e] = __builtin_fma(sg[x], pv, r[x][e]);
        }
      }
    }
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
      for (int e = 0; e < 16; ++e) sq[x] = dadd(sq[x], dmul(r[x][e], r[x][e]));
  }
#pragma unroll
  for (int x = 0; x < 4; ++x) xch[c][64 * x + lane] = sq[x];
  __syncthreads();
  const int key = blockIdx.x * kNormKeys + threadIdx.x;
  if (key < N)
    err[(size_t)bh * N + key] = (float)sqrt(dadd(dadd(xch[0][threadIdx.x], xch[1][threadIdx.x]),
                                                 dadd(xch[2][threadIdx.x], xch[3][threadIdx.x])));
}

hipError_t launch_norm(const uint16_t* K, int64_t sK_b, int64_t sK_h, int64_t sK_n, int B, int Hkv, int N, int L,
                       const float* P, int64_t sP_b, int64_t sP_h, const uint32_t* codes, int64_t sC_b, int64_t sC_h,
                       float* err, hipStream_t stream) {
  const dim3 grid((N + kNormKeys - 1) / kNormKeys, B * Hkv);
  switch (L) {
    case 32:
      norm_kernel<1><<<grid, 256, 0, stream>>>(K, sK_b, sK_h, sK_n, Hkv, N, P, sP_b, sP_h, codes, sC_b, sC_h, err);
      break;
    case 64:
      norm_kernel<2><<<grid, 256, 0, stream>>>(K, sK_b, sK_h, sK_n, Hkv, N, P, sP_b, sP_h, codes, sC_b, sC_h, err);
      break;
    default:
      norm_kernel<4><<<grid, 256, 0, stream>>>(K, sK_b, sK_h, sK_n, Hkv, N, P, sP_b, sP_h, codes, sC_b, sC_h, err);
      break;
  }
  return hipGetLastError();
}

// ============================================================================
// Algorithm 2 in the reference arithmetic, for decode-time append and for few
// keys.  Four lanes per key: lane q of a quad holds the fp64
// residual of coordinates [32q, 32q + 32) in registers, so each bit's dot
// product is four sequential block sums combined across the quad as
// ((b0 + b1) + (b2 + b3)) -- the fixed order -- and the residual update
// needs no communication.  The projection is staged in LDS once per
// workgroup (padded rows avoid bank conflicts between the four blocks).
// ============================================================================

// With a cache copy (cp.Kc non-null), decode-time append: each key row of K
// (the new keys) is also stored into the cache rows cp.Kc, and the matching
// value rows cp.Vn into cp.Vc; the four lanes of a key each move a quarter
// of both rows.
template <int L>
__global__ __launch_bounds__(256) void hash_kernel(const uint16_t* __restrict__ K, int64_t sK_b, int64_t sK_h,
                                                   int64_t sK_n, int Hkv, int N, const float* __restrict__ P,
                                                   int64_t sP_b, int64_t sP_h, uint32_t* __restrict__ codes,
                                                   int64_t sC_b, int64_t sC_h, float* __restrict__ err,
                                                   unsigned long long* __restrict__ fragile, AppendCopy cp) {
  constexpr int W = L / 32;
  constexpr int PAD = 33;
  __shared__ float p_s[L][4][PAD];
  __shared__ int frag_s;
  const int bh = blockIdx.y;
  const int b = bh / Hkv, h = bh % Hkv;
  const float* Pb = P + b * sP_b + h * sP_h;
  for (int e = threadIdx.x; e < L * kHeadDim; e += 256) {
    const int i = e / kHeadDim, d = e % kHeadDim;
    p_s[i][d >> 5][d & 31] = Pb[e];
  }
  if (threadIdx.x == 0) frag_s = 0;
  __syncthreads();

  const int key = blockIdx.x * 64 + (threadIdx.x >> 2);
  const int qd = threadIdx.x & 3;
  const bool valid = key < N;
  double r[32];
  if (valid) {
    const uint16_t* krow = K + b * sK_b + h * sK_h + (int64_t)key * sK_n + 32 * qd;
    uint4 kq[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const uint4 v = *reinterpret_cast<const uint4*>(krow + 8 * c);
      kq[c] = v;
      const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int e = 0; e < 8; ++e)
        r[8 * c + e] = bf16_to_f64((uint16_t)((e & 1) ? (w[e >> 1] >> 16) : (w[e >> 1] & 0xFFFFu)));
    }
    if (cp.Kc) {
      uint16_t* kc = cp.Kc + b * cp.sKc_b + h * cp.sKc_h + (int64_t)key * cp.sKc_n + 32 * qd;
      const uint16_t* vn = cp.Vn + b * cp.sVn_b + h * cp.sVn_h + (int64_t)key * cp.sVn_n + 32 * qd;
      uint16_t* vc = cp.Vc + b * cp.sVc_b + h * cp.sVc_h + (int64_t)key * cp.sVc_n + 32 * qd;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        reinterpret_cast<uint4*>(kc)[c] = kq[c];
        reinterpret_cast<uint4*>(vc)[c] = reinterpret_cast<const uint4*>(vn)[c];
      }
    }
  } else {
#pragma unroll
    for (int e = 0; e < 32; ++e) r[e] = 0.0;
  }
  uint32_t word = 0;
  int nfrag = 0;
  for (int i = 0; i < L; ++i) {
    double acc = 0.0;
#pragma unroll
    for (int e = 0; e < 32; ++e) acc = dadd(acc, dmul(r[e], (double)p_s[i][qd][e]));
    const double s01 = dadd(acc, __shfl_xor(acc, 1, 64));
    const double a = dadd(s01, __shfl_xor(s01, 2, 64));
    const bool u = a >= 0.0;
    if (qd == 0 && valid && fragile_decision(a)) ++nfrag;
    if ((i >> 5) == qd && u) word |= 1u << (i & 31);
#pragma unroll
    for (int e = 0; e < 32; ++e) {
      const double pv = (double)p_s[i][qd][e];
      r[e] = r[e] - (u ? pv : -pv);
    }
  }
  if (valid && qd < W) codes[b * sC_b + h * sC_h + (int64_t)key * W + qd] = word;
  if (err) {
    double sq = 0.0;
#pragma unroll
    for (int e = 0; e < 32; ++e) sq = dadd(sq, dmul(r[e], r[e]));
    const double s01 = dadd(sq, __shfl_xor(sq, 1, 64));
    const double tot = dadd(s01, __shfl_xor(s01, 2, 64));
    if (valid && qd == 0) err[(size_t)bh * N + key] = (float)sqrt(tot);
  }
  if (fragile) {
    int wsum = nfrag;
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) wsum += __shfl_xor(wsum, m, 64);
    if ((threadIdx.x & 63) == 0 && wsum) atomicAdd(&frag_s, wsum);
    __syncthreads();
    if (threadIdx.x == 0 && frag_s) atomicAdd(fragile, (unsigned long long)frag_s);
  }
}

// ---------------------------------------------------------------------------
// Decode-time append of a few tokens: one wavefront per new key, lane l holding
// coordinates 2 l and 2 l + 1 of the fp64 residual and of every row of P (all
// of its loads in flight at once).  With one key per quad of lanes, as above,
// each bit is a chain of 32 dependent fp64 multiplies and additions, 64 bits of
// it for one token.  Here the dot product is a wavefront sum in another order,
// which differs from the reference by at most 2^-44 sum_d |r_d P_id| (164
// roundings); outside that and the fragile threshold its sign is the
// reference's, else the products are summed again in the reference order.  The
// residual itself is the reference's.  16 x 8 heads, one token, L = 64: 16.6 us a
// call (39.7).
// ---------------------------------------------------------------------------
__device__ __forceinline__ double wave_sum_f64(double x) {
  auto dpp_add = [](double v, auto ctrl) {
    constexpr int C = decltype(ctrl)::value;
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), C, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), C, 0xF, 0xF, false);
    return v + __hiloint2double(hi, lo);
  };
  x = dpp_add(x, std::integral_constant<int, 0xB1>{});   // lane ^ 1
  x = dpp_add(x, std::integral_constant<int, 0x4E>{});   // lane ^ 2
  x = dpp_add(x, std::integral_constant<int, 0x141>{});  // 7 - lane within 8
  x = dpp_add(x, std::integral_constant<int, 0x140>{});  // 15 - lane within 16
  {
    const uint32_t lo = (uint32_t)__double2loint(x), hi = (uint32_t)__double2hiint(x);
    const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    x = __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
  }
  {
    const uint32_t lo = (uint32_t)__double2loint(x), hi = (uint32_t)__double2hiint(x);
    const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    x = __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
  }
  return x;
}

// ((b0 + b1) + (b2 + b3)) of the 128 values v0 (coordinate 2 l) and v1
// (2 l + 1), each block of 32 summed in ascending order from +0
__device__ __forceinline__ double ordered_sum_f64(double v0, double v1, double* fb) {
  const int l = threadIdx.x & 63;
  fb[2 * l] = v0, fb[2 * l + 1] = v1;
  wave_lds_sync();
  double s = 0.0;
  if (l < 4)
    for (int e = 0; e < 32; ++e) s = dadd(s, fb[32 * l + e]);
  const double s0 = readlane_f64(s, 0), s1 = readlane_f64(s, 1), s2 = readlane_f64(s, 2), s3 = readlane_f64(s, 3);
  wave_lds_sync();  // fb is rewritten by the next call only after these reads
  return dadd(dadd(s0, s1), dadd(s2, s3));
}

template <int L>
__global__ __launch_bounds__(64) void append_kernel(const uint16_t* __restrict__ K, int64_t sK_b, int64_t sK_h,
                                                    int64_t sK_n, int Hkv, int N, const float* __restrict__ P,
                                                    int64_t sP_b, int64_t sP_h, uint32_t* __restrict__ codes,
                                                    int64_t sC_b, int64_t sC_h, float* __restrict__ err,
                                                    unsigned long long* __restrict__ fragile, AppendCopy cp) {
  constexpr int W = L / 32;
  constexpr int C = L < 64 ? L : 64;  // rows of P held at a time
  __shared__ double fb[kHeadDim];
  const int lane = threadIdx.x, key = blockIdx.x;
  const int bh = blockIdx.y, b = bh / Hkv, h = bh % Hkv;
  const float2* Pl = reinterpret_cast<const float2*>(P + b * sP_b + h * sP_h) + lane;
  const uint32_t kk = reinterpret_cast<const uint32_t*>(K + b * sK_b + h * sK_h + (int64_t)key * sK_n)[lane];
  const uint32_t vv =
      reinterpret_cast<const uint32_t*>(cp.Vn + b * cp.sVn_b + h * cp.sVn_h + (int64_t)key * cp.sVn_n)[lane];
  double r0 = bf16_to_f64((uint16_t)(kk & 0xFFFFu)), r1 = bf16_to_f64((uint16_t)(kk >> 16));
  float top = fmaxf(fabsf(bf16_to_f32(kk & 0xFFFFu)), fabsf(bf16_to_f32(kk >> 16)));
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) top = fmaxf(top, __shfl_xor(top, o, 64));
  double rmax = (double)top;  // bounds every |r_d|, with the rows of P removed so far and in hand
  uint32_t word[W];
  int nfrag = 0;
#pragma unroll
  for (int w = 0; w < W; ++w) word[w] = 0u;
#pragma unroll 1
  for (int c = 0; c < L / C; ++c) {
    float2 p[C];
#pragma unroll
    for (int i = 0; i < C; ++i) p[i] = Pl[(C * c + i) * (kHeadDim / 2)];
    if (c == 0) {  // the copies, behind the loads of P
      reinterpret_cast<uint32_t*>(cp.Kc + b * cp.sKc_b + h * cp.sKc_h + (int64_t)key * cp.sKc_n)[lane] = kk;
      reinterpret_cast<uint32_t*>(cp.Vc + b * cp.sVc_b + h * cp.sVc_h + (int64_t)key * cp.sVc_n)[lane] = vv;
    }
    float pm = 0.f;
#pragma unroll
    for (int i = 0; i < C; ++i) pm = fmaxf(pm, fmaxf(fabsf(p[i].x), fabsf(p[i].y)));
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) pm = fmaxf(pm, __shfl_xor(pm, o, 64));
    rmax += (double)C * (double)pm;
    const double bound = 0x1p-44 * 128.0 * rmax * (double)pm + 1.01e-6;
#pragma unroll
    for (int i = 0; i < C; ++i) {
      const double p0 = (double)p[i].x, p1 = (double)p[i].y;
      double a = wave_sum_f64(__builtin_fma(r0, p0, r1 * p1));
      if (!(fabs(a) > bound)) {
        a = ordered_sum_f64(dmul(r0, p0), dmul(r1, p1), fb);
        nfrag += fragile_decision(a) ? 1 : 0;
      }
      const bool u = a >= 0.0;
      const double sg = u ? -1.0 : 1.0;
      r0 = __builtin_fma(sg, p0, r0);
      r1 = __builtin_fma(sg, p1, r1);
#pragma unroll
      for (int w = 0; w < W; ++w)
        if (w == (C * c + i) >> 5) word[w] |= (u ? 1u : 0u) << (i & 31);
    }
  }
  if (lane < W) {
    uint32_t x = word[0];
#pragma unroll
    for (int w = 1; w < W; ++w) x = lane == w ? word[w] : x;
    codes[b * sC_b + h * sC_h + (int64_t)key * W + lane] = x;
  }
  if (err) {
    const double sq = ordered_sum_f64(dmul(r0, r0), dmul(r1, r1), fb);
    if (lane == 0) err[(size_t)bh * N + key] = (float)sqrt(sq);
  }
  if (fragile && lane == 0 && nfrag) atomicAdd(fragile, (unsigned long long)nfrag);
}

// Whether each of N new keys gets a wavefront of its own: up to 16 always; up
// to 32 while the wavefronts are at most 16 per compute unit (4096 in all).
// Beyond, sixteen keys per wavefront issue less (wavefront per key against
// that; L = 64: 32 x 8 heads, T = 16 29.6 and 42.7 us, T = 32 46.4 and 42.2;
// 16 x 8 heads, T = 32 26 and 40; L = 128: 128 x 8 heads, T = 16 198 and 227,
// T = 20 243 and 228; 16 x 8 heads, T = 32 55 and 72).
static bool append_by_wave(int64_t BH, int N) { return N <= 16 || (N <= 32 && BH * N <= 4096); }

template <int L>
static hipError_t launch_hash_L(const uint16_t* K, int64_t sK_b, int64_t sK_h, int64_t sK_n, int B, int Hkv, int N,
                                const float* P, int64_t sP_b, int64_t sP_h, uint32_t* codes, int64_t sC_b,
                                int64_t sC_h, float* err, unsigned long long* fragile, hipStream_t stream,
                                const AppendCopy* append) {
  if (append && append_by_wave((int64_t)B * Hkv, N))
    append_kernel<L><<<dim3(N, B * Hkv), 64, 0, stream>>>(K, sK_b, sK_h, sK_n, Hkv, N, P, sP_b, sP_h, codes, sC_b,
                                                          sC_h, err, fragile, *append);
  else
    hash_kernel<L><<<dim3((N + 63) / 64, B * Hkv), 256, 0, stream>>>(K, sK_b, sK_h, sK_n, Hkv, N, P, sP_b, sP_h, codes,
                                                                     sC_b, sC_h, err, fragile,
                                                                     append ? *append : AppendCopy{});
  return hipGetLastError();
}

hipError_t launch_hash(const uint16_t* K, int64_t sK_b, int64_t sK_h, int64_t sK_n, int B, int Hkv, int N, int L,
                       const float* P, int64_t sP_b, int64_t sP_h, uint32_t* codes, int64_t sC_b, int64_t sC_h,
                       float* err, unsigned long long* fragile, hipStream_t stream, const AppendCopy* append) {
  switch (L) {
    case 32:
      return launch_hash_L<32>(K, sK_b, sK_h, sK_n, B, Hkv, N, P, sP_b, sP_h, codes, sC_b, sC_h, err, fragile, stream,
                               append);
    case 64:
      return launch_hash_L<64>(K, sK_b, sK_h, sK_n, B, Hkv, N, P, sP_b, sP_h, codes, sC_b, sC_h, err, fragile, stream,
                               append);
    default:
      return launch_hash_L<128>(K, sK_b, sK_h, sK_n, B, Hkv, N, P, sP_b, sP_h, codes, sC_b, sC_h, err, fragile, stream,
                                append);
  }
}

bool hash_few_keys(int64_t BH, int N, int L, bool norms) {
  const int64_t wgs = BH * ((N + 63) / 64);
  return norms ? wgs <= 512 || N <= 64 : L == 128 && N > 256 && wgs <= 256;
}

}  // namespace bpc
