// Error-Aware Safeguard, prefill side (Sec. 3.2 "Error-Aware Safeguard
// (EAS)", Eq. reconstruction_error): the hard-to-hash set S_err of each
// (sequence, KV head) is the m keys with the largest reconstruction errors
// ||k - h P||, which the prefill kernels already produce (err_out).
//
// One 1024-thread workgroup per (b, h) finds the m-th largest error by a
// three-pass radix select over the 32-bit order key of each float (11, 11
// and 10 bits, most significant first; each pass histograms, in LDS, the keys
// that match the digits fixed so far), then writes, in ascending index
// order, every key above the threshold and the lowest-index keys equal to it
// until m are taken.  The order key maps the IEEE total order of float32 onto
// unsigned integers (negative values complemented, others with the sign bit
// set), so larger errors have larger keys.

#include "bpc_internal.h"

namespace bpc {

constexpr int kHardThreads = 1024;
constexpr int kHardBins = 2048;       // 11-bit digits
constexpr int kHardChunk = 4 * kHardThreads;  // keys per compaction pass

__device__ __forceinline__ uint32_t order_key(uint32_t u) { return (u & 0x80000000u) ? ~u : (u | 0x80000000u); }

__global__ __launch_bounds__(kHardThreads) void select_hard_kernel(const float* __restrict__ err, int64_t sE_b,
                                                                   int64_t sE_h, int Hkv, int N, int m,
                                                                   int32_t* __restrict__ out) {
  __shared__ uint32_t hist[kHardBins];
  __shared__ int wave_tot[kHardThreads / 64];
  __shared__ int found[2];  // digit, keys above it
  const int bh = blockIdx.x;
  const int b = bh / Hkv, h = bh % Hkv;
  const uint32_t* e = reinterpret_cast<const uint32_t*>(err + b * sE_b + h * sE_h);
  const int t = threadIdx.x;

  // ---- the threshold key: `need` = rank of the m-th largest key among the
  // keys that share the digits fixed so far (1 = the largest of them)
  uint32_t prefix = 0u, pmask = 0u;
  int need = m;
  constexpr int kShift[3] = {21, 10, 0}, kBits[3] = {11, 11, 10};
#pragma unroll
  for (int pass = 0; pass < 3; ++pass) {
    const int shift = kShift[pass];
    const uint32_t dmask = (1u << kBits[pass]) - 1u;
    hist[2 * t] = 0u, hist[2 * t + 1] = 0u;
    __syncthreads();
    for (int i = t; i < N; i += kHardThreads) {
      const uint32_t k = order_key(e[i]);
      if ((k & pmask) == prefix) atomicAdd(&hist[(k >> shift) & dmask], 1u);
    }
    __syncthreads();
    // thread t holds bins 2047 - 2t (upper) and 2046 - 2t; the exclusive scan
    // in that order counts the keys in the bins above
    const int hi = (int)hist[kHardBins - 1 - 2 * t], lo = (int)hist[kHardBins - 2 - 2 * t];
    int total;
    const int above_hi = block_exclusive_scan<kHardThreads>(hi + lo, wave_tot, total);
    const int above_lo = above_hi + hi;
    if (above_hi < need && need <= above_hi + hi) found[0] = kHardBins - 1 - 2 * t, found[1] = above_hi;
    if (above_lo < need && need <= above_lo + lo) found[0] = kHardBins - 2 - 2 * t, found[1] = above_lo;
    __syncthreads();
    prefix |= (uint32_t)found[0] << shift;
    pmask |= dmask << shift;
    need -= found[1];
    __syncthreads();  // found[] and hist[] are rewritten by the next pass
  }
  // prefix is the threshold key; `need` keys equal to it are taken, lowest
  // indices first, after the m - need keys above it

  // ---- ordered compaction, kHardChunk keys at a time (four per thread)
  int written = 0, ties_seen = 0;
  for (int c0 = 0; c0 < N; c0 += kHardChunk) {
    uint32_t k[4];
    int nb = 0, nt = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = c0 + 4 * t + u;
      k[u] = (i < N) ? order_key(e[i]) : 0u;
      const bool valid = i < N;
      nb += valid && k[u] > prefix;
      nt += valid && k[u] == prefix;
    }
    int tot;
    const int pre = block_exclusive_scan<kHardThreads>((nt << 16) | nb, wave_tot, tot);
    int tie_rank = ties_seen + (pre >> 16);
    int rank = written + (pre & 0xFFFF) + max(0, min(tie_rank, need) - min(ties_seen, need));
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = c0 + 4 * t + u;
      if (i >= N) break;
      bool keep = k[u] > prefix;
      if (k[u] == prefix) {
        keep = tie_rank < need;
        ++tie_rank;
      }
      if (keep) out[(size_t)bh * m + rank] = i;
      rank += keep;
    }
    written += (tot & 0xFFFF) + max(0, min(ties_seen + (tot >> 16), need) - min(ties_seen, need));
    ties_seen += tot >> 16;
  }
}

// ---------------------------------------------------------------------------
// The same selection by segments of up to kTileKeys keys, one workgroup each
// with its keys in registers: every segment keeps its own m largest (lowest
// index first among equals), which hold every key of the result; the survivors,
// still in index order, are selected from again until one segment is left.
//
// With one workgroup per (b, h) the selection read every key four times with
// at most B Hkv compute units at work, and its first histogram (sign, exponent
// and two bits) put most keys into a handful of bins, whose LDS atomics run one
// after another.  Here the errors are read once, and the digits are taken from
// the key minus the segment's smallest, over the bits that the segment's range
// really has.  16 x 8 heads x 131072 keys, m = 263: 56 us
// (227 with one workgroup per (b, h)); 8 heads x 1048576, m = 2098: 73 us.  Above
// kTileMost a segment would keep too much of itself, and the one-workgroup
// kernel stays.
// ---------------------------------------------------------------------------
constexpr int kTileRounds = 16;
constexpr int kTileKeys = kTileRounds * kHardThreads;
constexpr int kTileMost = kTileKeys / 4;  // largest m: every level then keeps at most a quarter
// Up to here the one-workgroup kernel's loops are shorter than the segment
// kernel's 16 rounds (one against the other, 8 heads: 100 errors 6.1 and 12.1 us,
// 1000 6.7 and 12.4, 4096 9.3 and 12.7, 6000 11.8 and 12.9, 8192 14.8 and 13.3;
// 1024 heads x 4096 25 and 32, x 8192 40 and 34).
constexpr int kTileLeast = 6144;

struct TileSource {
  const uint32_t* key;    // floats' bits, or order keys where idx is given
  int64_t s_b, s_h;
  const int32_t* idx;     // the keys' indices (same strides), or nullptr: their positions
  int n;
};

// Workgroup (x, y): segment y of (b, h) = x (the y dimension is the one that is limited).
__global__ __launch_bounds__(kHardThreads, 8) void select_tile_kernel(TileSource src, int Hkv, int seg, int m,
                                                                      uint32_t* __restrict__ okey,
                                                                      int32_t* __restrict__ oidx, int64_t o_bh,
                                                                      int keep) {
  constexpr int NW = kHardThreads / 64;
  __shared__ uint32_t hist[kHardBins];
  __shared__ int wave_tot[NW];
  __shared__ int found[2];
  __shared__ uint32_t range[2];
  __shared__ int cnt_a[kTileRounds * NW], cnt_e[kTileRounds * NW];
  const int bh = blockIdx.x, sidx = blockIdx.y, b = bh / Hkv, h = bh % Hkv;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int begin = sidx * seg, cnt = min(seg, src.n - begin);
  const int rounds = (cnt - t + kHardThreads - 1) / kHardThreads;  // this thread's keys: j < rounds
  const uint32_t* e = src.key + b * src.s_b + h * src.s_h + begin;
  uint32_t k[kTileRounds];
#pragma unroll
  for (int j = 0; j < kTileRounds; ++j) {
    const int i = j * kHardThreads + t;
    k[j] = j < rounds ? e[i] : 0u;
  }
  if (t == 0) range[0] = 0xFFFFFFFFu, range[1] = 0u;
  __syncthreads();
  uint32_t lo = 0xFFFFFFFFu, hi = 0u;
#pragma unroll
  for (int j = 0; j < kTileRounds; ++j) {
    if (!src.idx) k[j] = order_key(k[j]);
    if (j < rounds) lo = min(lo, k[j]), hi = max(hi, k[j]);
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    lo = min(lo, (uint32_t)__shfl_xor((int)lo, o, 64));
    hi = max(hi, (uint32_t)__shfl_xor((int)hi, o, 64));
  }
  if (lane == 0) atomicMin(&range[0], lo), atomicMax(&range[1], hi);
  __syncthreads();
  lo = range[0];
  int bits = range[1] == lo ? 0 : 32 - __clz((int)(range[1] - lo));  // keys lie in [lo, lo + 2^bits)
  int need = min(m, cnt);
  while (bits > 0) {
    const int shift = max(0, bits - 11);
    hist[2 * t] = 0u, hist[2 * t + 1] = 0u;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kTileRounds; ++j) {
      const uint32_t x = k[j] - lo;
      if (j < rounds && k[j] >= lo && (bits == 32 || (x >> bits) == 0u))
        atomicAdd(&hist[x >> shift], 1u);
    }
    __syncthreads();
    // thread t holds bins 2047 - 2t (upper) and 2046 - 2t, as above
    const int up = (int)hist[kHardBins - 1 - 2 * t], dn = (int)hist[kHardBins - 2 - 2 * t];
    int total;
    const int above_up = block_exclusive_scan<kHardThreads>(up + dn, wave_tot, total);
    const int above_dn = above_up + up;
    if (above_up < need && need <= above_up + up) found[0] = kHardBins - 1 - 2 * t, found[1] = above_up;
    if (above_dn < need && need <= above_dn + dn) found[0] = kHardBins - 2 - 2 * t, found[1] = above_dn;
    __syncthreads();
    lo += (uint32_t)found[0] << shift;
    need -= found[1];
    bits = shift;
    __syncthreads();  // found[] and hist[] are rewritten by the next pass
  }
  // lo is the threshold key; `need` keys equal to it are taken, lowest indices
  // first.  Rounds and wavefronts in index order: 256 counts, scanned by one
  // wavefront.
#pragma unroll
  for (int j = 0; j < kTileRounds; ++j) {
    const bool valid = j < rounds;
    const unsigned long long a = __ballot(valid && k[j] > lo), q = __ballot(valid && k[j] == lo);
    if (lane == 0) cnt_a[j * NW + wave] = __popcll(a), cnt_e[j * NW + wave] = __popcll(q);
  }
  __syncthreads();
  if (wave == 0) {
    constexpr int C = kTileRounds * NW / 64;
    int a[C], q[C], sa = 0, sq = 0;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      a[c] = sa, q[c] = sq;
      sa += cnt_a[C * lane + c], sq += cnt_e[C * lane + c];
    }
    const int ba = wave_inclusive_sum(sa) - sa, bq = wave_inclusive_sum(sq) - sq;
#pragma unroll
    for (int c = 0; c < C; ++c) cnt_a[C * lane + c] = ba + a[c], cnt_e[C * lane + c] = bq + q[c];
  }
  __syncthreads();
  const int64_t out0 = bh * o_bh + (int64_t)sidx * keep;
  const int32_t* idx = src.idx ? src.idx + b * src.s_b + h * src.s_h + begin : nullptr;
#pragma unroll
  for (int j = 0; j < kTileRounds; ++j) {
    const int i = j * kHardThreads + t;
    const bool above = j < rounds && k[j] > lo, tie = j < rounds && k[j] == lo;
    const unsigned long long a = __ballot(above), q = __ballot(tie);
    const int ra = cnt_a[j * NW + wave] + __builtin_amdgcn_mbcnt_hi((uint32_t)(a >> 32),
                                                                     __builtin_amdgcn_mbcnt_lo((uint32_t)a, 0u));
    const int rq = cnt_e[j * NW + wave] + __builtin_amdgcn_mbcnt_hi((uint32_t)(q >> 32),
                                                                     __builtin_amdgcn_mbcnt_lo((uint32_t)q, 0u));
    if (above || (tie && rq < need)) {
      const int64_t at = out0 + ra + min(rq, need);
      if (okey) okey[at] = k[j];
      oidx[at] = idx ? idx[i] : begin + i;
    }
  }
}

// keys per segment of n: whole rounds, the segments about equal
static int tile_segment(int n) {
  const int s = (n + kTileKeys - 1) / kTileKeys;
  return ((n + s - 1) / s + kHardThreads - 1) / kHardThreads * kHardThreads;
}

size_t select_hard_workspace_bytes(int B, int Hkv, int N, int m) {
  if (m < 1 || m > kTileMost || N <= kTileKeys) return 0;
  // two lists of (key, index), the second level's a fraction of the first's
  const int s1 = (N + tile_segment(N) - 1) / tile_segment(N);
  const size_t n1 = (size_t)s1 * m, n2 = n1 / kTileKeys * 2 * m + 2 * (size_t)m;
  return (size_t)B * Hkv * (n1 + n2) * 8;
}

hipError_t launch_select_hard(const float* err, int64_t sE_b, int64_t sE_h, int B, int Hkv, int N, int m,
                              int32_t* out, void* ws, hipStream_t stream) {
  const size_t BH = (size_t)B * Hkv;
  const int segments = (N + tile_segment(N) - 1) / tile_segment(N);
  if (m > 0 && m <= kTileMost && N > kTileLeast && (N <= kTileKeys || ws) && segments < 65536) {
    TileSource src{reinterpret_cast<const uint32_t*>(err), sE_b, sE_h, nullptr, N};
    uint32_t* list = static_cast<uint32_t*>(ws);
    while (src.n > kTileKeys) {
      const int seg = tile_segment(src.n), S = (src.n + seg - 1) / seg;
      const int64_t per = (int64_t)S * m;  // list entries per (b, h); only the last segment may keep fewer than m
      uint32_t* okey = list;
      int32_t* oidx = reinterpret_cast<int32_t*>(list + BH * per);
      select_tile_kernel<<<dim3((unsigned)BH, S), kHardThreads, 0, stream>>>(src, Hkv, seg, m, okey, oidx, per, m);
      const int last = src.n - (S - 1) * seg;
      src = TileSource{okey, (int64_t)Hkv * per, per, oidx, (int)((S - 1) * m + (last < m ? last : m))};
      // (the next level writes past this list, the one after that over the first)
      list = list == static_cast<uint32_t*>(ws) ? list + 2 * BH * per : static_cast<uint32_t*>(ws);
    }
    select_tile_kernel<<<(unsigned)BH, kHardThreads, 0, stream>>>(src, Hkv, kTileKeys, m, nullptr, out, m, 0);
    return hipGetLastError();
  }
  if (m > 0) select_hard_kernel<<<B * Hkv, kHardThreads, 0, stream>>>(err, sE_b, sE_h, Hkv, N, m, out);
  return hipGetLastError();
}

}  // namespace bpc
