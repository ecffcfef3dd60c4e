// Block-mask producer on gfx950: for every query block, the key blocks whose
// mean-pooled keys score highest against the mean-pooled queries (top-k of
// the causal candidates, ties to the smaller block), plus the diagonal block.
//
// The paper builds its masks on the compute core instead of fetching them
// (Section III-B) and runs any block mask through the three tile classes of
// Section IV-A; this is the selection rule the sparse workload is defined
// with, moved onto the GPU ahead of the index build.
//
// Floating point decides which blocks are kept, so the arithmetic is fixed:
// float64 throughout, each block sum adds its rows in increasing order, the
// mean divides that sum by the row count (correctly rounded), and each score
// adds the D products in increasing d with every product and sum rounded on
// its own (no fused multiply-add).  Three launches:
//   block_means   one workgroup per (head, block) of Q and of K: the rows
//                 staged in LDS, one thread per column
//   block_scores  64 x 64 score tiles per workgroup from LDS-staged means
//                 (tiles above the diagonal skipped when causal)
//   topk_select   one wave per (head, query block): a search for the boundary
//                 over order-preserving integer keys of the scores (rows of up
//                 to 512 key blocks), or a bitonic sort of the candidates in
//                 LDS (longer rows), then the mask row
#include <algorithm>
#include <climits>

#include "internal.h"

namespace steel {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

// One workgroup per (head, block) of Q, then of K: the block's rows (contiguous
// in memory) are staged into LDS with 16-byte loads, all of them in flight at
// once, then thread d sums column d over the rows in increasing order.  Bound
// by HBM: 201 MB of Q and K.
template <int D>
__global__ __launch_bounds__(D) void k_block_means(const __bf16* __restrict__ q, int Sq, int nQB,
                                                   int nq, double* __restrict__ qm,
                                                   const __bf16* __restrict__ k, int Sk, int nKB,
                                                   double* __restrict__ km) {
  constexpr int kVec = kBlk / 8;  // 16-byte loads per thread of a whole block
  __shared__ __attribute__((aligned(16))) __bf16 tile[kBlk * D];
  const bool isq = (int)blockIdx.x < nq;
  const int g = isq ? (int)blockIdx.x : (int)blockIdx.x - nq;  // (head, block)
  const int S = isq ? Sq : Sk, nb = isq ? nQB : nKB;
  const int bh = g / nb, bi = g - bh * nb;
  const int r0 = bi * kBlk;
  const int cnt = min(kBlk, S - r0);
  const __bf16* p = (isq ? q : k) + ((size_t)bh * S + r0) * D;
  const int nvec = cnt * D / 8, t = threadIdx.x;
  bf16x8_t x[kVec];
#pragma unroll
  for (int u = 0; u < kVec; ++u) x[u] = *(const bf16x8_t*)(p + 8 * min(t + D * u, nvec - 1));
#pragma unroll
  for (int u = 0; u < kVec; ++u)
    if (t + D * u < nvec) *(bf16x8_t*)(tile + 8 * (t + D * u)) = x[u];
  __syncthreads();
  double acc = 0.0;
  if (cnt == kBlk) {
#pragma unroll 16
    for (int r = 0; r < kBlk; ++r) acc = acc + (double)(float)tile[r * D + t];
  } else {
    for (int r = 0; r < cnt; ++r) acc = acc + (double)(float)tile[r * D + t];
  }
  (isq ? qm : km)[(size_t)g * D + t] = acc / (double)cnt;
}

// scores[bh][qb][kb] = dot(qm[bh][qb], km[bh / G][kb]) for one 64 x 64 tile.
// Thread t owns rows 4*(t/16) .. +3 and columns 4*(t%16) .. +3 of the tile.
// Bound by the float64 rate and the LDS operand reads together (12 us each for
// 24 heads of 512 x 512 blocks, causal) and the two barriers per chunk between
// them; 8 x 4 per thread (fewer reads, half the waves) ran 33.6 us against 32.4,
// the tiles above the diagonal as empty workgroups 39.
__global__ __launch_bounds__(256) void k_block_scores(const double* __restrict__ qm,
                                                      const double* __restrict__ km, int nQB,
                                                      int nKB, int D, int G, int Hq, int Hkv,
                                                      int causal, int ntk, int ntiles,
                                                      double* __restrict__ scores) {
#pragma clang fp contract(off)
  constexpr int DC = 32;  // d chunk staged in LDS
  static_assert(kBlk * DC % 256 == 0, "whole staging rounds");
  // rows padded by 2 doubles: the staging writes step over banks and every row
  // stays 16-byte aligned for the paired operand reads
  __shared__ __attribute__((aligned(16))) double qs[DC][kBlk + 2];
  __shared__ __attribute__((aligned(16))) double ks[DC][kBlk + 2];
  const int t = threadIdx.x;
  const int bh = blockIdx.x / ntiles;  // b * Hq + h
  int tq, tk;
  const int ti = blockIdx.x - bh * ntiles;
  if (causal) {
    // tiles (tq, tk <= min(tq, ntk - 1)) row by row: those above the diagonal
    // hold no candidate
    const int sq = ntk * (ntk + 1) / 2;
    if (ti < sq) {
      tq = (int)((sqrtf(8.f * (float)ti + 1.f) - 1.f) * 0.5f);
      while (tq * (tq + 1) / 2 > ti) --tq;
      while ((tq + 1) * (tq + 2) / 2 <= ti) ++tq;
      tk = ti - tq * (tq + 1) / 2;
    } else {
      tq = ntk + (ti - sq) / ntk;
      tk = (ti - sq) % ntk;
    }
  } else {
    tq = ti / ntk;
    tk = ti % ntk;
  }
  const int b = bh / Hq, h = bh - b * Hq;
  const double* qrow = qm + (size_t)bh * nQB * D;
  const double* krow = km + ((size_t)b * Hkv + h / G) * nKB * D;
  const int i0 = 4 * (t >> 4), j0 = 4 * (t & 15);
  double acc[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[a][c] = 0.0;
  // stage qm / km rows of the tile, d-major; the next chunk's loads are issued
  // before this chunk's sums
  constexpr int PER = kBlk * DC / 256;
  double qv[PER], kv[PER];
  auto load = [&](int d0) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int e = t + 256 * u;
      const int r = e / DC, dd = e - r * DC;
      const int qb = tq * kBlk + r, kb = tk * kBlk + r;
      qv[u] = qb < nQB ? qrow[(size_t)qb * D + d0 + dd] : 0.0;
      kv[u] = kb < nKB ? krow[(size_t)kb * D + d0 + dd] : 0.0;
    }
  };
  load(0);
  for (int d0 = 0; d0 < D; d0 += DC) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int e = t + 256 * u;
      const int r = e / DC, dd = e - r * DC;
      qs[dd][r] = qv[u];
      ks[dd][r] = kv[u];
    }
    __syncthreads();
    if (d0 + DC < D) load(d0 + DC);
    // operands of step dd + 1 are read while step dd computes
    double a[2][4], c[2][4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      a[0][u] = qs[0][i0 + u];
      c[0][u] = ks[0][j0 + u];
    }
#pragma unroll
    for (int dd = 0; dd < DC; ++dd) {
      const int cur = dd & 1;
      if (dd + 1 < DC) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          a[cur ^ 1][u] = qs[dd + 1][i0 + u];
          c[cur ^ 1][u] = ks[dd + 1][j0 + u];
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int w = 0; w < 4; ++w) acc[u][w] = acc[u][w] + a[cur][u] * c[cur][w];
    }
    __syncthreads();
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int qb = tq * kBlk + i0 + u;
    if (qb >= nQB) continue;
    double* out = scores + ((size_t)bh * nQB + qb) * nKB;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const int kb = tk * kBlk + j0 + w;
      if (kb < nKB) out[kb] = acc[u][w];
    }
  }
}

// Does candidate a come before candidate b (larger score, then smaller kb)?
__device__ __forceinline__ bool before(double sa, int ia, double sb, int ib) {
  return sa > sb || (sa == sb && ia < ib);
}

// One wave per (head, query block) row, blockDim/64 rows per workgroup.  Each wave
// has its own LDS segment (n2max scores, n2max indices, nKB flags); the
// steps of the sort are separated by a wave-level wait, not a barrier.
__device__ __forceinline__ void wave_lds_sync() {
  // this wave's LDS accesses are done, and the compiler moves none across
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

__global__ __launch_bounds__(256) void k_topk_select(const double* __restrict__ scores, int nQB,
                                                     int nKB, int n2max, size_t seg, int causal,
                                                     long long keep_num, long long keep_den,
                                                     long long n_rows,
                                                     uint8_t* __restrict__ mask) {
  extern __shared__ __attribute__((aligned(16))) char sel_lds[];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const long long row = (long long)blockIdx.x * (blockDim.x >> 6) + w;  // (b*Hq + h)*nQB + qb
  if (row >= n_rows) return;  // the whole wave; no workgroup barrier follows
  char* base = sel_lds + (size_t)w * seg;
  double* s = reinterpret_cast<double*>(base);
  int* id = reinterpret_cast<int*>(base + 8 * (size_t)n2max);
  uint8_t* flag = reinterpret_cast<uint8_t*>(base + 12 * (size_t)n2max);
  const int qb = (int)(row % nQB);
  const int ncand = causal ? min(qb + 1, nKB) : nKB;
  const int keep = (int)((keep_num * ncand + keep_den - 1) / keep_den);
  int n2 = 1;
  while (n2 < ncand) n2 <<= 1;
  const double* src = scores + (size_t)row * nKB;
  for (int j = lane; j < n2; j += 64) {
    s[j] = j < ncand ? src[j] : -INFINITY;
    id[j] = j;
  }
  for (int j = lane; j < nKB; j += 64) flag[j] = 0;
  wave_lds_sync();
  // bitonic sort of n2 entries into "before" order; in each step every lane
  // takes whole compare-exchange pairs (i, i + j), i with bit j clear
  for (int k = 2; k <= n2; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      for (int pr = lane; pr < (n2 >> 1); pr += 64) {
        const int i = ((pr & ~(j - 1)) << 1) | (pr & (j - 1));
        const int l = i + j;
        const bool up = (i & k) == 0;
        const double si = s[i], sl = s[l];
        const int ii = id[i], il = id[l];
        const bool swap = up ? before(sl, il, si, ii) : before(si, ii, sl, il);
        if (swap) {
          s[i] = sl;
          s[l] = si;
          id[i] = il;
          id[l] = ii;
        }
      }
      wave_lds_sync();
    }
  }
  for (int j = lane; j < keep; j += 64) flag[id[j]] = 1;
  if (lane == 0 && qb < nKB) flag[qb] = 1;
  wave_lds_sync();
  uint8_t* dst = mask + (size_t)row * nKB;
  for (int kb = lane; kb < nKB; kb += 64) dst[kb] = flag[kb];
}

// Rows of at most 64 * kSelPerLane key blocks: a selection in registers.  Each
// score becomes an unsigned key in the order of the doubles (both zeros give
// the key of +0, so equal scores give equal keys).  The key T of the keep-th
// largest score is closed in from both sides: lo <= T < hi, where count(lo) =
// candidates with a key >= lo is at least need and count(hi) is less.  A pivot
// with count == need ends the search: the kept set is the keys >= pivot.
// Pivots halve the interval of the scores first (their values are spread more
// evenly than their keys: ~10 steps for 512 scores), from kValueSteps steps on
// the interval of the keys.  The search runs on the upper halves of the keys
// (32-bit compares) and goes on to the whole keys only when scores share the
// boundary's upper half; equal scores end with hi = lo + 1, and of those the
// smallest key block indices are kept, as many as are still missing.  The
// result is the same set as a full sort by (score descending, kb ascending).
// A step is at most 8 compares and bit counts per wave and no LDS.  12,288
// rows of 512 blocks, causal: 33 us with eight byte-wise histogram passes in
// LDS (whose atomics met in a few bins), 22.7 with 64-bit compares throughout,
// 26.4 with pivots interpolated from the counts in every other step, 21.7 so.
constexpr int kSelPerLane = 8;
constexpr int kValueSteps = 24;

__device__ __forceinline__ uint64_t order_key(double x) {
  if (x == 0.0) x = 0.0;  // -0 and +0 compare equal
  const uint64_t u = (uint64_t)__double_as_longlong(x);
  return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}
__device__ __forceinline__ double key_value(uint64_t k) {
  return __longlong_as_double((long long)((k >> 63) ? (k & 0x7fffffffffffffffull) : ~k));
}
__global__ __launch_bounds__(256) void k_topk_select_keys(const double* __restrict__ scores, int nQB,
                                                          int nKB, int causal, long long keep_num,
                                                          long long keep_den, long long n_rows,
                                                          uint8_t* __restrict__ mask) {
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const long long row = (long long)blockIdx.x * 4 + w;  // (b*Hq + h)*nQB + qb
  if (row >= n_rows) return;
  const int qb = (int)(row % nQB);
  const int ncand = causal ? min(qb + 1, nKB) : nKB;
  const int need = (int)((keep_num * ncand + keep_den - 1) / keep_den);  // 1 .. ncand
  const double* src = scores + (size_t)row * nKB;
  uint64_t key[kSelPerLane];  // 0: not a candidate (below every score's key)
  uint32_t hk[kSelPerLane];   // their upper halves
  uint32_t least = ~0u, most = 0u;
#pragma unroll
  for (int c = 0; c < kSelPerLane; ++c) {
    const int j = lane + 64 * c;
    key[c] = j < ncand ? order_key(src[j]) : 0ull;
    hk[c] = (uint32_t)(key[c] >> 32);
    if (j < ncand) least = min(least, hk[c]);
    most = max(most, hk[c]);
  }
  for (int off = 32; off > 0; off >>= 1) {
    least = min(least, (uint32_t)__shfl_xor((int)least, off));
    most = max(most, (uint32_t)__shfl_xor((int)most, off));
  }
  uint64_t lo = __builtin_amdgcn_readfirstlane(least);      // count(lo) = ncand >= need
  uint64_t hi = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane(most) + 1;  // count(hi) = 0
  int above = 0;               // candidates with a key >= hi
  bool whole = need == ncand;  // exactly the keys >= lo are kept
  // one step of the search: pivot mid, n candidates with a key >= mid
  auto close_in = [&](uint64_t mid, int n) {
    if (n >= need) {
      lo = mid;
      whole = n == need;
    } else {
      hi = mid;
      above = n;
    }
  };
  for (int step = 0; !whole && hi - lo > 1; ++step) {
    uint64_t mid = lo + (hi - lo) / 2;
    if (step < kValueSteps) {
      const double x = key_value(lo << 32), y = key_value(hi << 32);
      const uint64_t v = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(order_key(x + (y - x) * 0.5) >> 32));
      if (v > lo && v < hi) mid = v;  // not for NaN, infinities or neighbours
    }
    const uint32_t m32 = (uint32_t)mid;
    int n = 0;
#pragma unroll
    for (int c = 0; c < kSelPerLane; ++c)
      if (64 * c < ncand) n += __popcll(__ballot(hk[c] >= m32));
    close_in(mid, n);
  }
  lo <<= 32;
  hi = whole ? hi : lo + (1ull << 32);  // the boundary's upper half is known
  while (!whole && hi - lo > 1) {
    const uint64_t mid = lo + (hi - lo) / 2;
    int n = 0;
#pragma unroll
    for (int c = 0; c < kSelPerLane; ++c)
      if (64 * c < ncand) n += __popcll(__ballot(key[c] >= mid));
    close_in(mid, n);
  }
  uint8_t* dst = mask + (size_t)row * nKB;
  const int ties = need - above;  // of the keys equal to lo, unless whole
  int eq_before = 0;  // candidates with the boundary key in earlier lane groups
#pragma unroll
  for (int c = 0; c < kSelPerLane; ++c) {
    if (64 * c >= nKB) break;
    const int j = lane + 64 * c;
    bool keep = key[c] >= lo && j < ncand;
    if (!whole) {
      const bool eq = key[c] == lo;
      const uint64_t m = __ballot(eq);
      const int rank = eq_before + __popcll(m & ((1ull << lane) - 1ull));
      keep = key[c] > lo || (eq && rank < ties);
      eq_before += __popcll(m);
    }
    if (j < nKB) dst[j] = keep || j == qb ? 1 : 0;
  }
}

hipError_t launch_topk_mask(const Problem& p, const __bf16* q, const __bf16* k, int keep_num,
                            int keep_den, uint8_t* mask, double* qm, double* km, double* scores,
                            hipStream_t s) {
  const int ntq = (p.nQB + kBlk - 1) / kBlk, ntk = (p.nKB + kBlk - 1) / kBlk;
  const int nq = p.B * p.Hq * p.nQB, nk = p.B * p.Hkv * p.nKB;
  if (p.D == 64)
    hipLaunchKernelGGL(k_block_means<64>, dim3(nq + nk), dim3(64), 0, s, q, p.S_q, p.nQB, nq, qm, k,
                       p.S_k, p.nKB, km);
  else
    hipLaunchKernelGGL(k_block_means<128>, dim3(nq + nk), dim3(128), 0, s, q, p.S_q, p.nQB, nq, qm, k,
                       p.S_k, p.nKB, km);
  // score tiles of a head: all, or with causal structure those up to the diagonal
  const int ntiles = !p.causal ? ntq * ntk
                     : ntq <= ntk ? ntq * (ntq + 1) / 2 : ntk * (ntk + 1) / 2 + (ntq - ntk) * ntk;
  hipLaunchKernelGGL(k_block_scores, dim3(p.B * p.Hq * ntiles), dim3(256), 0, s, qm, km, p.nQB,
                     p.nKB, p.D, p.G, p.Hq, p.Hkv, p.causal, ntk, ntiles, scores);
  const long long rows = (long long)p.B * p.Hq * p.nQB;
  if (p.nKB <= 64 * kSelPerLane) {
    hipLaunchKernelGGL(k_topk_select_keys, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, s,
                       scores, p.nQB, p.nKB, p.causal, (long long)keep_num, (long long)keep_den,
                       rows, mask);
    return hipGetLastError();
  }
  int n2max = 1;
  while (n2max < p.nKB) n2max <<= 1;
  const size_t seg = (12 * (size_t)n2max + (size_t)p.nKB + 15) & ~(size_t)15;  // per wave
  const int wpg = (int)std::max<size_t>(1, std::min<size_t>(4, 65536 / seg));   // waves per group
  hipLaunchKernelGGL(k_topk_select, dim3((unsigned)((rows + wpg - 1) / wpg)), dim3(64 * wpg),
                     wpg * seg, s, scores, p.nQB, p.nKB, n2max, seg, p.causal, (long long)keep_num,
                     (long long)keep_den, rows, mask);
  return hipGetLastError();
}

}  // namespace steel
