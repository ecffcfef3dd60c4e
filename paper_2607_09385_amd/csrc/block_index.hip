// Live-block index build on gfx950: the public index (steel_block_index), and
// below it the form the attention kernels read.
//
// Section IV-A of the paper has every core track the coordinates (i, j) of a
// score tile and either skip it (fully masked), process it as is (unmasked)
// or mask it locally (partially masked).  Here that classification runs once
// per call over the 64x64 block grid and is stored as a compressed list per
// query block: row_ptr (exclusive prefix sum of live counts) and col (live kb,
// bit 31 = partial).  Section IV-C balances the masked work across the
// pipelines; the GPU analogue is a work order that hands out the heaviest
// query blocks first: a stable counting sort by count_bin of the live count.
//
// The public index, three launches in the common case (R <= kFastRows rows):
//   classify     one wave per row, 4 mask bytes per lane: live count
//   scan_small   one workgroup, in LDS: row_ptr and the per-chunk bin
//                histograms turned into scatter bases
//   fill_scatter one wave per row writes its live list; one workgroup per
//                chunk of 256 rows places them in the work order
// Larger problems build the histograms with one workgroup per chunk and scan
// them in a separate single-workgroup kernel.
#include "internal.h"

namespace steel {

__device__ __forceinline__ bool causal_dead(const Problem& p, int qb, int kb) {
  const int last_row = min((qb + 1) * kBlk, p.S_q) - 1;
  return p.causal && (long long)kb * kBlk > (long long)last_row + p.delta;
}

__device__ __forceinline__ bool partial_tile(const Problem& p, int qb, int kb) {
  return (p.causal && (long long)(kb + 1) * kBlk - 1 > (long long)qb * kBlk + p.delta) ||
         (long long)(kb + 1) * kBlk > p.S_k;
}

// Live bits of tiles (qb, kb0 .. kb0+3) of one row (bit e = tile kb0 + e).
// wide: the row holds whole 4-byte words (nKB % 4 == 0, aligned mask).
// Without a mask tensor every block is in the mask, or, in the structured
// mode (p.win_blocks > 0), the window and sink blocks of the coordinates.
__device__ __forceinline__ uint32_t live_quad(const Problem& p, const uint8_t* mrow, bool wide,
                                              int qb, int kb0) {
  uint32_t bytes;
  if (mrow == nullptr) {
    if (p.win_blocks > 0) {
      bytes = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int kb = kb0 + e;
        const bool in = (kb <= qb && kb > qb - p.win_blocks) || kb < p.sink_blocks;
        bytes |= (uint32_t)in << (8 * e);
      }
    } else {
      bytes = 0x01010101u;
    }
  } else if (wide) {
    bytes = kb0 < p.nKB ? *(const uint32_t*)(mrow + kb0) : 0u;
  } else {
    bytes = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (kb0 + e < p.nKB) bytes |= (uint32_t)(mrow[kb0 + e] != 0) << (8 * e);
  }
  uint32_t bits = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int kb = kb0 + e;
    const bool live = kb < p.nKB && ((bytes >> (8 * e)) & 0xffu) != 0 && !causal_dead(p, qb, kb);
    bits |= (uint32_t)live << e;
  }
  return bits;
}

// Live list of one row by one wave, in kb order; each(kb0, bits) sees every
// lane's live bits of tiles kb0 .. kb0 + 3.  Returns the live count.
template <typename Each>
__device__ __forceinline__ int write_list(const Problem& p, const uint8_t* mrow, int wide, int qb,
                                          int lane, uint32_t* list, Each&& each) {
  int pos = 0;
  for (int kb0 = 4 * lane; kb0 - 4 * lane < p.nKB; kb0 += 256) {
    const uint32_t bits = kb0 < p.nKB ? live_quad(p, mrow, wide, qb, kb0) : 0u;
    each(kb0, bits);
    // this 256-block's entries: lane-major, 4 per lane; the entries of earlier
    // lanes counted per bit position (one ballot and one masked bit count)
    int k = pos;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const unsigned long long m = __ballot((bits >> e) & 1u);
      k += (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
      pos += __popcll(m);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if ((bits >> e) & 1u) {
        const int kb = kb0 + e;
        list[k++] = (uint32_t)kb | (partial_tile(p, qb, kb) ? 0x80000000u : 0u);
      }
  }
  return pos;
}

__global__ __launch_bounds__(256) void k_classify(Problem p, const uint8_t* __restrict__ mask,
                                                  int wide, int32_t* __restrict__ cnt) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + wave;
  if (r >= p.R) return;
  const int qb = r % p.nQB;
  const uint8_t* mrow = mask ? mask + (size_t)r * p.nKB : nullptr;
  int c = 0;
  for (int kb0 = 4 * lane; kb0 < p.nKB; kb0 += 256) c += __popc(live_quad(p, mrow, wide, qb, kb0));
  for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off);
  if (lane == 0) cnt[r] = c;
}

// Exclusive scan of one value per thread over a 1024-thread workgroup; the
// sum of all values goes to total.  sh needs 32 ints.
__device__ int wg_exclusive_scan(int x, int* sh, int& total) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  int incl = x;
  for (int off = 1; off < 64; off <<= 1) {
    const int y = __shfl_up(incl, off);
    if (lane >= off) incl += y;
  }
  if (lane == 63) sh[wave] = incl;
  __syncthreads();
  if (wave == 0) {
    int w = lane < 16 ? sh[lane] : 0;
    for (int off = 1; off < 16; off <<= 1) {
      const int y = __shfl_up(w, off);
      if (lane >= off) w += y;
    }
    if (lane < 16) sh[16 + lane] = w;  // inclusive wave totals
  }
  __syncthreads();
  const int base = wave > 0 ? sh[16 + wave - 1] : 0;
  total = sh[31];
  __syncthreads();  // sh is free again
  return base + incl - x;
}

// In-place exclusive scan of a[0 .. n) (LDS or global) by a 1024-thread
// workgroup, contiguous segments per thread; returns the total.  The segment
// length is odd, so the 64 lanes of a wave walking their segments in step hit
// 64 different LDS banks (an even length put up to 8 lanes on one bank).
__device__ int wg_scan_array(int* a, long long n, int* sh) {
  const long long per = ((n + 1023) / 1024) | 1;
  const long long lo = min((long long)threadIdx.x * per, n), hi = min(lo + per, n);
  int s = 0;
  for (long long i = lo; i < hi; ++i) s += a[i];
  int total;
  int run = wg_exclusive_scan(s, sh, total);
  for (long long i = lo; i < hi; ++i) {
    const int x = a[i];
    a[i] = run;
    run += x;
  }
  __syncthreads();
  return total;
}

// Histogram index of (bin, chunk): bins descending from the top bin, then
// chunks, so one exclusive scan yields heaviest-first, stable scatter bases.
// *top_bin holds the top bin.
__device__ __forceinline__ int hist_at(int bin, int chunk, int nch, int top) {
  return (top - bin) * nch + chunk;
}

// Common case: one workgroup does the row_ptr scan and the work-order
// histograms and bases in LDS.
__global__ __launch_bounds__(1024) void k_scan_small(Problem p, const int32_t* __restrict__ cnt_g,
                                                     int32_t* __restrict__ row_ptr,
                                                     int32_t* __restrict__ hist_g,
                                                     int32_t* __restrict__ top_bin) {
  __shared__ int cnt[kFastRows];
  __shared__ int hist[kBins * (kFastRows / kChunk)];
  __shared__ int sh[32];
  constexpr int kPerThread = kFastRows / 1024;
  const int t = threadIdx.x;
  const int R = p.R;
  {
    int v[kPerThread];
#pragma unroll
    for (int j = 0; j < kPerThread; ++j) {
      const int i = t + 1024 * j;
      v[j] = i < R ? cnt_g[i] : 0;
    }
#pragma unroll
    for (int j = 0; j < kPerThread; ++j)
      if (t + 1024 * j < R) cnt[t + 1024 * j] = v[j];
  }
  __syncthreads();

  // row_ptr: prefix sums in hist (free so far), then stored coalesced
  for (int i = t; i < R; i += 1024) hist[i] = cnt[i];
  __syncthreads();
  const int total = wg_scan_array(hist, R, sh);
  for (int i = t; i < R; i += 1024) row_ptr[i] = hist[i];
  if (t == 0) row_ptr[R] = total;

  int top = 0;
  for (int i = t; i < R; i += 1024) top = max(top, count_bin(cnt[i]));
  for (int off = 32; off > 0; off >>= 1) top = max(top, __shfl_xor(top, off));
  if ((t & 63) == 0) sh[t >> 6] = top;
  __syncthreads();
  top = 0;
  for (int w = 0; w < 16; ++w) top = max(top, sh[w]);
  const int nch = nchunks(R), E = (top + 1) * nch;
  __syncthreads();
  for (int i = t; i < E; i += 1024) hist[i] = 0;
  __syncthreads();
  // a wave's 64 items are consecutive rows in one chunk, whose bins come in
  // runs: the first lane of each run of equal entries adds the run's length
  // (the active lanes are a prefix of the wave)
  for (int i = t; i < R; i += 1024) {
    const int at = hist_at(count_bin(cnt[i]), i / kChunk, nch, top);
    const int ln = t & 63;
    const int prev = __shfl_up(at, 1);
    const unsigned long long act = __ballot(true);
    const bool first = ln == 0 || prev != at;
    const unsigned long long starts = __ballot(first);
    if (first) {
      const unsigned long long above = ln == 63 ? 0ull : starts & (~0ull << (ln + 1));
      const int end = above != 0 ? __builtin_ctzll(above) : 64 - __builtin_clzll(act);
      atomicAdd(&hist[at], end - ln);
    }
  }
  __syncthreads();
  wg_scan_array(hist, E, sh);
  for (int i = t; i < E; i += 1024) hist_g[i] = hist[i];
  if (t == 0) *top_bin = top;
}

// Larger problems: per-chunk histograms ...
__global__ __launch_bounds__(256) void k_hist(Problem p, const int32_t* __restrict__ cnt,
                                              int32_t* __restrict__ hist, int nch) {
  __shared__ int h[kBins];
  for (int i = threadIdx.x; i < kBins; i += 256) h[i] = 0;
  __syncthreads();
  const int item = blockIdx.x * kChunk + threadIdx.x;
  if (item < p.R) atomicAdd(&h[count_bin(cnt[item])], 1);
  __syncthreads();
  for (int i = threadIdx.x; i < kBins; i += 256) hist[hist_at(i, blockIdx.x, nch, kBins - 1)] = h[i];
}

// ... and one workgroup scanning them and the counts in global memory.
__global__ __launch_bounds__(1024) void k_scan_large(Problem p, const int32_t* __restrict__ cnt,
                                                     int32_t* __restrict__ row_ptr, int32_t* hist,
                                                     long long nh, int32_t* __restrict__ top_bin) {
  __shared__ int sh[32];
  for (long long i = threadIdx.x; i < p.R; i += 1024) row_ptr[i] = cnt[i];
  __syncthreads();
  const int tot = wg_scan_array(row_ptr, p.R, sh);
  wg_scan_array(hist, nh, sh);
  if (threadIdx.x == 0) {
    row_ptr[p.R] = tot;
    *top_bin = kBins - 1;
  }
}

// Workgroups [0, rows_grid): one wave per row writes the live list of the
// row at row_ptr[r].  The rest: one workgroup per chunk of 256 rows puts each
// at its bin's base for the chunk plus its rank among the chunk's earlier rows
// of the same bin.
__global__ __launch_bounds__(256) void k_fill_scatter(
    Problem p, const uint8_t* __restrict__ mask, int wide, const int32_t* __restrict__ cnt,
    const int32_t* __restrict__ row_ptr, uint32_t* __restrict__ col,
    const int32_t* __restrict__ hist, const int32_t* __restrict__ top_bin,
    int32_t* __restrict__ order, int rows_grid, int nch) {
  __shared__ int bins[kChunk];
  const int t = threadIdx.x;
  if ((int)blockIdx.x < rows_grid) {
    const int wave = t >> 6, lane = t & 63;
    const int r = blockIdx.x * 4 + wave;
    if (r >= p.R) return;
    write_list(p, mask ? mask + (size_t)r * p.nKB : nullptr, wide, r % p.nQB, lane, col + row_ptr[r],
               [](int, uint32_t) {});
    return;
  }
  const int c = (int)blockIdx.x - rows_grid;
  const int item = c * kChunk + t;
  const bool present = item < p.R;
  const int bin = present ? count_bin(cnt[item]) : -1;
  bins[t] = bin;
  __syncthreads();
  if (!present) return;
  int rank = 0;
  const int4* b4 = reinterpret_cast<const int4*>(bins);
  for (int j = 0; j < (t >> 2); ++j) {
    const int4 v = b4[j];
    rank += (v.x == bin) + (v.y == bin) + (v.z == bin) + (v.w == bin);
  }
  for (int j = t & ~3; j < t; ++j) rank += bins[j] == bin;
  order[hist[hist_at(bin, c, nch, *top_bin)] + rank] = item;
}

// ---- index of the attention kernels: two launches ----
//
// The public index above packs the lists (row_ptr needs a scan over all rows)
// and sorts every row in one list.  The attention kernels need neither: a
// row's list may stand at a fixed place, and each XCD takes its own rows.

__device__ __forceinline__ void write_header(const Problem& p, int32_t* n_items) {
  int32_t* h = n_items + kPlanAt;
  h[kPfMagic] = kPlanMagic;
  h[kPfR] = p.R;
  h[kPfNKB] = p.nKB;
  h[kPfPack] = p.pack;
  h[kPfCausal] = p.causal;
  h[kPfDelta] = p.delta;
  h[kPfB] = p.B;
  h[kPfHq] = p.Hq;
  h[kPfHkv] = p.Hkv;
  h[kPfSq] = p.S_q;
  h[kPfSk] = p.S_k;
  n_items[kPackItems] = n_items[1];  // or 0, see kDemotePacks
}

// One wave per row: the live list at col[r * nKB], its length in cnt[r], with
// kUniformBit on the first row of a head pack whose members all have the same
// live set.  Reads each mask byte once (those of a pack's other heads again
// for the comparison, from L2).  Bound by latency: 12,288 rows of 512 blocks
// take 9.3 us against 7 + 10 us of separate count and fill kernels with a scan
// of 14 us between them; 8,192 rows of 256 blocks in packs of 4 7.5 us.
__global__ __launch_bounds__(256) void k_lists(Problem p, const uint8_t* __restrict__ mask, int wide,
                                               int32_t* __restrict__ cnt, uint32_t* __restrict__ col) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + wave;
  if (r >= p.R) return;
  const int qb = r % p.nQB;
  const int h = (r / p.nQB) % p.Hq;
  const uint8_t* mrow = mask ? mask + (size_t)r * p.nKB : nullptr;
  const bool leader = p.pack > 1 && h % p.pack == 0;
  bool same = true;
  const int pos = write_list(p, mrow, wide, qb, lane, col + (size_t)r * p.nKB, [&](int kb0, uint32_t bits) {
    if (leader && mrow && kb0 < p.nKB)
      for (int j = 1; j < p.pack; ++j)
        same &= live_quad(p, mrow + (size_t)j * p.nQB * p.nKB, wide, qb, kb0) == bits;
  });
  const bool uniform = leader && __ballot(!same) == 0ull;
  if (lane == 0) cnt[r] = pos | (uniform ? (int)kUniformBit : 0);
}

// Counting sort of n items by count_bin of their live count, heaviest first,
// by one 1024-thread workgroup: bin_of(i) gives item i's bin (-1: not in the
// list), put(pos, i) receives the items.  Equal bins keep the order of the
// items: each wave takes one sixteenth of them, in order, counts its bins
// (a run of equal bins adds its length once), one scan over (bin descending,
// wave) gives every wave its places, and the waves deal their items out.  (One
// wave dealing out all items in series took 11.5 us for 2,048 packs.)  hist:
// kBins * 16 ints.  Returns the item count.
template <typename Bin, typename Put>
__device__ int wg_sort(int n, int* hist, int* sh, Bin&& bin_of, Put&& put) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
#pragma unroll
  for (int u = 0; u < kBins * 16 / 1024; ++u) hist[t + 1024 * u] = 0;
  __syncthreads();
  // runs of equal bins within a wave: the run's first lane and, there, length
  auto run_of = [&](int bin, bool& first, int& len, int& lead) {
    const int prev = __shfl_up(bin, 1);
    first = lane == 0 || prev != bin;
    const unsigned long long starts = __ballot(first);
    const unsigned long long upto = lane == 63 ? ~0ull : (1ull << (lane + 1)) - 1;
    lead = 63 - __builtin_clzll(starts & upto);
    const unsigned long long above = lane == 63 ? 0ull : starts & (~0ull << (lane + 1));
    len = (above != 0 ? __builtin_ctzll(above) : 64) - lane;
  };
  const int seg = ((n + 1023) / 1024) * 64;  // items per wave
  const int i0 = min(wave * seg, n), i1 = min(i0 + seg, n);
  for (int i = i0 + lane; i - lane < i1; i += 64) {
    const int bin = i < i1 ? bin_of(i) : -1;
    bool first;
    int len, lead;
    run_of(bin, first, len, lead);
    if (first && bin >= 0) atomicAdd(&hist[(kBins - 1 - bin) * 16 + wave], len);
  }
  __syncthreads();
  constexpr int kPer = kBins * 16 / 1024;
  int v[kPer], mine = 0, total;
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    v[u] = mine;
    mine += hist[kPer * t + u];
  }
  const int base = wg_exclusive_scan(mine, sh, total);
#pragma unroll
  for (int u = 0; u < kPer; ++u) hist[kPer * t + u] = base + v[u];
  __syncthreads();
  for (int i = i0 + lane; i - lane < i1; i += 64) {
    const int bin = i < i1 ? bin_of(i) : -1;
    bool first;
    int len, lead;
    run_of(bin, first, len, lead);
    const int at = first && bin >= 0 ? atomicAdd(&hist[(kBins - 1 - bin) * 16 + wave], len) : 0;
    const int run = __shfl(at, lead);
    if (bin >= 0) put(run + lane - lead, i);
  }
  return total;
}

// Work orders.  Single-head rows are dealt to the XCDs by key/value head:
// bucket mb holds the rows of heads g = mb, mb + 8, ... (g = b*Hkv +
// key/value head), in at most kBucketRanges consecutive ranges of heads, and
// within a range heaviest first, so that the workgroups an XCD runs at one
// time read the key/value tiles of one head, which its L2 keeps.  Bucket mb's
// list starts at bucket_start (room for all its rows) and holds bucket[mb]
// items.  One workgroup per (bucket, range) sorts its own rows and counts
// those of the bucket's earlier ranges to find its place; with pack > 1 one
// more sorts the uniform head packs.  A short pack list next to a long
// single-head list (kDemotePacks, kDemoteMinSingle) is left empty and its
// rows go with the single heads.  5 to 7.5 us (24 heads S = 32768: 5.0, 2,048
// packs 7.5) against 8.6 of the partition of a global order it replaces, whose
// sort was part of the scan above.
__global__ __launch_bounds__(1024) void k_orders(Problem p, const int32_t* __restrict__ cnt,
                                                 int32_t* __restrict__ n_items,
                                                 int32_t* __restrict__ order_p,
                                                 int32_t* __restrict__ bucket) {
  __shared__ int hist[kBins * 16];
  __shared__ int sh[32];
  const int t = threadIdx.x;
  const int nkey = bucket_ranges(p), nsingle = kBuckets * nkey;
  int np = 0;  // uniform head packs
  if (p.pack > 1) {
    int mine = 0;
    for (int i = t; i < p.NP; i += 1024) {
      const int bh = i / p.nQB;
      mine += (cnt[bh * p.pack * p.nQB + (i - bh * p.nQB)] & (int)kUniformBit) != 0;
    }
    wg_exclusive_scan(mine, sh, np);
  }
  const int n = p.R - p.pack * np;  // single-head rows (pack 1: all)
  const bool demote = np > 0 && np < kDemotePacks && n >= kDemoteMinSingle;
  if (blockIdx.x == 0 && t == 0) {
    n_items[0] = demote ? p.R : n;
    n_items[1] = np;
    write_header(p, n_items);
    if (demote) n_items[kPackItems] = 0;  // the pack kernels take none
  }
  if ((int)blockIdx.x == nsingle) {
    if (!demote && np > 0)
      wg_sort(
          p.NP, hist, sh,
          [&](int i) {
            const int bh = i / p.nQB;
            const int c = cnt[bh * p.pack * p.nQB + (i - bh * p.nQB)];
            return c & (int)kUniformBit ? count_bin(c & ~(int)kUniformBit) : -1;
          },
          [&](int at, int i) { order_p[at] = i; });
    return;
  }
  const int mb = (int)blockIdx.x / nkey, kk = (int)blockIdx.x % nkey;
  const int rg = p.nQB * p.G, heads = p.B * p.Hkv;
  const int own_b = mb < heads ? (heads - mb + kBuckets - 1) / kBuckets : 0;  // heads of the bucket
  const int nsub = (heads + kBuckets - 1) / kBuckets;
  const int per = (nsub + nkey - 1) / nkey;
  const int h0 = min(kk * per, own_b), h1 = min(h0 + per, own_b);
  // row i of the bucket, and whether the single-head kernel runs it
  auto row_of = [&](int i) {
    const int s = i / rg;
    return (mb + kBuckets * s) * rg + (i - s * rg);
  };
  auto present = [&](int r) {
    if (p.pack == 1 || demote) return true;
    const int bh = r / p.nQB;
    return (cnt[(bh & ~(p.pack - 1)) * p.nQB + (r - bh * p.nQB)] & (int)kUniformBit) == 0;
  };
  int before = h0 * rg;  // items of the bucket's earlier ranges
  if (p.pack > 1 && !demote) {
    int mine = 0;
    for (int i = t; i < h0 * rg; i += 1024) mine += present(row_of(i));
    wg_exclusive_scan(mine, sh, before);
  }
  int32_t* list = bucket + kBuckets + 1 + bucket_start(p.B * p.Hkv, rg, mb) + before;
  const int first = h0 * rg;
  const int got = wg_sort(
      (h1 - h0) * rg, hist, sh,
      [&](int i) {
        const int r = row_of(first + i);
        return present(r) ? count_bin(cnt[r] & ~(int)kUniformBit) : -1;
      },
      [&](int at, int i) { list[at] = row_of(first + i); });
  if (kk == nkey - 1 && t == 0) bucket[mb] = before + got;
}

hipError_t launch_attn_index(const Problem& p, const uint8_t* mask, const IndexBuffers& w,
                             hipStream_t s) {
  const int wide = mask == nullptr || ((p.nKB % 4) == 0 && ((uintptr_t)mask & 3u) == 0);
  hipLaunchKernelGGL(k_lists, dim3((p.R + 3) / 4), dim3(256), 0, s, p, mask, wide, w.cnt, w.col);
  hipLaunchKernelGGL(k_orders, dim3(kBuckets * bucket_ranges(p) + (p.pack > 1 ? 1 : 0)), dim3(1024), 0, s,
                     p, w.cnt, w.n_items, w.order_p, w.bucket);
  return hipGetLastError();
}

hipError_t launch_block_index(const Problem& p, const uint8_t* mask, const PublicIndex& w,
                              hipStream_t s) {
  const int wide = mask == nullptr || ((p.nKB % 4) == 0 && ((uintptr_t)mask & 3u) == 0);
  const int rows_grid = (p.R + 3) / 4, nch = nchunks(p.R);
  hipLaunchKernelGGL(k_classify, dim3(rows_grid), dim3(256), 0, s, p, mask, wide, w.cnt);
  if (p.R <= kFastRows) {
    hipLaunchKernelGGL(k_scan_small, dim3(1), dim3(1024), 0, s, p, w.cnt, w.row_ptr, w.hist, w.top_bin);
  } else {
    hipLaunchKernelGGL(k_hist, dim3(nch), dim3(256), 0, s, p, w.cnt, w.hist, nch);
    hipLaunchKernelGGL(k_scan_large, dim3(1), dim3(1024), 0, s, p, w.cnt, w.row_ptr, w.hist,
                       (long long)kBins * nch, w.top_bin);
  }
  hipLaunchKernelGGL(k_fill_scatter, dim3(rows_grid + nch), dim3(256), 0, s, p, mask, wide, w.cnt,
                     w.row_ptr, w.col, w.hist, w.top_bin, w.order, rows_grid, nch);
  return hipGetLastError();
}

}  // namespace steel
