// Internal interfaces between the C ABI layer and the gfx950 kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace steel {

constexpr int kBlk = 64;          // mask block edge = tile edge
constexpr int kBins = 512;        // work-order bins (count_bin < kBins)
constexpr int kChunk = 256;       // items per work-order chunk

// Work-order bin of a live count c in [0, 2^31): c itself below 128; above,
// 16 bins per octave, 128 + 16*(e - 7) + (the 4 bits below the leading one),
// e = floor(log2 c).  Monotone in c, exact where the counts are small, and
// within 1/16 of the count where they are large.
__host__ __device__ inline int count_bin(int c) {
  if (c < 128) return c;
  const int e = 31 - __builtin_clz((unsigned)c);
  return 128 + 16 * (e - 7) + ((c >> (e - 4)) & 15);
}

// Problem description shared by the index build and the attention kernels.
struct Problem {
  int B, Hq, Hkv, S_q, S_k, D;
  int G;        // Hq / Hkv
  int pack;     // query heads of one group processed together (1, 2 or 4)
  int nQB, nKB;
  int causal;
  int delta;    // S_k - S_q
  int R;        // B*Hq*nQB rows of the live-block list
  int NP;       // B*(Hq/pack)*nQB head packs (0 when pack == 1)
  // Block mask from coordinates instead of a mask tensor (win_blocks > 0):
  // block (qb, kb) is in the mask iff qb - win_blocks < kb <= qb (a window
  // of win_blocks blocks ending at the block diagonal) or kb < sink_blocks.
  // The index kernels then read no mask (the paper generates masks on the
  // core rather than fetching them, Section III-B; windowed attention is the
  // masking scheme Section IV-A names).
  int win_blocks, sink_blocks;
  // Set by the fused calls when every query head has the same block mask (no
  // mask tensor, or the structured mask): with pack > 1 every head pack is
  // then uniform and the single-head list is empty, so it is not launched.
  int heads_share_mask;
  // Set by the fused calls without a mask tensor: the attention kernels compute
  // rows and live lists from the coordinates, and no index is built.
  int coord;
  int out_bf16;  // output in bf16 (RNE of the fp32 result) instead of fp32
  int fp8;       // operand precision of the products: a Prec value
};

// Operand precision of Algorithm 1's two products: bf16 (the paper's AIE
// datapath, Section II-C), E4M3 for P V only, or E4M3 for both (see
// Fp8Buffers); accumulation is fp32 in every case.
enum Prec { kBf16 = 0, kFp8Pv = 1, kFp8All = 2 };

// Operands of the fp8 form, written by the pre-pass (quant_fp8.hip) and read
// by the attention kernels.  Both tensors are cut into the 64-key tiles of
// the mask, tile (b*Hkv + g, kb) at byte (b*Hkv + g) * nKB * 64 * D +
// kb * 64 * D, keys past S_k zero; each tile is stored exactly as the
// kernels keep it in LDS, so one straight copy moves it:
//   k8  row r (key 64 kb + r) of D bytes E4M3(K s_k); its 16-byte chunk c
//       (dims 16c .. 16c + 15) at chunk slot c ^ kswz(r) of the row;
//   v8  row d of 64 bytes E4M3(V s_v) over the tile's keys in the order of
//       the P operand (byte j = 32 h + b holds key 32 (b/16) + 8 ((b%16)/4)
//       + 4 h + b%4); its chunk c at slot c ^ ((d >> 2) & 3).
// The swizzles keep the 16-byte operand reads of 16 lanes on distinct LDS
// banks.  scale: per (b*Hkv + g) the two inverse scales {1/s_k, 1/s_v};
// part: the per-chunk maxima the scales come from.  k8 is nullptr when
// only P V takes E4M3 operands.
struct Fp8Buffers {
  uint8_t* k8;
  uint8_t* v8;
  float* part;   // [B*Hkv][kFp8Chunks][2]
  float* scale;  // [B*Hkv][2]
};
constexpr int kFp8Chunks = 128;
constexpr float kE4M3Max = 448.f;

template <int D>
__host__ __device__ inline int kswz8(int r) {
  return D == 128 ? (r >> 1) & 7 : (r >> 2) & 3;
}

// Power-of-two scale 2^floor(log2(448 / amax)) of a tensor whose largest
// magnitude is amax (1 for 0 or a non-finite amax).
__host__ __device__ inline float e4m3_scale(float amax) {
  if (!(amax > 0.f) || !(amax <= 3.4e38f)) return 1.f;
  const float x = kE4M3Max / amax;  // >= 1.3e-36: a normal float
  uint32_t bits;
  __builtin_memcpy(&bits, &x, 4);
  bits &= 0x7f800000u;              // 2^floor(log2 x)
  if (bits == 0x7f800000u) bits = 0x7f000000u;  // x overflowed: 2^127
  float sc;
  __builtin_memcpy(&sc, &bits, 4);
  return sc;
}

// Index read by the attention kernels.
struct IndexBuffers {
  int32_t* cnt;        // [R]   live blocks per row (| kUniformBit, see below)
  uint32_t* col;       // [R*nKB] the list of row r at r * nKB
  int32_t* order_p;    // [NP]  uniform head packs, heaviest first
  int32_t* n_items;    // [kHeaderInts] {single items, pack items, plan header,
                       //   pack items the pack kernels take}
  // single-head items dealt to the 8 XCDs by key/value head: [kBuckets] item
  // counts, one unused, then bucket mb's items from bucket_start on
  int32_t* bucket;
};

// Public index and its workspace.
struct PublicIndex {
  int32_t* cnt;      // [R]
  int32_t* hist;     // [kBins * chunks] per-chunk bin counts, then bases
  int32_t* top_bin;  // [1]
  int32_t* row_ptr;  // [R+1]
  uint32_t* col;     // [R*nKB] capacity
  int32_t* order;    // [R] rows, heaviest first
};

// XCD buckets of single-head items: bucket (b*Hkv + g) % kBuckets, so that the
// workgroups of one XCD read the key/value tensors of only a few heads and
// its L2 keeps them.
constexpr int kBuckets = 8;

// Head ranges of a bucket: its key/value heads g = mb, mb + 8, ... (at most
// ceil(B*Hkv / 8)) split into at most kBucketRanges consecutive ranges.
constexpr int kBucketRanges = 8;
__host__ __device__ inline int bucket_ranges(const Problem& p) {
  const int nsub = (p.B * p.Hkv + kBuckets - 1) / kBuckets;
  return nsub < kBucketRanges ? nsub : kBucketRanges;
}

// Plan header written after the two item counts; the attention kernels check
// it against their own arguments before touching the index, so a run with
// other sizes, another causal limit or another head packing than the plan
// leaves its output untouched.  Layout of n_items: [0] single-head items,
// [1] head-pack items, [kPlanAt + f] field f of PlanField, [kPackItems] the
// head-pack items the pack kernels take (n_items[1], or 0 when a short pack
// list goes to the single-head kernel, see kDemotePacks).
constexpr int kPlanMagic = 0x5354454c;  // "STEL"
enum PlanField { kPfMagic, kPfR, kPfNKB, kPfPack, kPfCausal, kPfDelta, kPfB, kPfHq, kPfHkv,
                 kPfSq, kPfSk, kPlanFields };
constexpr int kPlanAt = 2;
constexpr int kPackItems = kPlanAt + kPlanFields;
constexpr int kHeaderInts = kPackItems + 1;

// A head-pack list shorter than kDemotePacks (a quarter of the CUs) is run
// by the single-head kernel, as pack-many rows per item, when that kernel
// has at least kDemoteMinSingle items of its own: a pack kernel for a few
// items would add one item's latency to the run while most CUs idle, and the
// single-head kernel absorbs the rows.  The rows of a uniform pack have one
// live list, so either kernel computes the same rows.
constexpr int kDemotePacks = 64;
constexpr int kDemoteMinSingle = 1024;

// Calls without a mask tensor whose query blocks are too few to fill the chip
// (decoding, short chunks of queries against a long key cache), bf16 only:
// every live list is cut into ns segments, each run by a workgroup of its own
// that leaves its partial (m, l, O) in scratch, and k_attn_join combines them.
// With a single query block, split or not, the hp query heads of a group whose
// rows fit one 64-row tile together are run as one item (hp = 1: one head per tile).
struct SplitPlan {
  int ns;             // segments per list (1: not split)
  int hp;             // query heads packed into one tile's rows
  size_t unit_bytes;  // scratch per unit (hp heads, or the heads of a pack) when ns > 1
  int units;
};
SplitPlan plan_split(const Problem& p);

// Up to this many head packs of 4 at D = 128 (bf16) are run two heads to a
// workgroup (k_attn_h) instead of four (k_attn_ws): with one persistent
// workgroup per CU and no more packs than CUs, CUs stand idle or wait for the
// longest pack.  Runs of plans, us, by fours / by twos: 64 packs causal S = 2048
// 56.2 / 41.2, 128 packs 57.0 / 41.1, 192 57.6 / 51.0, 256 59.4 / 54.5, 384 64.2 / 72.8.
// From 129 packs on lists of about one length go the other way (1536 queries
// against 9000 keys, 192 packs 212.7 / 251.1; 128 packs 206.2 / 151.8; windows of 8
// blocks S = 2048, 192 packs 27.2 / 29.2), which a plan does not tell, and by fours
// the scaled Q is rounded to bf16: one line for both.
constexpr int kFewPacks = 256;

// Order of the items of a call without an index (unit * nQB + query block; a
// unit is a head, or the heads of a pack or of a tile).  XCD x takes positions
// 0, 1, ... of its share, coord_items of them; coord_item is -1 past the end.
// range > 0: the units are taken in ranges of that many (a multiple of 8);
//   within a range heaviest query blocks first (the live count grows with the
//   query block but for a window's first blocks), the units of one query block
//   next to each other.  XCD x takes every eighth item, which are those of
//   every eighth unit of a range of whole eights.  The m units of a key/value
//   group (heads that read the same keys and values) are placed on one XCD, as
//   long as eight groups are left (coord_unit).
// range == 0: unit by unit, XCD x takes the x-th eighth.
// (Single-head units D = 128, batch of 8, 1000 queries against 4000 keys, 40/8
// heads: 1,055 us with the units of a group on all XCDs, 638 on one; batch of
// 64, 17 queries, 727 and 428.)
__host__ __device__ inline int coord_unit(int units, int m, int v) {
  if (m == 1 || v >= units / (8 * m) * (8 * m)) return v;
  const int b = v / (8 * m), in = v - b * (8 * m);
  return (8 * b + in % 8) * m + in / 8;
}
__host__ __device__ inline int coord_items(int units, int nQB, int range, int x) {
  const int n = units * nQB, per = (n + 7) / 8;
  if (range > 0) return (n - x + 7) / 8;
  const int left = n - x * per;
  return left < 0 ? 0 : left < per ? left : per;
}
__host__ __device__ inline int coord_item(int units, int nQB, int range, int m, int x, int pos) {
  if (pos >= coord_items(units, nQB, range, x)) return -1;
  if (range == 0) {
    const int idx = x * ((units * nQB + 7) / 8) + pos, u = idx / nQB;
    return u * nQB + (nQB - 1 - (idx - u * nQB));
  }
  const int idx = 8 * pos + x, u0 = idx / (range * nQB) * range;
  const int in = idx - u0 * nQB, n = units - u0 < range ? units - u0 : range, k = in / n;
  return coord_unit(units, m, u0 + in - k * n) * nQB + (nQB - 1 - k);
}

// Whether the lists of a call without an index are of about one length: they
// differ by a quarter of the longest at most (windows: but for their first
// blocks).
inline bool equal_lists(const Problem& p) {
  if (!p.causal || p.win_blocks > 0) return true;
  auto len = [&](long long row) {  // blocks up to the last key that the row sees
    const long long end = row + p.delta + 1;
    const long long n = end > 0 ? (end + kBlk - 1) / kBlk : 0;
    return n < p.nKB ? n : p.nKB;
  };
  const long long most = len(p.S_q - 1), least = len(kBlk - 1 < p.S_q ? kBlk - 1 : p.S_q - 1);
  return 4 * (most - least) <= most;
}

// The range, for an L2 of 4 MiB per XCD: the workgroups an XCD runs at one time
// (32 to 192) should read the keys and values of few units.  Lists of equal
// length (no causal limit) lose nothing by short ranges: 128 items per XCD.
// Causal ones restart with the heaviest query blocks in each range, so ranges
// are longer: 512 items.  32 heads D = 128, batch of 16, S = 2048, no causal
// limit: 2,315 us as one range, 1,206 with 128 items, 1,888 with 512 (an index
// per call, head by head: 1,461); causal 1,155, 730 and 731 (956); batch of 8,
// S = 4096, window of 16 blocks: 1,060, 674 and 742 (874).
// Without a window a range also has no more units than 8 MiB of keys and values, or
// 8 (16 where causal lists differ by more than a quarter): with few query blocks
// more of them lie so far apart that they do not read a unit's keys together.  256 causal queries D = 64, with
// 512 items / 128 (32 units) / 16 units / 8 (head by head): 40 heads, batch of 16, 2816
// keys 255 / 182 / 168 / 173 us (203), 24 heads, 15616 keys 763 / 633 / 593 / 555
// (570); 32 heads D = 128, batch of 16, 512 queries against 2048 keys, 512 items 474,
// 8 units 322 (359); 64 heads, 640 against 1280, 512 items 703, 16 units 489 (551).
// The ranges are of about one size: a last one of few heads would begin the
// heaviest lists when the others end (24 heads batch of 3 S = 4096 causal, 8 + 1
// heads per XCD: 225 us at D = 64, 192 as one range of 9).
// Windows over single heads, not a multiple of 8: eight contiguous shares,
// since every eighth item would have each XCD read every head (6 heads S =
// 32768 D = 128, 16 blocks: 244 -> 129 us; 20 heads batch of 3 S = 4096: 255 ->
// 155).  From 1,024 items on: below, a share without a unit's light first
// blocks takes a round longer (282 items 18.8 -> 22.4 us).  Packs stay in ranges
// (12/3 heads batch of 3 S = 4096: 83 us against 101).
inline int coord_range(int units, const Problem& p, bool single) {
  const int nQB = p.nQB;
  const bool window = p.win_blocks > 0;
  if (window && single && units % 8 != 0 && units * nQB >= 1024) return 0;
  const int items = p.causal || window ? 512 : 128;
  int per = (items + nQB - 1) / nQB;
  if (!window) {
    const int least = equal_lists(p) ? 8 : 16;
    const int bytes = p.fp8 == kFp8All ? 2 : p.fp8 ? 3 : 4;  // of a key's and its value's element
    const long long kv = ((long long)8 << 20) / ((long long)p.S_k * p.D * bytes);
    const int most = kv > least ? (int)(kv < per ? kv : per) : least;
    if (most < per) per = most;
  }
  const int all = (units + 7) / 8;
  const int n = (2 * all + per) / (2 * per);  // all / per, rounded to nearest
  return 8 * (n > 1 ? (all + n - 1) / n : all);
}

__host__ __device__ inline int nchunks(int n) { return (n + kChunk - 1) / kChunk; }

// Set in cnt[r] of the first row of a head pack whose rows all have the same
// live list (counts are below 2^30: R * nKB < 2^31).
constexpr uint32_t kUniformBit = 1u << 30;

// Up to this many rows one workgroup scans the counts and the work-order
// histograms in LDS (4 + 4 * kBins / kChunk = 12 bytes per row: 144 KiB).
constexpr int kFastRows = 12288;

// Size of the fixed per-device scratch array of steel_attn_fwd_noalloc (the
// live-block index of one call: counts, histograms, row_ptr, the list
// capacity R * nKB and the work orders).  Equals STEEL_NOALLOC_SCRATCH_BYTES.
constexpr size_t kNoAllocBytes = (size_t)32 << 20;

// Device address of this device's copy of that array (looked up on the
// first call for a device, with the device made current, then cached).
hipError_t noalloc_scratch(int dev, char** ptr);

// First list position of bucket mb: the rows of the heads of the buckets before
// it (heads = B*Hkv, rg = rows of a key/value head).
__host__ __device__ inline int bucket_start(int heads, int rg, int mb) {
  const int rest = heads % kBuckets;
  return rg * (mb * (heads / kBuckets) + (mb < rest ? mb : rest));
}

// Enqueue the build of the index the attention kernels read: cnt, col with the
// list of row r at r * nKB, order_p, bucket and the header.  With p.pack == 1
// every row is a single-head item.
hipError_t launch_attn_index(const Problem& p, const uint8_t* mask, const IndexBuffers& w,
                             hipStream_t stream);

// Enqueue the build of the public index (row_ptr, col, order).
hipError_t launch_block_index(const Problem& p, const uint8_t* mask, const PublicIndex& w,
                              hipStream_t stream);

// Enqueue the top-k mean-pooled block selection (block_select.hip): writes the
// whole block mask [B][Hq][nQB][nKB].  qm, km, scores: float64 workspace of
// B*Hq*nQB*D, B*Hkv*nKB*D and B*Hq*nQB*nKB values.  Needs nKB <= 4096.
hipError_t launch_topk_mask(const Problem& p, const __bf16* q, const __bf16* k, int keep_num,
                            int keep_den, uint8_t* mask, double* qm, double* km, double* scores,
                            hipStream_t stream);

// Enqueue the fp8 pre-pass: per (b, g) maxima of |K| and |V|, their scales
// and the E4M3 tiles of Fp8Buffers.
hipError_t launch_fp8_prepass(const Problem& p, const void* k, const void* v, const Fp8Buffers& f,
                              hipStream_t stream);

// Enqueue the fused attention over both item lists; lse (nullable) receives
// the row log-sum-exp [B][Hq][S_q].  f: the fp8 operands when p.fp8, else
// ignored.
// part: scratch for the partial results of plan_split (at least one unit's; the
// units are taken in as many batches as it needs), or nullptr when ns == 1.
hipError_t launch_attention(const Problem& p, const void* q, const void* k, const void* v,
                            float* out, float* lse, float scale, const IndexBuffers& w,
                            const Fp8Buffers& f, float* part, size_t part_bytes, hipStream_t stream);

// Enqueue the merge of n_parts partial results over disjoint key sets
// (attn_merge.hip): o_parts [n_parts][rows][D], lse_parts [n_parts][rows].
hipError_t launch_merge(const float* o_parts, const float* lse_parts, int n_parts, long long rows,
                        int D, float* out, float* lse_out, hipStream_t stream);

}  // namespace steel
