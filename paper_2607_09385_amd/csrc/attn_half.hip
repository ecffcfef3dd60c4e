// Fused sparse attention forward in bf16 on gfx950: two waves per query head,
// each holding all 64 query rows of the block and taking half the keys of
// every 64-key tile; or, where workgroups are few, four, each with 32 rows.
//
// The online softmax of Algorithm 1 over the live tiles of a query block
// (Section IV-A masking, Section IV-C work order), split over keys: wave kh of
// a head runs the recurrence over keys 32 kh .. 32 kh + 31 of every tile with
// its own (m, l, O), and the two states of a row are merged at the item's end.
//
// Why this split.  Per tile a wave of 64 rows issues D/4 MFMAs of 32x32x16 and
// the softmax of 64 rows x 32 keys.  Measured on unrolled loops: an MFMA holds
// the matrix core for 32 cycles and the wave's issue for 8, a wave issues other
// VALU instructions every 4 cycles and exponentials every 8.  Counted (D = 64, the
// 24-head S = 32768 top-10% workload): 198 VALU instructions per wave and tile,
// about 150 of them on the common path (32 exponentials), the rest some 0.7
// rescales of 32 rows and the item's start and end; 1,000 cycles of a SIMD's VALU
// against 512 of its matrix core, 1,430 in all.  At D = 128 (Bernoulli masks): 196
// instructions, 1,050 cycles of VALU, 1,024 of the matrix core, 2,590 in all.
// With all 64 rows in one wave a K or V fragment read from LDS feeds two MFMAs
// (with 32 rows: one), which halves the LDS reads, and the per-tile overhead
// (copies, list, waits) is paid once per 64 rows.  Half the keys, because O (64
// rows x D), Q and the scores of 64 keys do not fit the 256 VGPRs that two waves
// per SIMD leave each.  At D = 64 three waves per SIMD fit (162 VGPRs).  Waves of
// 32 rows (RH = 2) have the shorter chain per tile, for calls that do not fill the
// chip; launch_attention_half has the line between the two.
//
// What it is near: on the top-10% workload the VALU is busy 70% of the time, the
// matrix core 36%, the copies into LDS (16 KiB per tile and head, 63 bytes per
// cycle and CU when they hit L2) a third, and the chip's power limit holds the
// clock at 1.9 GHz.  Tried and not faster: rings private to a wave without any
// barrier, deeper rings, two-stage rings for single heads of 64-row waves (fewer
// workgroups per CU), two waves per SIMD at D = 64, the first list entries loaded
// beside the list's length or Q asked for before them (windows of one block, whose
// items are all start and end: equal).
//
// Measured against the kernel it replaced (32 query rows per wave), whole
// calls, that library and this one in turn on one card: 24 heads S = 32768 D = 64
// top-10% 518 -> 486 us, 32 heads S = 8192 D = 128 Bernoulli masks 229 -> 192, 32/8
// heads S = 8192 D = 64 window (packs, prebuilt index) 183 -> 149.
#include <cfloat>
#include <utility>

#include "attn_common.h"

namespace steel {

namespace {

typedef const __attribute__((address_space(3))) char* lds_cp;
typedef const __attribute__((address_space(3))) bf16x8* lds_bf16x8;
typedef __attribute__((address_space(3))) f32x4* lds_f32x4;

template <typename F, int... S>
__device__ __forceinline__ void h_static_for_impl(F&& f, std::integer_sequence<int, S...>) {
  (f(Par<S>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void h_static_for(F&& f) {
  h_static_for_impl(f, std::make_integer_sequence<int, N>{});
}

__device__ __forceinline__ void h_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ uint64_t uniform64(uint64_t p) {
  return ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(p >> 32)) << 32) |
         (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)p);
}

// N (1, 2 or 4) 16-byte global -> LDS copies per lane from one SGPR base: copy
// j writes LDS bytes [lds + 1024 j + 16 lane, +16) from base + off_j.
// The nops: 5 wait states between a VALU write of an SGPR the copies read and
// the first copy, and 1 after each M0 write.
template <int N>
__device__ __forceinline__ void h_copy(uint64_t base, uint32_t lds, const uint32_t* o) {
  static_assert(N == 1 || N == 2 || N == 4, "copies per block");
  if constexpr (N == 4)
    asm volatile(
        "s_mov_b32 m0, %0\n\t"
        "s_nop 4\n\t"
        "global_load_lds_dwordx4 %2, %1\n\t"
        "s_add_u32 m0, m0, 0x400\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %3, %1\n\t"
        "s_add_u32 m0, m0, 0x400\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %4, %1\n\t"
        "s_add_u32 m0, m0, 0x400\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %5, %1"
        :
        : "s"(lds), "s"(base), "v"(o[0]), "v"(o[1]), "v"(o[2]), "v"(o[3])
        : "memory", "m0", "scc");
  else if constexpr (N == 2)
    asm volatile(
        "s_mov_b32 m0, %0\n\t"
        "s_nop 4\n\t"
        "global_load_lds_dwordx4 %2, %1\n\t"
        "s_add_u32 m0, m0, 0x400\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %3, %1"
        :
        : "s"(lds), "s"(base), "v"(o[0]), "v"(o[1])
        : "memory", "m0", "scc");
  else
    asm volatile(
        "s_mov_b32 m0, %0\n\t"
        "s_nop 4\n\t"
        "global_load_lds_dwordx4 %2, %1"
        :
        : "s"(lds), "s"(base), "v"(o[0])
        : "memory", "m0");
}

// The lane number, computed where it stands: values derived from it in rarely
// taken branches of the tile loop then hold no register across it.
__device__ __forceinline__ int opaque_lane() {
  int ln;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(ln));
  return ln;
}

}  // namespace

// The row sums add the bf16-rounded P that the MFMAs consume (v_dot2 against
// (1, 1)), so O / l weights the value rows exactly as used.
template <int NT>
__device__ __forceinline__ void add_rows(const bf16x8 (&pa)[2][NT], float (&l)[NT]) {
  const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      u32x4 w = __builtin_bit_cast(u32x4, pa[t][nt]);
      asm("" : "+v"(w));  // the packed words: the compiler would convert the weights again
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t we = w[e];
        l[nt] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, we), ones, l[nt], false);
      }
    }
}

// End of an item: the two waves of a head hold (m_h, l_h, O_h) over their
// keys, with O_h = sum 2^(s - m_h) v and l_h the sum of the same weights.  With
// M = max(m_0, m_1) and w_h = 2^(m_h - M) the row's state is l = w_0 l_0 + w_1
// l_1, O = w_0 O_0 + w_1 O_1.  Each wave finishes half of the d tiles: it
// leaves the other half of its O, its m and its row sums in its LDS record
// (record wave ^ 1 is its partner's) and reads its partner's.
template <int D, int NT>
__device__ __forceinline__ void merge_rows(const AttnArgs& a, f32x16 (&o)[NT][D / 32], const float (&m)[NT],
                                           const float (&l)[NT], char* smem, int wave, int kh, int lane,
                                           size_t bh, int row0, int nrows, int seg) {
  constexpr int DT = D / 32, HD = DT / 2;
  constexpr int REC = (4 + NT * 16 * HD) * 256;
  const int n = lane & 31, hf = lane >> 5;
  h_barrier();  // the ring is free
  float* mine = (float*)(smem + wave * REC) + lane * 4;
  const float* part = (const float*)(smem + (wave ^ 1) * REC) + lane * 4;
  float lt[NT];
  f32x4 ml_mine = {};
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    lt[nt] = half_pair_sum(l[nt]);
    ml_mine[nt] = m[nt];
    ml_mine[2 + nt] = lt[nt];
  }
  *(f32x4*)mine = ml_mine;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int j = 0; j < HD; ++j) {
      const f32x16 lo = o[nt][j], hi = o[nt][HD + j];
      f32x16 give;
#pragma unroll
      for (int r = 0; r < 16; ++r) give[r] = kh ? lo[r] : hi[r];
#pragma unroll
      for (int r = 0; r < 4; ++r)
        *(f32x4*)(mine + (1 + (nt * HD + j) * 4 + r) * 256) =
            f32x4{give[4 * r], give[4 * r + 1], give[4 * r + 2], give[4 * r + 3]};
    }
  h_barrier();
  const f32x4 pm = *(const f32x4*)part;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const float mp = pm[nt], ltp = pm[2 + nt];
    const float M = fmaxf(m[nt], mp);
    const float w = __builtin_amdgcn_exp2f(m[nt] - M);
    const float wp = __builtin_amdgcn_exp2f(mp - M);
    const float ls = w * lt[nt] + wp * ltp;
    const float inv = ls > 0.f ? 1.f / ls : 0.f;
    const int qrow = row0 + 32 * nt + n;
    if (a.ns > 1) {  // one segment's share: unnormalised, for k_attn_join
      if (qrow < nrows) {
        const size_t row = (size_t)seg * a.part_rows + (bh * a.S_q + qrow - (size_t)a.row0);
        float* ml = a.part + (size_t)a.ns * a.part_rows * D + 2 * row;
        if (hf == 0 && kh == 0) {
          ml[0] = M;
          ml[1] = ls;
        }
#pragma unroll
        for (int j = 0; j < HD; ++j) {
          const f32x16 lo = o[nt][j], hi = o[nt][HD + j];
#pragma unroll
          for (int gq = 0; gq < 4; ++gq) {
            const f32x4 po = *(const f32x4*)(part + (1 + (nt * HD + j) * 4 + gq) * 256);
            f32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = w * (kh ? hi[4 * gq + e] : lo[4 * gq + e]) + wp * po[e];
            *(f32x4*)(a.part + row * D + 32 * (kh * HD + j) + 4 * hf + 8 * gq) = v;
          }
        }
      }
    } else if (qrow < nrows) {
      const size_t row = bh * a.S_q + qrow;
      // log sum_j exp(scale s_ij) = (M + log2 l) ln 2 (Algorithm 1's statistics)
      if (a.lse != nullptr && hf == 0 && kh == 0)
        a.lse[row] = ls > 0.f ? (M + log2f(ls)) * 0.69314718055994531f : -INFINITY;
      const size_t at = row * D + 4 * hf;
#pragma unroll
      for (int j = 0; j < HD; ++j) {
        const int dt = kh * HD + j;
        const f32x16 lo = o[nt][j], hi = o[nt][HD + j];
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
          const f32x4 po = *(const f32x4*)(part + (1 + (nt * HD + j) * 4 + gq) * 256);
          f32x4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = (w * (kh ? hi[4 * gq + e] : lo[4 * gq + e]) + wp * po[e]) * inv;
          if (a.out_bf16)
            *(bf16x4*)((__bf16*)a.out + at + 32 * dt + 8 * gq) =
                bf16x4{(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
          else
            *(f32x4*)(a.out + at + 32 * dt + 8 * gq) = v;
        }
      }
    }
  }
}

// D: head dimension; PACK: heads per workgroup; RH: row halves of a block with a
// wave pair of their own (1: waves of 64 rows, 2: of 32; the same arithmetic,
// bit for bit, since each 32 rows move their maximum by themselves); 2 RH PACK
// waves; ST: stages of the K and of the V ring (1: K and V tiles refilled in turn behind two
// barriers per tile; 2: both one tile ahead, one barrier); RAGGED: S_k is not
// a multiple of the block; WPE: waves per SIMD the registers must allow.
// Single heads with 64-row waves take ST = 1: more workgroups per CU hide more
// than a second stage does (S = 32768 top-10%: 501 us against 560, S = 8192
// Bernoulli 219 against 248).  Packs take ST = 2: their workgroups share each tile between
// two heads, and two (D = 128) or three (D = 64) of them fit a CU either way.
template <int D, int PACK, int RH, int ST, bool RAGGED, int WPE>
__global__ __launch_bounds__(128 * RH * PACK) __attribute__((amdgpu_waves_per_eu(WPE, WPE))) void k_attn_h(AttnArgs a) {
  constexpr int NW = 2 * RH * PACK;  // waves
  constexpr int NT = 2 / RH;         // 32-row N-tiles of a wave
  constexpr int C = D / 8;           // 16-byte chunks per row = 1 KiB copies per tile
  constexpr int RB = D * 2;          // row bytes
  constexpr int TB = kBlk * RB;      // tile bytes
  constexpr int LPW = C / NW;        // copies per wave and tile
  constexpr int CB = LPW < 4 ? LPW : 4;  // copies per assembly block
  constexpr int KS = D / 16, DT = D / 32, HD = DT / 2;
  constexpr float TAU = 8.0f;  // rescale only when a row max grows by > 2^8
  constexpr int V_AT = ST * TB;
  constexpr int REC = (4 + NT * 16 * HD) * 256;  // merge record bytes per wave
  constexpr int LDS_BYTES = 2 * ST * TB > NW * REC ? 2 * ST * TB : NW * REC;
  static_assert(LPW >= 1 && C % NW == 0, "tile copy split");
  __shared__ __attribute__((aligned(1024))) char smem[LDS_BYTES];

  // ---- work item: the item of the list, and the head group within it ----
  const int hp = PACK == 1 ? a.hp : 1;  // heads in the rows of a tile
  const int pk = PACK == 1 ? hp : a.pack, split = PACK == 1 ? 1 : pk / PACK;
  const int x = (int)blockIdx.x & 7, j = (int)blockIdx.x >> 3;
  int sub = j % split, seg = 0;
  int item;
  if (a.coord) {
    // segment by segment, so that the workgroups of one run together
    const int per = (a.units * a.nQB + 7) / 8 * split;  // workgroups of an XCD and segment, at most
    seg = a.ns > 1 ? j / per : 0;
    item = seg < a.ns ? coord_item(a, x, (j - seg * per) / split) : -1;
    if (item < 0) return;
    sub = (j - seg * per) % split;
    item += a.unit0 * a.nQB;
  } else if (PACK == 1) {
    const cint_p bk = (cint_p)a.bucket;
    const int n_b = bk[x];
    const bool ok = plan_matches(a);
    if (j >= n_b) return;
    if (!ok) return;  // index planned for another problem: out untouched
    item = bk[kBuckets + 1 + bucket_start(a.B * a.Hkv, a.nQB * a.G, x) + j];
    if ((unsigned)item >= (unsigned)a.R) return;  // never for a well-formed index
  } else {
    if (!plan_matches(a)) return;  // index planned for another problem: out untouched
    const int idx = xcd_slot((j / split) * 8 + x);
    if (idx >= ((cint_p)a.n_items)[0]) return;
    item = ((cint_p)a.order)[idx];
  }
  const int qb = item % a.nQB;
  const int bh0 = (item / a.nQB) * pk;  // b*Hq + first head of the item
  const int b = bh0 / a.Hq;
  const int h0 = bh0 % a.Hq;
  const int g = h0 / a.G;
  LiveRow lr = live_row(a, bh0 * a.nQB + qb, qb);
  int L = lr.L, p0 = 0;  // list positions p0 .. p0 + L - 1 are this workgroup's
  if (a.ns > 1) {
    p0 = (int)((long long)L * seg / a.ns);
    L = (int)((long long)L * (seg + 1) / a.ns) - p0;
  }

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kh = wave & 1;
  const int r0 = RH == 1 ? 0 : 32 * ((wave >> 1) & 1);  // the wave's first row of the block
  const int head = h0 + sub * PACK + wave / (2 * RH);
  const int n = lane & 31, hf = lane >> 5;
  const size_t kvoff = ((size_t)b * a.Hkv + g) * a.S_k * D;
  const __bf16* kg = a.k + kvoff;
  const __bf16* vg = a.v + kvoff;
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_addr(smem));

  // Copy c = wave*LPW + j of a tile fills its bytes [1024 c + 16 lane, +16):
  // row r = c*(64/C) + lane/C, chunk slot lane % C, which holds source chunk
  // (lane % C) ^ swz(r).  j reaches the row only through bits that are clear
  // in wave*LPW, so the source offset of copy j is that of copy 0 with those
  // bits of the row and of the swizzle flipped.
  auto cp_row = [&](int j) { return (wave * LPW + j) * (64 / C) + lane / C; };
  auto cp_off = [&](int j) -> uint32_t {
    const int r = cp_row(j);
    return (uint32_t)(r * RB + ((lane % C) ^ swz<D>(r)) * 16);
  };
  constexpr int JF = D == 128 ? 1 << 4 : 1 << 5;  // swizzle bits of an odd copy
  uint32_t co0 = cp_off(0);
  auto issue_copy = [&](const __bf16* src, uint32_t dst, int kb) __attribute__((always_inline)) {
    const uint32_t lbase = lds0 + dst + (uint32_t)(wave * LPW) * 1024u;
    if (!RAGGED || (kb + 1) * kBlk <= a.S_k) {
      const uint64_t p = uniform64((uint64_t)(uintptr_t)(src + (size_t)kb * kBlk * D));
      asm volatile("" : "+v"(co0));
      uint32_t co[CB];
#pragma unroll
      for (int j = 0; j < CB; ++j)
        co[j] = co0 ^ (uint32_t)((j << 10) | (D == 128 ? j : j & 1) * JF);
#pragma unroll
      for (int u = 0; u < LPW / CB; ++u)
        h_copy<CB>(p + u * CB * 1024, __builtin_amdgcn_readfirstlane(lbase + u * CB * 1024u), co);
    } else {
      const int ln = opaque_lane();
      for (int j = 0; j < LPW; ++j) {
        const int r = (wave * LPW + j) * (64 / C) + ln / C;
        const int key = min(kb * kBlk + r, a.S_k - 1);
        const uint32_t off = (uint32_t)(key * RB + ((ln % C) ^ swz<D>(r)) * 16);
        copy16_to_lds(src, off, lbase + j * 1024u);
      }
    }
  };
  // ---- live list: 64 entries in a VGPR ----
  uint32_t win = lane < L ? live_entry(a, lr, qb, p0 + lane) : 0u;
  asm volatile("" ::"v"(win));
  uint32_t cw = (uint32_t)__builtin_amdgcn_readlane((int)win, 0), nw = 0;

  if (L > 0) {
    issue_copy(kg, 0, (int)(cw & 0x7fffffffu));
    issue_copy(vg, V_AT, (int)(cw & 0x7fffffffu));
  }
  // Q rows as the B operand (lane: row 32*nt + n, d = 16*ks + 8*hf + 0..7)
  bf16x8 qf[NT][KS];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    // with hp heads in a tile its rows are consecutive rows of q; rows past the
    // end read the last one
    const int br = r0 + 32 * nt + n;
    const size_t row = hp > 1 ? (size_t)min(br, hp * a.S_q - 1) : (size_t)min(qb * kBlk + br, a.S_q - 1);
    const __bf16* qr = a.q + (((size_t)b * a.Hq + head) * a.S_q + row) * D + 8 * hf;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[nt][ks] = *(const bf16x8*)(qr + 16 * ks);
  }
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" ::"v"(qf[nt][ks]));

  // LDS read bases: K fragment ks at kb_ ^ (ks << 5); V^T fragment (t, cc, dt)
  // at (vb_ ^ (dt << 6 | cc << 5)) + (16 t + 8 cc) rows
  const int tg = lane >> 4, tr = (lane >> 2) & 3, tq = lane & 3;
  uint32_t kbase = lds0 + (uint32_t)(kh * 32 * RB + tile_elem<D>(n, hf) * 2);
  uint32_t vbase = lds0 + V_AT +
                   (uint32_t)(kh * 32 * RB +
                              (tile_elem<D>(4 * (tg >> 1) + tr, 2 * (tg & 1) + (tq >> 1)) + 4 * (tq & 1)) * 2);
  auto ld_k = [&](int ks) -> bf16x8 { return *(lds_bf16x8)(lds_cp)(kbase ^ (uint32_t)(ks << 5)); };
  auto ld_v = [&](int q) -> bf16x8 {  // q = t*DT + dt
    const int t = q / DT, dt = q % DT;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (lds_s16x4*)(lds_cp)((vbase ^ (uint32_t)(dt << 6)) + 16 * t * RB));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (lds_s16x4*)(lds_cp)((vbase ^ (uint32_t)((dt << 6) | 32)) + (16 * t + 8) * RB));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };

  f32x16 o[NT][DT];
  float m[NT], l[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    m[nt] = -FLT_MAX;
    l[nt] = 0.f;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[nt][dt] = f32x16{};
  }
  wait_vm<0>();
  h_barrier();

  // K and V^T fragments read ahead of their MFMA.  At D = 128, where O takes
  // 128 registers, two leave the scheduler more room than three (32 heads S =
  // 8192 Bernoulli masks 192 -> 188 us, 1000 queries against 12000 keys 228.5 ->
  // 226.5); at D = 64 three are the better count (469 us against 471 on the 24
  // heads' top-10%, four: 469).
  constexpr int KA = D == 128 ? 2 : 3;
  constexpr int NQ = 2 * DT;
  constexpr int VA = KA;
  if (L > 0) {
#pragma clang loop unroll(disable)
    for (int i = 0;; ++i) {
      const bool more = i + 1 < L;
      // the next entry of the live list (the last tile's again at the end)
      const int in = more ? i + 1 : i;
      if ((in & 63) == 0) {
        const int ln = opaque_lane();
        win = in + ln < L ? live_entry(a, lr, qb, p0 + in + ln) : 0u;
        asm volatile("" ::"v"(win));
      }
      nw = (uint32_t)__builtin_amdgcn_readlane((int)win, in & 63);
      const int nkb = (int)(nw & 0x7fffffffu);
      if constexpr (ST == 2) {
        if (more) {
          const uint32_t at = (uint32_t)(in & 1) * TB;
          issue_copy(kg, at, nkb);
          issue_copy(vg, V_AT + at, nkb);
        }
      }
      // S^T = K Q^T over this wave's 32 keys
      f32x16 sc[NT];
      asm volatile("" : "+v"(kbase), "+v"(vbase));
      {
        bf16x8 kf[KA];
#pragma unroll
        for (int u = 0; u < KA; ++u) kf[u] = ld_k(u);
        __builtin_amdgcn_sched_barrier(0);
        h_static_for<KS>([&](auto kc) __attribute__((always_inline)) {
          constexpr int ks = decltype(kc)::value;
#pragma unroll
          for (int nt = 0; nt < NT; ++nt)
            sc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks % KA], qf[nt][ks],
                                                             ks == 0 ? f32x16{} : sc[nt], 0, 0, 0);
          if constexpr (ks + KA < KS) {
            kf[ks % KA] = ld_k(ks + KA);
            __builtin_amdgcn_sched_barrier(0);
          }
        });
      }
      if constexpr (ST == 1) {
        wait_vm<0>();  // V of this tile
        h_barrier();   // K is free
        if (more) issue_copy(kg, 0, nkb);
      }
      bf16x8 vf[VA];
#pragma unroll
      for (int u = 0; u < VA; ++u) vf[u] = ld_v(u);
      __builtin_amdgcn_sched_barrier(0);
      if (cw >> 31) {  // element mask of a partial tile (Section IV-A case iii)
        const int kb = (int)(cw & 0x7fffffffu), ln = opaque_lane();
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          int row = r0 + 32 * nt + (ln & 31);
          row = hp > 1 ? row % a.S_q : qb * kBlk + row;
          const int lim_abs = min(a.causal ? row + a.delta : INT_MAX - kBlk, a.S_k - 1);
          int lim = lim_abs - (kb * kBlk + 32 * kh + 4 * (ln >> 5));
          asm volatile("" : "+v"(lim));  // one threshold per row, compared with constants
#pragma unroll
          for (int r = 0; r < 16; ++r)
            sc[nt][r] = 8 * (r >> 2) + (r & 3) > lim ? -INFINITY : sc[nt][r];
        }
      }
      // row maxima: the running maximum m of 32 rows moves only when one of them
      // grew by more than TAU (P <= 2^TAU, and m cancels in O / l), so the common
      // tile only compares each lane's own maximum, without the exchange between
      // halves.  2^8 and not more: close to its true maximum a row's largest
      // weights round to bf16 with less error (a weight of 1 with none), which
      // shows where few keys hold a row's mass (24 heads S = 32768 D = 64 top-10%:
      // error against float64 2.5e-4 of the output, 3.4e-4 with 2^24, which is 3%
      // faster there and equal elsewhere).  Each 32 rows by themselves: 503 us
      // there, 508 when both halves are rescaled together.
      {
        float mx[NT];
        bool grow = false;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          mx[nt] = fmaxf(fmaxf(sc[nt][0], sc[nt][1]), sc[nt][2]);
#pragma unroll
          for (int r = 3; r < 15; r += 2) mx[nt] = fmaxf(fmaxf(mx[nt], sc[nt][r]), sc[nt][r + 1]);
          mx[nt] = fmaxf(mx[nt], sc[nt][15]);
          grow |= mx[nt] * a.c > m[nt] + TAU;
        }
        if (__builtin_amdgcn_ballot_w64(grow)) {
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) {
            if (NT > 1 && !__builtin_amdgcn_ballot_w64(mx[nt] * a.c > m[nt] + TAU)) continue;
            const float mnew = fmaxf(m[nt], other_half_max(mx[nt]) * a.c);
            const float alpha = __builtin_amdgcn_exp2f(m[nt] - mnew);
            l[nt] *= alpha;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) o[nt][dt] *= alpha;
            m[nt] = mnew;
          }
        }
      }
      // P = 2^(S c - m) and O^T += V^T P^T, in two 16-key chunks
      bf16x8 pa[2][NT];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
          for (int e = 0; e < 8; ++e)
            pa[t][nt][e] = (__bf16)__builtin_amdgcn_exp2f(__builtin_fmaf(sc[nt][8 * t + e], a.c, -m[nt]));
        }
      h_static_for<NQ>([&](auto qc) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value, t = q / DT, dt = q % DT;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
          o[nt][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[q % VA], pa[t][nt], o[nt][dt], 0, 0, 0);
        if constexpr (q + VA < NQ) vf[q % VA] = ld_v(q + VA);
      });
      add_rows<NT>(pa, l);
      if (!more) break;
      wait_vm<0>();
      h_barrier();
      if constexpr (ST == 1) {
        issue_copy(vg, V_AT, nkb);
      } else {
        const uint32_t step = (i & 1) ? (uint32_t)-TB : (uint32_t)TB;
        kbase += step;
        vbase += step;
      }
      cw = nw;
    }
  }

  merge_rows<D, NT>(a, o, m, l, smem, wave, kh, lane, (size_t)b * a.Hq + head,
                    (hp > 1 ? 0 : qb * kBlk) + r0, hp * a.S_q, seg);
}

// Combines the segments of split lists: with M = max m_s over the segments and
// w_s = 2^(m_s - M), O = sum w_s O_s / sum w_s l_s.  One wave per row: lane s
// holds segment s's m, l and weight (at most 64 segments), then every lane
// adds its D/64 columns over the segments, 8 loads in flight.  Latency bound:
// the parts of 128 rows are 2 MB.
template <int D>
__global__ __launch_bounds__(256) void k_attn_join(AttnArgs a) {
  constexpr int V = D / 64;
  typedef float vec __attribute__((ext_vector_type(V)));
  const int lane = threadIdx.x & 63;
  const long long r = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= a.part_rows) return;
  const float* ml = a.part + (size_t)a.ns * a.part_rows * D;
  const size_t at = 2 * ((size_t)min(lane, a.ns - 1) * a.part_rows + r);
  const float m = ml[at];
  float M = m;
  for (int off = 32; off > 0; off >>= 1) M = fmaxf(M, __shfl_xor(M, off));
  const float w = lane < a.ns ? __builtin_amdgcn_exp2f(m - M) : 0.f;
  float ls = w * ml[at + 1];
  for (int off = 32; off > 0; off >>= 1) ls += __shfl_xor(ls, off);
  const float* src = a.part + (size_t)r * D + V * lane;
  const size_t step = (size_t)a.part_rows * D;
  float v[V] = {};
#pragma unroll 8
  for (int s = 0; s < a.ns; ++s) {
    const float ws = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(w), s));
    const vec o = *(const vec*)(src + s * step);
#pragma unroll
    for (int e = 0; e < V; ++e) v[e] += ws * o[e];
  }
  const float inv = ls > 0.f ? 1.f / ls : 0.f;
  const size_t row = (size_t)a.row0 + r;
  if (a.lse != nullptr && lane == 0)
    a.lse[row] = ls > 0.f ? (M + log2f(ls)) * 0.69314718055994531f : -INFINITY;
#pragma unroll
  for (int e = 0; e < V; ++e) {
    if (a.out_bf16) ((__bf16*)a.out)[row * D + V * lane + e] = (__bf16)(v[e] * inv);
    else a.out[row * D + V * lane + e] = v[e] * inv;
  }
}

template <int D, int PACK, int RH, int ST, int WPE>
static void launch_h(const AttnArgs& a, int grid, hipStream_t s) {
  if (a.S_k % kBlk != 0)
    hipLaunchKernelGGL((k_attn_h<D, PACK, RH, ST, true, WPE>), dim3(grid), dim3(128 * RH * PACK), 0, s, a);
  else
    hipLaunchKernelGGL((k_attn_h<D, PACK, RH, ST, false, WPE>), dim3(grid), dim3(128 * RH * PACK), 0, s, a);
}

// 32-row waves (RH = 2) or 64-row waves, from the workgroups an XCD gets at
// most.  64 rows halve the LDS reads and cost a workgroup half the waves, so
// they are the better form once the chip is full; while it is not, a call lasts
// as long as the chain of its longest list, and 32-row waves have the shorter
// chain per tile.  At one tile in LDS (ST = 1) more workgroups fit a CU, at two
// a tile's copy hides behind the one before it.  Single heads, us, by
// workgroups per XCD, 64-row waves / 32-row waves:
//   D = 64 (6 / 4 workgroups per CU), causal lists from an index: 64 of S =
//   2048 41.6 / 26.4, 128 44.6 / 41.1, 256 62.2 / 59.6, 512 105.4 / 101.5;
//   windows of 8 blocks: 320 38.3 / 35.5, 768 74.3 / 73.9; random 10%: 24 heads S =
//   16384 (768) 122.4 / 120.1, 32/8 (1,024) 155 / 161, 24 heads S = 32768 (1,536) 434 /
//   447.  Dense, no index, S = 2048: 320 112 / 108, 384 126 / 128,
//   causal 320 62 / 64, 384 72 / 77.  Just full with 64-row waves (161 to 192)
//   equal lists run 65.7 / 67.7, causal ones from an index 58.1 / 44.1; decoding, 15/5
//   heads, batch of 64, 6000 keys (160) 92.3 / 101.3.
//   D = 128 (4 of 64-row waves; 2 of 32-row waves with two tiles, 3 with one),
//   causal lists from an index, S = 2048: 64 57.2 / 39.3 / 37.6, 128 65.5 / 56.1 /
//   55.3, 192 82.1 / 78.2 / 75.3, 256 103.4 / 101.4 / 95.9; 512 tokens against
//   4000, batch of 4 (64) 95.1 / 69.8 / 90.7.  Dense, no index, S = 2048: 96 63.9 /
//   67.0 / 59.6, 128 76.5 / 82.8 / 81.4 (causal 54.2 / 51.1 / 46.6), 192 129.6 / 121.8 /
//   113.2, 256 147 / 167 / 149; 256 causal queries against 4096 keys (128, nearly equal
//   lists) 176 / - / 217.  An index does not tell whether its lists are of
//   one length: windows of 8 blocks at 128 take 29.5 / 32.7 / 32.5 (S = 1024, where
//   lists differ by less: 28.4 / 31.5 / 31.7, causal 39.2 / 39.4 / 38.0).  Decoding, 32
//   heads, batch of 64, 2000 keys (256; HBM): 372 / 349 / 355.
static bool rows32_d64(const AttnArgs& a, int per, bool equal) {
  return per <= (a.coord ? 320 : 800) && !(equal && per > (a.nQB == 1 ? 136 : 160) && per <= 192);
}
static bool rows32_d128(const AttnArgs& a, int per, bool equal) {
  const bool some = a.nKB > 16;
  if (!a.coord) return per <= 256 && (some || per <= 112 || per > 128);
  return per <= 96 || (per <= 128 ? !equal && some : per <= 192);
}

hipError_t launch_attention_half(const AttnArgs& a, int D, int pack, int items, bool equal, hipStream_t s) {
  if (items <= 0) return hipSuccess;
  if (pack == 1) {
    const int grid = a.coord ? items * a.ns : items, per = grid / 8;
    if (D == 64) {
      if (rows32_d64(a, per, equal)) launch_h<64, 1, 2, 2, 4>(a, grid, s);
      else launch_h<64, 1, 1, 1, 3>(a, grid, s);
    } else {
      if (per <= 64 || (a.coord && a.nQB == 1 && per > 192)) launch_h<128, 1, 2, 2, 2>(a, grid, s);
      else if (rows32_d128(a, per, equal)) launch_h<128, 1, 2, 1, 3>(a, grid, s);
      else launch_h<128, 1, 1, 1, 2>(a, grid, s);
    }
  } else {
    // Pairs of heads: 16/8 heads S = 2048 causal from an index, 64-row / 32-row
    // waves, by workgroups per XCD: D = 64 (3 / 2 per CU) 32 31.0 / 26.9, 64 33.1 /
    // 31.9, 96 41.9 / 44.4; D = 128 (2 / 1) 32 42.6 / 37.4, 64 53.0 / 56.9.
    const int grid = (a.coord ? (items + 7) / 8 * 8 * a.ns : xcd_grid(items)) * (pack / 2);
    const int per = (items + 7) / 8 * a.ns * (pack / 2);
    if (D == 64) {
      if (per <= 64) launch_h<64, 2, 2, 2, 4>(a, grid, s);
      else launch_h<64, 2, 1, 2, 3>(a, grid, s);
    } else {
      if (per <= 32) launch_h<128, 2, 2, 2, 2>(a, grid, s);
      else launch_h<128, 2, 1, 2, 2>(a, grid, s);
    }
  }
  return hipGetLastError();
}

hipError_t launch_attention_join(const AttnArgs& a, int D, hipStream_t s) {
  const dim3 grid((unsigned)((a.part_rows + 3) / 4));
  if (D == 64) hipLaunchKernelGGL(k_attn_join<64>, grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL(k_attn_join<128>, grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace steel
