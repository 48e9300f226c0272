// The tile kernel of short calls: launches of one round of workgroups whose pieces walk few key blocks (see attn_short).  Part of
// vs_attn.hip.
#pragma once

#include "vs_common.h"

namespace vs {

// x / d for x d < 2^32, with m = short_magic(d): the quotients of a call's shape, one instruction each
static inline uint32_t short_magic(uint32_t d) { return d > 1 ? (uint32_t)((0x100000000ull + d - 1) / d) : 0u; }
__device__ __forceinline__ int short_quotient(int x, uint32_t m) { return m ? (int)(((uint64_t)(uint32_t)x * m) >> 32) : x; }

struct ShortArgs {
  const __bf16* q;
  const __bf16* k;
  const __bf16* v;
  __bf16* out;
  float* lse;
  float* part_o;    // as in AttnArgs
  float* part_ml;
  int64_t q_stride_head, k_stride_head, v_stride_head, o_stride_head;
  int32_t q_stride_tok, k_stride_tok, v_stride_tok, o_stride_tok;   // (below 2^23)
  int32_t n_pieces, each, n_units, n_qtiles, n_hs, n_split;
  uint32_t by_units, by_qtiles, by_hs, by_split;   // short_magic of them
  int32_t pack, group, row_pad, q_rows, m_first, n_k;   // m_first: query block of the first row
  float scale_log2;
  // index sets (SETS)
  const int32_t* v_idx;
  const int32_t* v_cnt;
  const int32_t* s_idx;
  const int32_t* s_cnt;
  int32_t v_budget, s_budget;
  // LISTED: the heads' bitmaps and the words of each (see build_list)
  const uint32_t* bm;
  int32_t bm_words;
};

constexpr int kShortBlocks = 512;   // key blocks of a call at most: flags of its diagonals in LDS
constexpr int kShortRange = 64;     // key-block distances of a range at most: one per lane
constexpr int kShortThreads = 512, kShortSets = kShortThreads / 256;
constexpr int short_stages(int d) { return d == 128 ? 2 : 4; }   // tiles of a set in LDS
template <int D>
constexpr int short_lds_bytes() {
  return kShortSets * (short_stages(D) * 2 * 64 * D * 2 + short_stages(D) * 4 * 64) + kShortThreads * 8 + 4 * kShortBlocks + 16;
}

// One piece per workgroup of eight waves, one workgroup per compute unit: two sets of four waves take the range's tiles in turn and
// fold their results at the end.  Layouts and masks are those of k_attention; left out is its pipeline.  Bound by trips to memory, by
// dependent instructions and by the instructions' own way to the compute unit, which meets each of them for the first time: of 15 us
// of k_attention for 1,024 rows of 4 heads of 64 at 4,096 keys, 3.8 passed before the first product (divisions, the search in the block
// list, arguments), 3.5 in the first two steps of eight (four bodies of code for a tile, 25 KB in all) and 1 in the last stores.  So: one
// body of code for every tile, no divisions, no block list (the diagonals of the tile's heads are collected in LDS from the selected
// offsets, 1.5 us, which spares a launch of 5.5), and as many tiles as the LDS holds on their way before the first is waited for.
// Two sets instead of two workgroups of four waves: half the partial results (512 ranges of 4 blocks 22.1 us with their fold, 256 of 8
// blocks 19.4, 256 of two sets 18.0), which go past the caches (0.4 to 1 us at the end of the launch).
// Measured (us, before and after): that chunk 45.8 -> 38.5; 70 rows of 28 heads of 128 at 2,048 keys 48.2 -> 42.5, 300 at 2,500 63 -> 55;
// dense, 2,000 rows of 4 heads at 2,000 keys 21.8 -> 16.7, 138 of 28 at 2,869 29.1 -> 24.5, 4 at 5,000 16.6 -> 14.9.
// LISTED: the diagonals come from the bitmaps of k_build_blocklist, where there are too many offsets to look through here (kShortOffsets).
template <int D, bool SETS, bool LISTED = false>
__global__ __launch_bounds__(kShortThreads) void k_attn_short(const ShortArgs a) {
  static_assert(SETS || !LISTED, "dense calls have no lists");
  constexpr int NQB = kAttnQBlocks, DCH = D / 8, DSTEPS = D / 16, DB = D / 32, TILE = 64 * D;
  constexpr int RPG = 512 / D, GPW = 64 / RPG / 4, R = 128 / D, NST = short_stages(D);
  static_assert(NQB == 2, "two query blocks per tile");
  extern __shared__ __attribute__((aligned(16))) unsigned char short_lds[];
  const int tid = threadIdx.x, lane = tid & 63, hh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), set = wave >> 2, wv = wave & 3;
  __bf16* const tiles = (__bf16*)short_lds + set * (NST * 2 * TILE);                       // [set][stage][K, V][TILE], as in k_attention
  uint8_t* const need_all = short_lds + kShortSets * NST * 2 * TILE * 2;                   // [set][stage][wave][64]
  uint8_t* const need_s = need_all + set * (NST * 4 * 64);
  float2* const ml_s = (float2*)(need_all + kShortSets * NST * 4 * 64);                    // [set][wave][64]
  uint8_t* const flags = (uint8_t*)(ml_s + kShortThreads);                                 // [diagonal][head of the tile]
  const uint32_t tiles_addr = __builtin_amdgcn_readfirstlane(lds_address(tiles));

  // consecutive pieces on one XCD: they share K/V rows
  const int piece = (blockIdx.x & 7) * a.each + (blockIdx.x >> 3);
  if (piece >= a.n_pieces) return;
  const int sp = short_quotient(piece, a.by_units), e = piece - sp * a.n_units;
  const int hs = short_quotient(e, a.by_qtiles), qt = a.n_qtiles - 1 - (e - hs * a.n_qtiles);
  const int g = short_quotient(hs, a.by_hs), h = g * a.group + (hs - g * a.n_hs) * a.pack;
  const int pack = a.pack, n_heads = (g + 1) * a.group - h < pack ? (g + 1) * a.group - h : pack;   // heads of the tile
  // this wave's rows (as in k_attention)
  int t = wv >> 1, th = 0, il0 = (wv & 1) << 5;
  if (pack > 1) {
    t = 0;
    th = pack == 4 ? wv : wv >> 1;
    il0 = a.row_pad + (pack == 4 ? 0 : il0);
  }
  const int il = il0 + (lane & 31) < 64 ? il0 + (lane & 31) : 63;
  const bool head_ok = th < n_heads;
  const int hw = head_ok ? h + th : h;
  const int row0 = qt * (64 * NQB), row = row0 + 64 * t + il0 + (lane & 31);
  const int m0 = a.m_first + qt * NQB, rows = a.row_pad + a.q_rows;
  const bool wave_valid = head_ok && row0 + 64 * t + il0 < rows;
  bf16x8 qreg[DSTEPS];
  {
    int rc = row - a.row_pad;
    rc = rc < 0 ? 0 : (rc < a.q_rows ? rc : a.q_rows - 1);
    const __bf16* const qp = a.q + (int64_t)rc * a.q_stride_tok + (int64_t)hw * a.q_stride_head + 8 * hh;
#pragma unroll
    for (int st = 0; st < DSTEPS; ++st) qreg[st] = *(const bf16x8*)(qp + 16 * st);
  }
  // ---- what is walked: a bit of `live` per key-block distance of the range, and tiles of 64 gathered columns ---------------
  const int n_blk = (a.n_k + 63) >> 6, shift = pack > 1 ? 2 : 0;
  const int cc_last = m0 + NQB - 1, per = short_quotient(cc_last + a.n_split, a.by_split), cc_lo = sp * per;
  const int cc_end = cc_lo + per - 1 < cc_last ? cc_lo + per - 1 : cc_last;
  int vcnt_l = 0;   // lane p: columns to gather of head h + p
  uint32_t heads_bits = (1u << n_heads) - 1u;
  if constexpr (SETS) {
    vcnt_l = a.v_cnt[h + (lane < n_heads ? lane : 0)];
    if constexpr (LISTED) {
      const uint32_t* const bm = a.bm + (int64_t)h * a.bm_words;
      for (int x = tid; x < n_blk << shift; x += kShortThreads) {
        const int p = pack > 1 ? x & 3 : 0, ad = x >> shift;
        flags[x] = p < n_heads ? (uint8_t)(bm[p * a.bm_words + (ad >> 5)] >> (ad & 31) & 1u) : 0;
      }
    } else {
      for (int x = tid; x < (kShortBlocks * 4 + 16) / 4; x += kShortThreads) ((uint32_t*)flags)[x] = 0u;
      __syncthreads();
      collect_flags<kShortThreads, 8>(flags, shift, 0, n_blk, kShortBlocks, a.s_idx + (int64_t)h * a.s_budget, a.s_cnt + h, a.s_budget, n_heads);
    }
    __syncthreads();
    // a head that has every diagonal has no column left to gather
    uint32_t missing = 0;
    for (int x0 = 0; x0 < n_blk; x0 += 64) {
      const int x = x0 + lane;
      uint32_t f = 0x01010101u;
      if (x < n_blk) f = pack > 1 ? ((const uint32_t*)flags)[x] : flags[x];
#pragma unroll
      for (int p = 0; p < 4; ++p) missing |= __ballot(!((f >> (8 * p)) & 255u)) ? 1u << p : 0u;
    }
    if (!((missing >> (lane & 3)) & 1u) || lane >= n_heads) vcnt_l = 0;
  }
  uint32_t mask_l = 0;   // lane x: who uses key block m0 + 1 - (cc_lo + x): bit t: query block t, or bit p: head h + p
  {
    const int cc = cc_lo + lane;
    if (cc <= cc_end) {
      if (pack > 1) {
        mask_l = cc >= 1 ? heads_bits : 0u;
        if (SETS && cc >= 1) mask_l &= ((const uint32_t*)flags)[cc - 1] * 0x01020408u >> 24;
      } else {
        mask_l = (cc >= 1 ? 1u : 0u) | (row0 + 64 < rows ? 2u : 0u);
        if (SETS) {
          if (cc >= 1 && !flags[cc - 1]) mask_l &= ~1u;
          if (cc >= n_blk || !flags[cc]) mask_l &= ~2u;
        }
      }
    }
  }
  // The range's tiles, key blocks first, go to the two sets of waves in turn.  `live`: the key blocks from the set's next one on.
  uint64_t live = __ballot(mask_l != 0u);
  const int n_live = __popcll(live);
  int n_tiles = n_live;
  if constexpr (SETS) {
    int n_vt = 0;
#pragma unroll
    for (int p = 0; p < 4; ++p) n_vt += (__builtin_amdgcn_readlane(vcnt_l, p) + 63) >> 6;
    n_tiles += n_vt > sp ? short_quotient(n_vt - sp + a.n_split - 1, a.by_split) : 0;
  }
  if (set) live &= live - 1;
  int at = set;   // the set's next tile
  const __bf16* const kbase = a.k + (int64_t)g * a.k_stride_head;
  const __bf16* const vbase = a.v + (int64_t)g * a.v_stride_head;

  // copies: as in k_attention
  const int lr = lane / DCH, lc = lane % DCH, r0 = wv * RPG + lr;
  const int kch = lc ^ ((r0 / R) % DCH), vch = lc ^ ((((r0 / R) & 3) << 2) & (DCH - 1));
  uint32_t koff[GPW], voff[GPW];
#pragma unroll
  for (int x = 0; x < GPW; ++x) {
    koff[x] = (uint32_t)((x * 4 * RPG + r0) * a.k_stride_tok * 2 + kch * 16);
    voff[x] = (uint32_t)((x * 4 * RPG + r0) * a.v_stride_tok * 2 + vch * 16);
  }
  // Finds the next tile and launches its copies into stage st.  What this wave is to do with it: bit 0 takes part, bit 1 the
  // diagonal of its query block, bit 2 thresholds in need_s; -1: there is none.
  auto issue = [&](int st) -> int {
    const int tile = at;
    at += kShortSets;
    if (tile >= n_tiles) return -1;
    const uint32_t kdst = tiles_addr + (uint32_t)(st * 2 * TILE * 2 + wv * 1024), vdst = kdst + TILE * 2;
    if (!SETS || tile < n_live) {
      const int x = __builtin_ctzll(live);
      live &= live - 1;
      live &= live - 1;
      const int mask = __builtin_amdgcn_readlane(mask_l, x), cc = cc_lo + x, j0 = (m0 + NQB - 1 - cc) * 64;
      if (__builtin_expect(j0 + 64 <= a.n_k, 1)) {
        const char* const kt = (const char*)(kbase + (int64_t)j0 * a.k_stride_tok);
        const char* const vt = (const char*)(vbase + (int64_t)j0 * a.v_stride_tok);
        if constexpr (GPW == 4) {
          dma16x4(kdst, kt, koff[0], koff[1], koff[2], koff[3], 4096);
          dma16x4(vdst, vt, voff[0], voff[1], voff[2], voff[3], 4096);
        } else {
          dma16x2(kdst, kt, koff[0], koff[1], 4096);
          dma16x2(vdst, vt, voff[0], voff[1], 4096);
        }
      } else {
#pragma unroll
        for (int y = 0; y < GPW; ++y) {
          int j = j0 + y * 4 * RPG + r0;
          j = j < a.n_k ? j : a.n_k - 1;
          dma16_lane_ptr(kdst + y * 4096, kbase + (int64_t)j * a.k_stride_tok + kch * 8);
        }
#pragma unroll
        for (int y = 0; y < GPW; ++y) {
          int j = j0 + y * 4 * RPG + r0;
          j = j < a.n_k ? j : a.n_k - 1;
          dma16_lane_ptr(vdst + y * 4096, vbase + (int64_t)j * a.v_stride_tok + vch * 8);
        }
      }
      const bool mine = (mask >> (pack > 1 ? th : t)) & 1;
      return (wave_valid && mine ? 1 : 0) | (cc - (NQB - 1) + t == 0 ? 2 : 0);
    }
    if constexpr (SETS) {
      int x = sp + (tile - n_live) * a.n_split, hd = 0, n_cols = 0;   // the heads' columns one after the other
      for (; hd < n_heads; ++hd) {
        n_cols = __builtin_amdgcn_readlane(vcnt_l, hd);
        const int nt = (n_cols + 63) >> 6;
        if (x < nt) break;
        x -= nt;
      }
      const int pos = 64 * x + lane;
      const int col = a.v_idx[(int64_t)(h + hd) * a.v_budget + (pos < n_cols ? pos : n_cols - 1)];
      const int ad = (m0 + t) - (col >> 6);
      const bool ok = pos < n_cols && ad >= 0 && (pack == 1 || hd == th) && !flags[(ad > 0 ? ad : 0) << shift | (pack > 1 ? th : 0)];
      need_s[(st * 4 + wv) * 64 + lane] = (uint8_t)(ok ? (ad == 0 ? col & 63 : 0) : 64);
#pragma unroll
      for (int y = 0; y < GPW; ++y)
        dma16_lane_ptr(kdst + y * 4096, kbase + (int64_t)__shfl(col, y * 4 * RPG + r0) * a.k_stride_tok + kch * 8);
#pragma unroll
      for (int y = 0; y < GPW; ++y)
        dma16_lane_ptr(vdst + y * 4096, vbase + (int64_t)__shfl(col, y * 4 * RPG + r0) * a.v_stride_tok + vch * 8);
      return (wave_valid && __ballot(ok) != 0 ? 1 : 0) | 4;
    }
    return -1;
  };

  // MFMA operands in LDS: as in k_attention
  int k_ofs[DSTEPS], v_ofs[DB];
  {
    const int y = hh ^ (((lane & 31) / R) % DCH);
#pragma unroll
    for (int st = 0; st < DSTEPS; ++st) k_ofs[st] = (lane & 31) * D + ((2 * st) ^ y) * 8;
    const int rl = ((lane & 15) >> 2) + 4 * hh, gl = (((rl / R) & 3) << 2) & (DCH - 1), ul = 2 * ((lane >> 4) & 1) + ((lane >> 1) & 1);
#pragma unroll
    for (int db = 0; db < DB; ++db) v_ofs[db] = rl * D + (((4 * db + ul) ^ gl) * 8) + 4 * (lane & 1);
  }
  f32x16 oacc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int x = 0; x < 16; ++x) oacc[db][x] = 0.f;
  float l_run = 0.f, m_o = -INFINITY;
  bool have_max = false;   // every row of this wave has a reference
  const float c = a.scale_log2;

  // `todo`: four bits per tile on its way, the oldest lowest
  uint32_t todo = 0;
  int n_todo = 0;   // tiles on their way
  bool more = true;
  auto fill = [&](int st) {
    const int w = issue(st);
    more = w >= 0;
    if (more) { todo |= (uint32_t)w << (4 * n_todo); ++n_todo; }
  };
#pragma clang loop unroll(disable)
  for (int st = 0; st < NST && more; ++st) fill(st);
  // Q is waited for here, with the first copies: at its first use it would be waited for in every turn of the loop, and all copies with it
#pragma unroll
  for (int k = 0; k < DSTEPS; ++k) asm volatile("" : "+v"(qreg[k]));
  int st = 0;
#pragma clang loop unroll(disable)
  for (int tile = 0; tile < n_tiles; tile += kShortSets) {
    // this tile's copies are done when at most those of the later ones are outstanding
    constexpr int CPT = 2 * GPW;
    if (n_todo <= 1) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    else if (NST == 2 || n_todo == 2) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(CPT) : "memory");
    else if (n_todo == 3) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(2 * CPT) : "memory");
    else asm volatile("s_waitcnt vmcnt(%0)" :: "n"(3 * CPT) : "memory");
    __syncthreads();   // (all waves' copies; and nobody reads the tile before this one any more)
    if (tile > 0 && more) fill((st + NST - 1) & (NST - 1));
    if (todo & 1u) {
      const __bf16* const kb = tiles + st * 2 * TILE;
      const __bf16* const vb = kb + TILE;
      f32x16 s[2];
#pragma unroll
      for (int jb = 0; jb < 2; ++jb) {
#pragma unroll
        for (int x = 0; x < 16; ++x) s[jb][x] = 0.f;
#pragma unroll
        for (int k = 0; k < DSTEPS; ++k)
          s[jb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8*)&kb[k_ofs[k] + 32 * jb * D], qreg[k], s[jb], 0, 0, 0);
      }
      if (todo & 6u) {   // element x of block jb is key 32 jb + 8 (x/4) + 4 hh + (x%4) of the tile
#pragma unroll
        for (int jb = 0; jb < 2; ++jb)
#pragma unroll
          for (int xq = 0; xq < 4; ++xq) {
            const int r = 32 * jb + 8 * xq + 4 * hh;
            uint32_t nd = (uint32_t)r * 0x01010101u + 0x03020100u;   // on the diagonal: key r from row r on
            if (SETS && (todo & 4u)) nd = *(const uint32_t*)&need_s[(st * 4 + wv) * 64 + r];
#pragma unroll
            for (int x = 0; x < 4; ++x)
              if (il < (int)((nd >> (8 * x)) & 255u)) s[jb][4 * xq + x] = -INFINITY;
          }
      }
      // probabilities relative to one reference per row: the largest score of its first tile, raised where a score outruns it by 2^64
      // (seen from the sum, as in k_attention)
      bf16x8 pp[4];
      float ps;
#pragma clang loop unroll(disable)
      for (bool exact = !have_max;; exact = true) {
        if (exact) {
          float mx = fmaxf(s[0][0], s[1][0]);
#pragma unroll
          for (int x = 1; x < 16; ++x) mx = fmaxf(fmaxf(mx, s[0][x]), s[1][x]);
          mx = fmaxf(mx, __shfl_xor(mx, 32)) * c;
          if (mx > m_o + 64.f || m_o == -INFINITY) mx = fmaxf(m_o, mx);
          else mx = m_o;
          const float alpha = mx == m_o ? 1.f : __builtin_amdgcn_exp2f(m_o - mx);
          m_o = mx;
          l_run *= alpha;
#pragma unroll
          for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int x = 0; x < 16; ++x) oacc[db][x] *= alpha;
          have_max = !__any(m_o == -INFINITY);
        }
        const float m_use = m_o == -INFINITY ? 0.f : m_o;
        ps = 0.f;
#pragma unroll
        for (int jb = 0; jb < 2; ++jb)
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            f32x8 pf;
#pragma unroll
            for (int x = 0; x < 8; ++x) pf[x] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[jb][8 * u + x], c, -m_use));
#pragma unroll
            for (int x = 0; x < 8; ++x) ps += pf[x];
            pp[2 * jb + u] = __builtin_convertvector(pf, bf16x8);
          }
        if (exact || !__any(!(ps < 1.8446744e19f))) break;
      }
      l_run += ps;
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int db = 0; db < DB; ++db) {
          typedef bf16x4 __attribute__((address_space(3))) * lds_b4;
          const __bf16* const vp = &vb[v_ofs[db] + 16 * u * D];
          const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_b4)(vp));
          const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_b4)(vp + 8 * D));
          const bf16x8 va = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
          oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pp[u], oacc[db], 0, 0, 0);
        }
    }
    todo >>= 4;
    --n_todo;
    st = (st + 1) & (NST - 1);
  }

  // ---- the two sets' results folded: each wave keeps half of its columns and hands the other half to its partner ----------
  constexpr int HB = DB / 2;
  const float l_own = l_run + __shfl_xor(l_run, 32);
  __syncthreads();   // (the tiles are done with)
  f32x4* const swap = (f32x4*)short_lds + wv * (4 * HB * 64) + lane;   // [set][wave][4 HB][64]
  constexpr int kSwap = 4 * 4 * HB * 64;
  f32x16 o[HB];
#pragma unroll
  for (int db = 0; db < HB; ++db)
#pragma unroll
    for (int vq = 0; vq < 4; ++vq) {
      f32x4 give;
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        give[x] = set ? oacc[db][4 * vq + x] : oacc[db + HB][4 * vq + x];
        o[db][4 * vq + x] = set ? oacc[db + HB][4 * vq + x] : oacc[db][4 * vq + x];
      }
      swap[set * kSwap + (4 * db + vq) * 64] = give;
    }
  ml_s[wave * 64 + lane] = make_float2(m_o, l_own);
  __syncthreads();
  const float2 other = ml_s[(wave ^ 4) * 64 + lane];
  const float M = fmaxf(m_o, other.x), M0 = M == -INFINITY ? 0.f : M;
  const float w_own = __builtin_amdgcn_exp2f(m_o - M0), w_other = __builtin_amdgcn_exp2f(other.x - M0);
  const float l_tot = l_own * w_own + other.y * w_other;
#pragma unroll
  for (int db = 0; db < HB; ++db)
#pragma unroll
    for (int vq = 0; vq < 4; ++vq) {
      const f32x4 got = swap[(1 - set) * kSwap + (4 * db + vq) * 64];
#pragma unroll
      for (int x = 0; x < 4; ++x) o[db][4 * vq + x] = o[db][4 * vq + x] * w_own + got[x] * w_other;
    }

  const int ro = row - a.row_pad, d0 = set * (D / 2) + 4 * hh;
  if (!head_ok || ro < 0 || ro >= a.q_rows) return;
  if (a.n_split > 1) {
    const int64_t pr = (int64_t)(sp * a.n_units + e) * kTileRows + 32 * wv + (lane & 31);
    float* const op = a.part_o + pr * D + d0;
#pragma unroll
    for (int db = 0; db < HB; ++db)
#pragma unroll
      for (int vq = 0; vq < 4; ++vq) {
        f32x4 o4;
#pragma unroll
        for (int x = 0; x < 4; ++x) o4[x] = o[db][4 * vq + x];
        __builtin_nontemporal_store(o4, (f32x4*)(op + 32 * db + 8 * vq));
      }
    if (set == 0 && hh == 0) *(float2*)(a.part_ml + 2 * pr) = make_float2(M, l_tot);
    return;
  }
  const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
  __bf16* const op = a.out + (int64_t)ro * a.o_stride_tok + (int64_t)hw * a.o_stride_head + d0;
#pragma unroll
  for (int db = 0; db < HB; ++db)
#pragma unroll
    for (int vq = 0; vq < 4; ++vq) {
      f32x4 o4;
#pragma unroll
      for (int x = 0; x < 4; ++x) o4[x] = o[db][4 * vq + x] * inv;
      *(bf16x4*)(op + 32 * db + 8 * vq) = __builtin_convertvector(o4, bf16x4);
    }
  if (a.lse && set == 0 && hh == 0) a.lse[(int64_t)hw * a.q_rows + ro] = l_tot > 0.f ? (M + __builtin_amdgcn_logf(l_tot)) * kLn2 : -INFINITY;
}

}  // namespace vs
