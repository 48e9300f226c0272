// The walk of single tokens over their shares of the keys (see vs_decode.hip for what it is and what bounds it): for the kernels of
// vs_decode.hip, and for the one that takes longer requests beside them (vs_attn.hip).
#pragma once
#include <type_traits>

#include "vs_common.h"

namespace vs {

constexpr int kDecThreads = 256;
constexpr int kDecWaves = kDecThreads / 64;
constexpr int kDecMinBlocks = 2;     // 64-key blocks per share at least, of all its KV heads: one 32-key chunk for every wave
constexpr int kDecListThreads = 1024;
constexpr int kDecListBytes = 128 << 10;   // a byte per diagonal and head in LDS at a time: 1M keys of up to 8 heads

// From this many 64-key blocks on (of all requests and KV heads) the waves of a workgroup take two neighbouring KV heads side by side, rows of
// 256 bytes each: 512 bytes in one place are read faster than 256 (a bare copy loop of this shape 6.2 TB/s against 5.5, with four
// heads no more), but a head has twice the partial results.  28 / 4 heads of 128, by themselves and side by side: one token at 12,000 keys
// 9.7 us and 12.0, 100,000 35.9 and 37.9, 140,000 (8,752 blocks) 50.1 and 50.6, 200,000 79.7 and 77.8, 1M 381 and 361; 40 / 8 heads, 60,000
// keys (7,504) 41.3 and 41.0, 70,000 (8,752) 49.8 and 48.3; tables of 30 tokens of up to 3,000 keys 25.3 and 25.5, 8 of 20,000 (10,016) 64.2
// and 62.9, 24 at 2K to 64K keys 223 and 212.
// Only where the rows of neighbouring heads lie next to each other: in caches of [KV heads][keys][128] 140,000 keys 48.1 -> 50.9, 1M 377 ->
// 387, 24 tokens 208 -> 212.  Heads of 64 (8 / 2, 300,000 keys): 36.5 -> 37.8, so not these.  With index sets the two walks drift
// apart: one token at 600,000 keys 209 -> 221, 64 of 16 heads per group at 60,000 917 -> 968; unless every head has every diagonal, and
// the walks are those of tokens without sets.  So: a single token without index sets by its length; a table whose bounds are as
// large by its requests' own lengths and sets, on the device (a request of 12,000 keys under a bound of 262,144 13.4 -> 15.2 by the bounds
// alone).
constexpr int64_t kDecSideBlocks = 8192;

struct DecodeArgs {
  vs_request one;         // the request of a call without a table (req null)
  const vs_request* req;
  int32_t n_req;
  int32_t n_q_heads, n_kv_heads, group;
  int64_t q_stride_head, k_stride_tok, k_stride_head, v_stride_tok, v_stride_head, o_stride_head;
  float scale_log2;
  int32_t v_budget, s_budget;
  int64_t max_n_k;
  // index sets: block-diagonal bitmap per (request, head), union list and its lengths per (request, KV head)
  uint32_t* bm;           // [n_req][Hq][words]
  uint2* ent;             // [n_req][Hkv][ent_stride] (diagonal, heads that have it)
  void* len;              // [n_req][Hkv] (entries, entries + tiles of 64 gathered columns, heads that have every diagonal): int4, or int2 in a
                          // workspace without room for the third, in which the columns of every head are gathered (template parameter Len)
  int32_t words, ent_stride;
  // shares: plan[0] = units in all (a unit: 64 keys of the KV heads that go side by side), plan[1] = shares, plan[2 + r] = units before request r; of one request without index sets the
  // host knows them (one_T units, one_n shares; 0: the device finds them)
  int64_t* plan;
  int64_t one_T, one_n;
  float* part_o;          // [share + (request, segment)][heads of a segment][D]
  float* part_ml;         // [share + (request, segment)][heads of a segment][2] (reference, sum)
  // (behind what a short token waits for)
  int32_t shares, side;   // most of them; KV heads side by side at most
};

__device__ __forceinline__ vs_request decode_request(const DecodeArgs& a, int r) {
  vs_request rq = a.one;
  if (a.req) {
    rq = a.req[r];
    rq.q = uniform64(rq.q); rq.k = uniform64(rq.k); rq.v = uniform64(rq.v); rq.out = uniform64(rq.out);
    rq.lse = uniform64(rq.lse); rq.v_idx = uniform64(rq.v_idx); rq.v_cnt = uniform64(rq.v_cnt);
    rq.s_idx = uniform64(rq.s_idx); rq.s_cnt = uniform64(rq.s_cnt);
    rq.q_start = uniform64(rq.q_start); rq.q_len = uniform64(rq.q_len);
  }
  return rq;
}
// a single token inside the stated bounds
__device__ __forceinline__ bool decode_takes(const DecodeArgs& a, const vs_request& rq) {
  if (!rq.q || !rq.k || !rq.v || !rq.out) return false;
  if (rq.q_len != 1 || rq.q_start < 0 || rq.q_start + 1 > a.max_n_k) return false;
  return rq.s_idx == nullptr || (rq.v_idx && rq.v_cnt && rq.s_cnt);
}
__device__ __forceinline__ int decode_blocks(const vs_request& rq) { return (int)((rq.q_start + kBlock) / kBlock); }
// units of request r with every KV head by itself; uneven: set where it has index sets that leave out a key
template <typename Len>
__device__ __forceinline__ int64_t decode_units(const DecodeArgs& a, int r, const vs_request& rq, bool& uneven) {
  if (!decode_takes(a, rq)) return 0;
  if (!rq.s_idx) return (int64_t)decode_blocks(rq) * a.n_kv_heads;
  int64_t n = 0;
  for (int g = 0; g < a.n_kv_heads; ++g) {
    const Len l = ((const Len*)a.len)[(int64_t)r * a.n_kv_heads + g];
    n += l.y;
    if constexpr (sizeof(Len) > 8) uneven |= (~(uint32_t)l.z & ((1u << a.group) - 1u)) != 0u;
  }
  return n;
}
// Those of all requests, and of request tid (mine).  Called by a whole workgroup.
template <typename Len>
__device__ __forceinline__ int64_t decode_total(const DecodeArgs& a, int64_t& mine, bool& uneven) {
  __shared__ int64_t sum_s[kDecWaves];
  __shared__ uint32_t uneven_s[kDecWaves];
  const int tid = threadIdx.x, wv = tid >> 6;
  uneven = false;
  auto of = [&](int r) -> int64_t {
    const vs_request rq = a.req ? a.req[r] : a.one;
    return decode_units<Len>(a, r, rq, uneven);
  };
  int64_t T = mine = 0;
  if (a.n_req == 1) return of(0);
  if (tid < a.n_req) T = mine = of(tid);
  for (int r = tid + kDecThreads; r < a.n_req; r += kDecThreads) T += of(r);
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) T += __shfl_xor((long long)T, d);
  const uint32_t any = __ballot(uneven) ? 1u : 0u;
  if ((tid & 63) == 0) { sum_s[wv] = T; uneven_s[wv] = any; }
  __syncthreads();
  T = 0;
  for (int w = 0; w < kDecWaves; ++w) { T += sum_s[w]; uneven |= uneven_s[w] != 0u; }
  return T;
}
// share w of n covers units [w T / n, (w + 1) T / n)
// (quotients of 64 bits, most of which fit 32: a fifth of the instructions)
__device__ __forceinline__ int64_t short_div(int64_t x, int64_t y) {
  return (uint64_t)(x | y) >> 32 ? x / y : (int64_t)((uint32_t)x / (uint32_t)y);
}
__device__ __forceinline__ int64_t share_start(int64_t w, int64_t n, int64_t T) { return short_div(w * T, n); }
__device__ __forceinline__ int64_t share_of(int64_t block, int64_t n, int64_t T) { return short_div((block + 1) * n - 1, T); }

template <int D>
constexpr int decode_lds_bytes() { return kDecWaves * 2 * 2 * 32 * D * 2; }

// one 1 KiB copy global -> LDS: lane L's 16 bytes land at lds_addr + 16 L
__device__ __forceinline__ void dec_dma(uint32_t lds_addr, const void* sbase, uint32_t off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :: "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(off), "s"(uniform64(sbase)) : "memory");
}
__device__ __forceinline__ void dec_dma_lane(uint32_t lds_addr, const void* ptr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
               :: "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(ptr) : "memory");
}

// ONE: a single request without index sets (no table, no lists; the host has counted its units).  In a kernel of its own, because a short
// token waits for its instructions: 5,003 keys 11.40 us where the kernel of all requests had 3,756 instructions, 11.55 with
// 3,770 of them, 9.9 with the 1,893 of this one.
// T: units of all requests, mine0: of request tid with every KV head by itself.  SIDE > 1: nobody has index sets that leave out a key.
// LEAN: half the LDS, one buffer per wave: the next chunk's keys are fetched while this one's values are waited for, and its values while its
// scores are.  For the kernel that has longer requests beside the tokens; by itself, 24 tokens at 2K to 64K keys 212.1 us and 211.9, 8 sparse
// ones at 256K 780 and 755, but two dense and two sparse ones 387 and 424.  n_wg: workgroups that have shares.
template <int D, int SIDE, bool ONE, typename Len, bool LEAN = false>
__device__ __forceinline__ void decode_body(const DecodeArgs& a, int64_t T, int64_t mine0, int n_wg) {
  constexpr int DCH = D / 8;         // 16-byte pieces per row
  constexpr int KS = D / 32;         // MFMA steps of K Q^T
  constexpr int DB = D / 16;         // 16-row blocks of O^T
  constexpr int RPG = 512 / D;       // rows per 1 KiB copy
  constexpr int NC = 32 / RPG;       // copies of 32 rows
  constexpr int R = 128 / D;         // rows per 256 bytes of LDS
  constexpr int TILE = 32 * D;
  // LDS: per wave [2 buffers][K tile, V tile].  Row r of a tile starts at r D; its 16-byte piece c lies in slot c ^ f(r) for
  // K (16 rows of one piece in one read) and c ^ g(r) for V (4 rows x 2 pieces in one transposing read): no bank conflicts.
  extern __shared__ __attribute__((aligned(16))) unsigned char dec_lds[];
  __shared__ int64_t scan_s[kDecWaves];
  __shared__ int64_t at_s[2];
  __shared__ float ml_s[kDecWaves][16][2];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15, g4 = lane >> 4;   // MFMA column (query head of the group) and k-group / row-group of the lane
  __bf16* const buf = (__bf16*)dec_lds + wv * ((LEAN ? 2 : 4) * TILE);
  const uint32_t buf_addr = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)(const __attribute__((address_space(3))) char*)buf);

  // ---- this workgroup's share ------------------------------------------------------------------
  auto units_of = [&](int r) -> int64_t {
    const vs_request rq = a.req ? a.req[r] : a.one;
    bool unused;
    return decode_units<Len>(a, r, rq, unused) / SIDE;
  };
  int64_t first = 0;
  constexpr int min_units = kDecMinBlocks / SIDE;
  int64_t n_share = (T + min_units - 1) / min_units;
  if (n_share > n_wg) n_share = n_wg;
  if (!ONE && blockIdx.x == 0 && tid == 0) { a.plan[0] = T; a.plan[1] = n_share | (int64_t)SIDE << 32; }
  if (ONE) {
    if (blockIdx.x >= n_share) return;
  } else if (a.n_req == 1) {
    if (blockIdx.x == 0 && tid == 0) a.plan[2] = 0;
    if (blockIdx.x >= n_share) return;
  } else if (blockIdx.x != 0 && blockIdx.x >= n_share) {
    return;
  }
  const int64_t u_begin = n_share ? share_start(blockIdx.x, n_share, T) : 0, u_end = n_share ? share_start(blockIdx.x + 1, n_share, T) : 0;
  int r = 0;
  first = u_begin;
  if (!ONE && a.n_req > 1) {
    int64_t before = 0;
    for (int rb = 0; rb < a.n_req; rb += kDecThreads) {
      const int64_t mine = rb == 0 ? mine0 / SIDE : (rb + tid < a.n_req ? units_of(rb + tid) : 0);
      int64_t inc = mine;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const int64_t y = __shfl_up((long long)inc, d);
        if (lane >= d) inc += y;
      }
      __syncthreads();
      if (lane == 63) scan_s[wv] = inc;
      __syncthreads();
      for (int w = 0; w < kDecWaves; ++w) {
        if (w < wv) inc += scan_s[w];
      }
      inc += before;
      for (int w = 0; w < kDecWaves; ++w) before += scan_s[w];
      if (blockIdx.x == 0 && rb + tid < a.n_req) a.plan[2 + rb + tid] = inc - mine;
      if (inc - mine <= u_begin && u_begin < inc) { at_s[0] = rb + tid; at_s[1] = u_begin - (inc - mine); }
      if (blockIdx.x != 0 && before > u_begin) break;   // (uniform; the first workgroup writes all of the plan)
    }
    if (n_share == 0) return;
    __syncthreads();
    r = __builtin_amdgcn_readfirstlane((int)at_s[0]);
    first = uniform64(at_s[1]);
  }

  // ---- lane constants ---------------------------------------------------------------------------
  const int lr = lane / DCH, lc = lane % DCH;   // row inside a copy, and the slot there
  // the piece of its row that the lane fetches (the slot, swizzled): copy e of a tile holds rows e RPG + lr
  const int vpc = lc ^ ((((lr / R) & 3) << 2) & (DCH - 1));
  auto k_piece = [&](int e) -> int { return lc ^ (((e * RPG + lr) / R) % DCH); };
  // this wave's KV head in a segment, its place among the waves of that head, and their number
  const int sub = wv % SIDE, w_of = wv / SIDE;
  constexpr int w_n = kDecWaves / SIDE;
  int64_t left = u_end - u_begin;
  int sg = 0;
  bool fresh = true;   // the request's fields are to be read
  vs_request rq;
  int64_t blk = first;
  while (left > 0) {
    if (ONE) {
      rq = a.one;
    } else if (fresh) {
      rq = decode_request(a, r);
      sg = 0;
      if (!decode_takes(a, rq)) { ++r; continue; }
      fresh = false;
    }
    bool with_sets = !ONE && SIDE == 1 && rq.s_idx != nullptr;
    const int64_t n_k = rq.q_start + 1;
    const int g = sg * SIDE + sub;   // this wave's KV head
    int n_ent = decode_blocks(rq), seg_len = n_ent, full = 0;
    if (with_sets) {
      const Len l2 = ((const Len*)a.len)[(int64_t)r * a.n_kv_heads + g];
      n_ent = __builtin_amdgcn_readfirstlane(l2.x);
      seg_len = __builtin_amdgcn_readfirstlane(l2.y);
      if constexpr (sizeof(Len) > 8) {
        // (a KV head all of whose heads have every diagonal is walked as without sets: 19 tokens of up to 4,419 keys, 40 heads, 48.8 us ->
        // 46.4, 16 of up to 8,000, half of them without sets, 52.2 -> 49.5)
        full = l2.z;
        with_sets = __builtin_amdgcn_readfirstlane(~full & ((1 << a.group) - 1)) != 0;
      }
    }
    if (blk >= seg_len) {   // the share starts in a later segment of this request
      blk -= seg_len;
      if (++sg == a.n_kv_heads / SIDE && !ONE) { ++r; fresh = true; }
      continue;
    }
    const int64_t take64 = seg_len - blk < left ? seg_len - blk : left;
    const bool whole = blk == 0 && take64 == seg_len;
    const int b0 = (int)blk, b1 = (int)(blk + take64);
    const int h0 = g * a.group;

    // The piece, with and without index sets: a request without them does not wait for the instructions of the others.
    const auto walk = [&](auto sets) __attribute__((always_inline)) {
    constexpr bool sparse = decltype(sets)::value;
    // ---- Q^T operand: lane (head h0 + col, k-group g4); columns beyond the group repeat its first head and are not stored (zeros in
    // their place had to wait for the loads before the first copies went out: 0.7 us) --------------------
    bf16x8 qreg[KS];
    {
      const __bf16* qp = (const __bf16*)rq.q + (int64_t)(h0 + (col < a.group ? col : 0)) * a.q_stride_head + 8 * g4;
#pragma unroll
      for (int st = 0; st < KS; ++st) qreg[st] = *(const bf16x8*)(qp + 32 * st);
    }
    f32x4 oacc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) oacc[db] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m_run = -INFINITY, l_run = 0.f;

    const __bf16* const kb = (const __bf16*)rq.k + (int64_t)g * a.k_stride_head;
    const __bf16* const vb = (const __bf16*)rq.v + (int64_t)g * a.v_stride_head;
    const uint2* const ents = a.ent + ((int64_t)r * a.n_kv_heads + g) * a.ent_stride;
    const int m_blk = (int)(rq.q_start / kBlock);
    const int pos_in_block = (int)(rq.q_start % kBlock);

    // chunk c: 32 keys.  Dense: keys 32 c ...; with index sets entry c / 2 of the union list, then the columns.
    int c = 2 * b0 + w_of;
    int c_end = 2 * b1;
    if (!sparse && c_end > (int)((n_k + 31) / 32)) c_end = (int)((n_k + 31) / 32);
    // columns to gather of head h0 + lane: none where it has every diagonal
    const int cnt_cache = sparse && !(full >> (lane & 15) & 1) ? rq.v_cnt[h0 + (lane < a.group ? lane : 0)] : 0;
    uint2 ecache = make_uint2(0u, 0u);
    int ebase = -64;
    // what the next chunk is: its live keys (bit k: key k) and live rows (bit q), both uniform
    struct Chunk { uint32_t keys, rows; };
    // (what: its keys, its values, or both)
    constexpr int kKeys = 1, kValues = 2;
    auto issue = [&](int ci, int b, auto part) __attribute__((always_inline)) -> Chunk {
      constexpr int what = decltype(part)::value;
      Chunk ch;
      ch.keys = ~0u;
      ch.rows = 0xFFFFu;
      const uint32_t kd = buf_addr + (uint32_t)(b * 2 * TILE * 2), vd = kd + TILE * 2;
      int64_t j0 = (int64_t)32 * ci;
      bool columns = false;
      if (sparse) {
        const int e = ci >> 1;
        if (e < n_ent) {
          if (e >= ebase + 64) {
            ebase = e;
            const int x = ebase + lane;
            ecache = ents[x < n_ent ? x : n_ent - 1];
          }
          const int diag = __builtin_amdgcn_readlane(ecache.x, e - ebase);
          ch.rows = __builtin_amdgcn_readlane(ecache.y, e - ebase);
          j0 = (int64_t)(m_blk - diag) * kBlock + 32 * (ci & 1);
        } else {
          columns = true;
        }
      }
      if (!columns) {
        const int64_t over = j0 + 32 - n_k;   // keys of the chunk behind the token
        if (over > 0) ch.keys = over >= 32 ? 0u : ~0u >> over;
        if (over <= 0) {
          const char* kt = (const char*)(kb + j0 * a.k_stride_tok);
          const char* vt = (const char*)(vb + j0 * a.v_stride_tok);
#pragma unroll
          for (int e = 0; e < (what & kKeys ? NC : 0); ++e)
            dec_dma(kd + e * 1024, kt + (int64_t)e * RPG * a.k_stride_tok * 2,
                    (uint32_t)(lr * a.k_stride_tok * 2 + k_piece(e) * 16));
#pragma unroll
          for (int e = 0; e < (what & kValues ? NC : 0); ++e)
            dec_dma(vd + e * 1024, vt + (int64_t)e * RPG * a.v_stride_tok * 2,
                    (uint32_t)(lr * a.v_stride_tok * 2 + vpc * 16));
        } else {
#pragma unroll
          for (int e = 0; e < NC; ++e) {
            int64_t j = j0 + e * RPG + lr;
            j = j < n_k ? j : n_k - 1;
            if (what & kKeys) dec_dma_lane(kd + e * 1024, kb + j * a.k_stride_tok + k_piece(e) * 8);
            if (what & kValues) dec_dma_lane(vd + e * 1024, vb + j * a.v_stride_tok + vpc * 8);
          }
        }
      } else {
        // columns: 64 per unit, the heads of the group one after the other
        int u = (ci >> 1) - n_ent, jh = 0, vc = 0;
        for (; jh < a.group; ++jh) {
          vc = __builtin_amdgcn_readlane(cnt_cache, jh);
          const int nt = (vc + 63) >> 6;
          if (u < nt) break;
          u -= nt;
        }
        if (jh == a.group) { jh = 0; u = 0; vc = 0; }   // a group without any line: one unit without live keys
        const int32_t* vi = rq.v_idx + (int64_t)(h0 + jh) * a.v_budget;
        const uint32_t* bm = a.bm + ((int64_t)r * a.n_q_heads + h0 + jh) * a.words;
        const int p0 = 64 * u + 32 * (ci & 1);
        // (clamped to the list, so that the loads go out together)
        auto column = [&](int k) -> int { return vi[p0 + k < vc ? p0 + k : vc - 1]; };
        int j = 0, jr[NC];
#pragma unroll
        for (int e = 0; e < NC; ++e) jr[e] = 0;
        const int k = lane & 31;
        if (vc > 0) {
          j = column(k);
#pragma unroll
          for (int e = 0; e < NC; ++e) jr[e] = column(e * RPG + lr);
        }
        // a column counts if it is not behind the token and not on a computed diagonal of its own head
        const int ad = m_blk - (j >> 6);
        bool ok = p0 + k < vc && ad >= 0 && !(ad == 0 && (j & 63) > pos_in_block);
        ok = ok && !((bm[ad >= 0 ? ad >> 5 : 0] >> (ad & 31)) & 1u);
        ch.keys = (uint32_t)__ballot(ok);
        ch.rows = 1u << jh;
#pragma unroll
        for (int e = 0; e < NC; ++e) {
          if (what & kKeys) dec_dma_lane(kd + e * 1024, kb + (int64_t)jr[e] * a.k_stride_tok + k_piece(e) * 8);
          if (what & kValues) dec_dma_lane(vd + e * 1024, vb + (int64_t)jr[e] * a.v_stride_tok + vpc * 8);
        }
      }
      return ch;
    };

    Chunk cur;
    cur.keys = cur.rows = 0u;
    const auto keys_part = std::integral_constant<int, kKeys>{};
    const auto values_part = std::integral_constant<int, kValues>{};
    const auto both_parts = std::integral_constant<int, kKeys | kValues>{};
    if (LEAN) {
      if (c < c_end) { cur = issue(c, 0, keys_part); issue(c, 0, values_part); }
    } else if (c < c_end) {
      cur = issue(c, 0, both_parts);
    }
    // Q is waited for here, with the first copies: at its first use it would be waited for in every turn of the loop, and the next
    // chunk's copies, which the compiler does not see, with it
#pragma unroll
    for (int st = 0; st < KS; ++st) asm volatile("" : "+v"(qreg[st]));
    for (int b = 0; c < c_end; c += w_n, b ^= LEAN ? 0 : 1) {
      Chunk nxt;
      nxt.keys = nxt.rows = 0u;
      if (LEAN) {   // (its values are outstanding)
        if constexpr (NC == 8) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
      } else if (c + w_n < c_end) {
        nxt = issue(c + w_n, b ^ 1, both_parts);
        // this chunk's copies are done when at most the next chunk's are outstanding
        if constexpr (NC == 8) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
      } else {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      }
      const __bf16* const Kt = buf + b * 2 * TILE;
      const __bf16* const Vt = Kt + TILE;
      // S^T: two blocks of 16 keys; lane (head col, keys 16 jb + 4 g4 + 0..3)
      f32x4 s[2];
#pragma unroll
      for (int jb = 0; jb < 2; ++jb) {
        s[jb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int st = 0; st < KS; ++st) {
          const int row = 16 * jb + col;
          const bf16x8 ka = *(const bf16x8*)&Kt[row * D + (((4 * st + g4) ^ ((row / R) % DCH)) * 8)];
          s[jb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka, qreg[st], s[jb], 0, 0, 0);
        }
      }
      if constexpr (LEAN) {
        // (the keys are read: the products above have waited for them)
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (c + w_n < c_end) nxt = issue(c + w_n, 0, keys_part);
      }
      if (cur.keys != ~0u || cur.rows != 0xFFFFu) {   // uniform
        const bool row_ok = (cur.rows >> col) & 1u;
#pragma unroll
        for (int jb = 0; jb < 2; ++jb)
#pragma unroll
          for (int x = 0; x < 4; ++x)
            if (!row_ok || !((cur.keys >> (16 * jb + 4 * g4 + x)) & 1u)) s[jb][x] = -INFINITY;
      }
      // The probabilities are 2^(score - m_run) with a reference that moves only when a score outruns it by 2^64 (or on the
      // first live keys of a row): a true maximum of the moment, so nothing overflows and the sums stay exact.
      float mx = s[0][0];
#pragma unroll
      for (int x = 1; x < 4; ++x) mx = fmaxf(mx, s[0][x]);
#pragma unroll
      for (int x = 0; x < 4; ++x) mx = fmaxf(mx, s[1][x]);
      mx *= a.scale_log2;
      if (__any(mx > m_run + 64.f || (m_run == -INFINITY && mx != -INFINITY))) {
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float m_new = fmaxf(m_run, mx);
        const float alpha = m_new == m_run ? 1.f : __builtin_amdgcn_exp2f(m_run - m_new);
        m_run = m_new;
        l_run *= alpha;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int x = 0; x < 4; ++x) oacc[db][x] *= alpha;
      }
      const float m_use = m_run == -INFINITY ? 0.f : m_run;
      bf16x8 p;   // contraction slots of the lane: keys 4 g4 + 0..3 and 16 + 4 g4 + 0..3
      f32x8 pf;
#pragma unroll
      for (int x = 0; x < 8; ++x) {
        pf[x] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[x >> 2][x & 3], a.scale_log2, -m_use));
        l_run += pf[x];
      }
      p = __builtin_convertvector(pf, bf16x8);
      if constexpr (LEAN) {   // the next chunk's keys are outstanding
        if (c + w_n >= c_end) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        else if constexpr (NC == 8) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
      }
      // O^T += V^T P^T; V^T through the transposing read: in each 16-lane group lane L supplies V[J0 + L / 4][D0 + 4 (L % 4) ...]
      // and receives V[J0 .. J0 + 3][D0 + L]
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        typedef bf16x4 __attribute__((address_space(3))) * lds_b4;
        const int row = 4 * g4 + (col >> 2), piece = 2 * db + ((col >> 1) & 1);
        const int slot = piece ^ ((((row / R) & 3) << 2) & (DCH - 1));
        const __bf16* const vp = &Vt[row * D + slot * 8 + 4 * (col & 1)];
        const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_b4)(vp));
        const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_b4)(vp + 16 * D));
        const bf16x8 va = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        oacc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, p, oacc[db], 0, 0, 0);
      }
      cur = nxt;
      // (the reads of this buffer are done: the products above have waited for them)
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if constexpr (LEAN)
        if (c + w_n < c_end) issue(c + w_n, 0, values_part);
    }

    // ---- fold the waves and store -----------------------------------------------------------------
    l_run += __shfl_xor(l_run, 16);
    l_run += __shfl_xor(l_run, 32);
    if (g4 == 0) { ml_s[wv][col][0] = m_run; ml_s[wv][col][1] = l_run; }
    __syncthreads();   // (all tiles are done with as well: the LDS takes the accumulators)
    float M = ml_s[sub][col][0];
#pragma unroll
    for (int w = 1; w < w_n; ++w) M = fmaxf(M, ml_s[sub + SIDE * w][col][0]);
    const float own = m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run - M);
    float* const fold = (float*)dec_lds;   // [wave][16 heads][D + 4]
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      f32x4 o4;
#pragma unroll
      for (int x = 0; x < 4; ++x) o4[x] = oacc[db][x] * own;
      *(f32x4*)&fold[(wv * 16 + col) * (D + 4) + 16 * db + 4 * g4] = o4;
    }
    __syncthreads();
    const int64_t slot = ((int64_t)blockIdx.x + (int64_t)r * (a.n_kv_heads / SIDE) + sg) * SIDE * a.group;
    for (int x = tid; x < SIDE * a.group * (D / 4); x += kDecThreads) {
      // query head qs of the segment: row q of the waves w0, w0 + side, ...
      const int qs = x / (D / 4), w0 = SIDE > 1 ? qs / a.group : 0, q = qs - w0 * a.group, d = 4 * (x % (D / 4));
      f32x4 o = *(const f32x4*)&fold[(w0 * 16 + q) * (D + 4) + d];
      float Mq = ml_s[w0][q][0];
#pragma unroll
      for (int w = 1; w < w_n; ++w) {
        const f32x4 y = *(const f32x4*)&fold[((w0 + SIDE * w) * 16 + q) * (D + 4) + d];
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] += y[e];
        Mq = fmaxf(Mq, ml_s[w0 + SIDE * w][q][0]);
      }
      float L = 0.f;
      if (Mq != -INFINITY)
#pragma unroll
        for (int w = 0; w < w_n; ++w) {
          const float* const ml = ml_s[w0 + SIDE * w][q];
          L += ml[0] == -INFINITY ? 0.f : ml[1] * __builtin_amdgcn_exp2f(ml[0] - Mq);
        }
      if (whole) {
        const float inv = L > 0.f ? 1.0f / L : 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] *= inv;
        const int h = sg * SIDE * a.group + qs;
        *(bf16x4*)((__bf16*)rq.out + (int64_t)h * a.o_stride_head + d) = __builtin_convertvector(o, bf16x4);
        if (rq.lse && d == 0) rq.lse[h] = L > 0.f ? (Mq + __builtin_amdgcn_logf(L)) * kLn2 : -INFINITY;
      } else {
        *(f32x4*)&a.part_o[(slot + qs) * D + d] = o;
        if (d == 0) {
          a.part_ml[(slot + qs) * 2] = Mq;
          a.part_ml[(slot + qs) * 2 + 1] = L;
        }
      }
    }
    };
    // (in this order: 16 tokens of up to 4,000 keys 21.9 us the other way round, 21.2 so)
    if (__builtin_expect(!with_sets, 1)) walk(std::false_type{});
    else walk(std::true_type{});
    __syncthreads();   // the LDS is reused by the next piece
    left -= take64;
    blk = 0;
    if (++sg == a.n_kv_heads / SIDE && !ONE) { ++r; fresh = true; }
  }
}

// out = sum_s O_s 2^(m_s - M) / sum_s l_s 2^(m_s - M) over the shares that a (request, segment of KV heads) lies in; one workgroup for
// query head h of request r, shares folded in a fixed order (run-to-run identical): wave w takes every NW-th share, then
// the waves are added in order.  Bound by latency: the partial results of 8 NW shares are all on their way before the references
// are compared (four waves, and the references first: one token at 5,003 keys 14.1 us with its two launches, 12.1 so and with the
// shares counted on the host).  Eight waves where a KV head lies in more than 32 shares, else four: 60 tokens of 40 heads, a share or
// two each, 71 us with four, 75 with eight.
// SIDE: KV heads side by side; 0: as the walk's plan says.
template <int D, int NW, int SIDE, typename Len = int4>
__device__ __forceinline__ void decode_fold(const DecodeArgs& a, int h, int r) {
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const vs_request rq = decode_request(a, r);
  if (!decode_takes(a, rq)) return;
  const int64_t T = a.one_T ? a.one_T : a.plan[0], planned = a.one_T ? 0 : a.plan[1], n = a.one_T ? a.one_n : planned & 0xFFFFFFFF;
  const int side = SIDE ? SIDE : __builtin_amdgcn_readfirstlane((int)(planned >> 32));
  const int rows = side * a.group, sg = h / rows, q = h - sg * rows;
  int64_t from = a.one_T ? 0 : a.plan[2 + r];
  int seg_len = decode_blocks(rq);
  if (rq.s_idx && (SIDE == 1 || side == 1)) {
    const Len* const len = (const Len*)a.len + (int64_t)r * a.n_kv_heads;
    for (int x = 0; x < sg; ++x) from += len[x].y;
    seg_len = len[sg].y;
  } else {
    from += (int64_t)sg * seg_len;
  }
  const int s0 = (int)share_of(from, n, T), s1 = (int)share_of(from + seg_len - 1, n, T);
  if (s0 == s1) return;   // finished by its one share
  const int64_t row0 = ((int64_t)s0 + (int64_t)r * (a.n_kv_heads / side) + sg) * rows + q;   // row of share s: row0 + (s - s0) rows
  const int cnt = s1 - s0 + 1;
  constexpr int E = D / 64, U = 8;
  float acc[E], L = 0.f, o[U][E], w[U], l[U];
  auto fetch = [&](int sb) {   // shares sb, sb + NW, ...
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int s = sb + NW * u < cnt ? sb + NW * u : cnt - 1;
      const int64_t row = row0 + (int64_t)s * rows;
      const float2 ml = *(const float2*)(a.part_ml + 2 * row);
      w[u] = ml.x;
      l[u] = ml.y;
#pragma unroll
      for (int e = 0; e < E; ++e) o[u][e] = a.part_o[row * D + 64 * e + lane];
    }
  };
  float M = lane < cnt ? a.part_ml[2 * (row0 + (int64_t)lane * rows)] : -INFINITY;
  fetch(wv);
  for (int s = 64 + lane; s < cnt; s += 64) M = fmaxf(M, a.part_ml[2 * (row0 + (int64_t)s * rows)]);
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) M = fmaxf(M, __shfl_xor(M, d));
#pragma unroll
  for (int e = 0; e < E; ++e) acc[e] = 0.f;
  if (M != -INFINITY) {
    for (int sb = wv; sb < cnt; sb += NW * U) {
      if (sb != wv) fetch(sb);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (sb + NW * u >= cnt || w[u] == -INFINITY) continue;
        const float x = __builtin_amdgcn_exp2f(w[u] - M);
        L += l[u] * x;
#pragma unroll
        for (int e = 0; e < E; ++e) acc[e] += o[u][e] * x;
      }
    }
  }
  __shared__ float acc_s[NW][D], l_s[NW];
#pragma unroll
  for (int e = 0; e < E; ++e) acc_s[wv][64 * e + lane] = acc[e];
  if (lane == 0) l_s[wv] = L;
  __syncthreads();
  if (tid >= D) return;
  float out = acc_s[0][tid];
  L = l_s[0];
#pragma unroll
  for (int x = 1; x < NW; ++x) { out += acc_s[x][tid]; L += l_s[x]; }
  ((__bf16*)rq.out)[(int64_t)h * a.o_stride_head + tid] = (__bf16)(L > 0.f ? out / L : 0.f);
  if (rq.lse && tid == 0) rq.lse[h] = L > 0.f ? (M + __builtin_amdgcn_logf(L)) * kLn2 : -INFINITY;
}

// Bitmaps of the heads of a KV group and the union of their block lists, one workgroup per (KV head, request), for single
// tokens with index sets.  Diagonals are collected as bytes in LDS (see collect_flags), 8 or 16 heads side by side, a window at a time;
// every wave has consecutive groups of 64 diagonals, a lane per diagonal.
// flags: BYTES + 16 of LDS.
template <typename Len, int BYTES>
__device__ __forceinline__ void decode_lists(const DecodeArgs& a, int g, int r, uint8_t* flags) {
  constexpr int NW = kDecListThreads / 64;
  __shared__ uint32_t wsum[NW], missing_s;   // (a bit per head that lacks a diagonal)
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int G = a.group;
  const vs_request rq = decode_request(a, r);
  if (!decode_takes(a, rq) || !rq.s_idx) return;
  const int n_blk = decode_blocks(rq), n_words = (n_blk + 31) / 32, shift = G > 8 ? 4 : 3, win = BYTES >> shift;
  uint2* const E = a.ent + ((int64_t)r * a.n_kv_heads + g) * a.ent_stride;
  uint32_t* const B = a.bm + ((int64_t)r * a.n_q_heads + (int64_t)g * G) * a.words;
  const int64_t h0 = (int64_t)g * G;
  uint32_t running = 0, missing = 0;
  if (tid == 0) missing_s = 0u;
  for (int b0 = 0; b0 < n_blk; b0 += win) {
    const int n = n_blk - b0 < win ? n_blk - b0 : win, n_grp = (n + 63) >> 6;
    for (int x = tid; x < n_grp << (2 + shift); x += kDecListThreads) ((u32x4*)flags)[x] = u32x4{0u, 0u, 0u, 0u};
    __syncthreads();
    collect_flags<kDecListThreads, 16>(flags, shift, b0, n, win, rq.s_idx + h0 * a.s_budget, rq.s_cnt + h0, a.s_budget, G);
    __syncthreads();
    // heads that have diagonal b0 + x: bytes of 0 and 1 to bits
    auto heads_of = [&](int x) -> uint32_t {
      auto four = [](uint32_t v) -> uint32_t { return (v * 0x01020408u >> 24) & 15u; };
      if (shift == 3) {
        const uint2 v = ((const uint2*)flags)[x];
        return four(v.x) | four(v.y) << 4;
      }
      const u32x4 v = ((const u32x4*)flags)[x];
      return four(v[0]) | four(v[1]) << 4 | four(v[2]) << 8 | four(v[3]) << 12;
    };
    const int each = (n_grp + NW - 1) / NW, g0 = wv * each, g1 = g0 + each < n_grp ? g0 + each : n_grp;
    uint32_t c = 0;
    for (int grp = g0; grp < g1; ++grp) {
      const uint32_t heads = heads_of(64 * grp + lane);
      c += __popcll(__ballot(heads != 0u));
      if (b0 + 64 * grp + lane < n_blk) missing |= ~heads;
      // the bitmaps: lanes 2 j, 2 j + 1 write the words of head j
      uint64_t bits = 0;
      for (int j = 0; j < G; ++j) {
        const uint64_t b = __ballot((heads >> j) & 1u);
        bits = (lane >> 1) == j ? b : bits;
      }
      const int w = (b0 >> 5) + 2 * grp + (lane & 1);
      if (lane < 2 * G && w < n_words) B[(int64_t)(lane >> 1) * a.words + w] = (uint32_t)(bits >> (32 * (lane & 1)));
    }
    if (lane == 0) wsum[wv] = c;
    uint32_t lacks = 0;
    for (int j = 0; j < G; ++j) lacks |= __ballot((missing >> j) & 1u) ? 1u << j : 0u;
    if (lane == 0) atomicOr(&missing_s, lacks);
    __syncthreads();
    uint32_t pos = running;
    for (int x = 0; x < NW; ++x) {
      if (x < wv) pos += wsum[x];
      running += wsum[x];
    }
    for (int grp = g0; grp < g1; ++grp) {
      const uint32_t heads = heads_of(64 * grp + lane);
      const uint64_t m = __ballot(heads != 0u);
      if (heads)
        E[pos + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] =
            make_uint2((uint32_t)(b0 + 64 * grp + lane), heads);
      pos += __popcll(m);
    }
    __syncthreads();   // wsum and flags are rewritten by the next window
  }
  if (tid == 0) {
    int tiles = 0;
    for (int j = 0; j < G; ++j) tiles += sizeof(Len) == 8 || missing_s >> j & 1u ? (rq.v_cnt[g * G + j] + 63) >> 6 : 0;
    const int units = (int)running + tiles;   // (at least one: a token without any key gets its 0 / -inf too)
    Len l = {};
    l.x = (int)running;
    l.y = units > 0 ? units : 1;
    if constexpr (sizeof(Len) > 8) l.z = (int)~missing_s;
    ((Len*)a.len)[(int64_t)r * a.n_kv_heads + g] = l;
  }
}

// The arguments of a table whose longer requests another kernel takes (vs_decode.hip)
DecodeArgs decode_args(const vs_params& p, const vs_request* req, int n_req, void* ws);

}  // namespace vs
