// Block-sparse / dense causal online-softmax attention for gfx950 (CDNA4), bf16 MFMA with
// fp32 accumulation.  One kernel serves both the vertical-slash sparse path and the dense
// fallback: it walks a per-head bitmap of block diagonals (dense = all ones) and then the
// gathered vertical columns.
//
// What is computed (section 5.2, MInference paragraph: attention only on the selected
// critical tokens; softmax_lse as in the "Sparsity refinement" paragraph): row i at position
// p attends key j <= p iff j is a selected column or floor(p/64) - floor(j/64) is a computed
// block diagonal.
//
// Layout of the work
//  * workgroup = NQB query blocks of 64 rows (2 waves each, a wave owns 32 rows) of one head.
//    Key block n = m0 - c is staged once in LDS and used by query block t iff diagonal
//    c + t is computed, so adjacent diagonals share their K/V fetch.
//  * S^T = K Q^T with v_mfma_f32_32x32x16_bf16: the accumulator then holds, per lane, one
//    query and 16 keys, so the row maximum / sum need one cross-lane step, and P^T is already
//    the B operand of the second MFMA (O^T = V^T P^T) -- P never goes through LDS.
//  * V stays row-major in LDS and is read with the transposing LDS load (ds_read_b64_tr_b16)
//    as the A operand of the PV contraction, which runs over keys.
//  * K/V tiles go from global memory straight into LDS (global_load_lds_dwordx4, no staging
//    registers), double-buffered: the copy of tile t+1 runs under the MFMA work of tile t,
//    one barrier per tile.  Rows are unpadded; 16-byte chunks are XOR-swizzled instead.
//  * the exponentials use one fixed reference per row (the maximum of the row's first tile;
//    an exact path with the true maximum is kept for masked tiles, first tiles and an
//    overflow guard), so the steady state has no running-maximum update.  The V^T P^T product
//    of a tile runs one step behind its K Q^T product, in one hand-interleaved instruction
//    stream with the exponentials, operands three LDS reads ahead.
//  * the tile walk reads a per-head list of (key block, query-block mask) entries through
//    a 64-entry lane cache and lives entirely in scalar registers.
//  * persistent launch: two workgroups per compute unit in eight groups (one per XCD).  Where keys
//    are many (heads of 128 from 256K keys on, and some calls of few heads of 64) a group works on consecutive query tiles of one
//    head per round and keeps its members within a few sync segments of keys, so that K/V blocks
//    are shared through the L2.  Which group takes which round is decided on the device from the
//    lengths of the block lists.  Elsewhere the pieces of the launch wait in one queue per XCD.
//  * template parameters: DCA (three rotations of the queries, chosen per (query, key)
//    pattern; section 5.1) and SPLIT (short chunks, and what whole rounds leave of longer ones:
//    the key walk cut into pieces that wait in queues, partial results folded by k_attn_combine;
//    heads of a KV group share a tile where the rows leave half of it empty).  The plain kernel is
//    its own instantiation, and so is the one whose ranges may follow the lists' lengths (k_attention_own).
//    k_attention_paced keeps pace over the whole units and goes on with the pieces of the rest in the
//    same launch; k_attention_mixed walks a batch's longer requests beside its single tokens.
//  * calls of one round whose pieces walk few key blocks have a kernel of their own (vs_attn_short.h).
#include <atomic>
#include <cstddef>
#include <mutex>

#include "vs_common.h"
#include "vs_decode_walk.h"

namespace vs {

// Where the pieces of request r of a batch begin among those of all requests, the ranges each of its units is cut into
// (0: the request is skipped) and, from bit 16 on, the heads of a tile, its first slot of partial results, and its first unit among those that are cut.  Written by
// k_build_blocklist; entry n_req holds the numbers of pieces, slots and cut units.
struct BatchPlan {
  int32_t first, split_pack, slot, cut;
};
// The last request whose first piece (cut unit) is piece (cut unit) x or one before it: the one that has it, because a request
// without any begins where the next one does.  64 probes at a time: one step for 64 requests, two for 4,096.
template <int32_t BatchPlan::*Field>
__device__ __forceinline__ int batch_find(const BatchPlan* plan, int n_req, int x) {
  const int lane = threadIdx.x & 63;
  int r = 0, left = n_req;
  while (left > 1) {
    const int step = (left + 63) >> 6, y = lane * step;
    const int n = __popcll(__ballot(y < left && plan[r + (y < left ? y : 0)].*Field <= x));   // (the first one always)
    r += (n - 1) * step;
    left = left - (n - 1) * step < step ? left - (n - 1) * step : step;
  }
  return __builtin_amdgcn_readfirstlane(r);
}

// A piece of an uneven cut (own_cut): its unit, range and number of ranges, slot of partial results, and the key-block distances
// [cc_lo, cc_hi] that it walks.
struct OwnPiece {
  int32_t unit, sp, n_sp, slot, cc_lo, cc_hi, pad[2];
};

struct AttnArgs {
  const __bf16* q;
  // Dual Chunk Attention (template parameter DCA): the chunk's queries rotated for the
  // successive-chunk and the inter-chunk pattern (q is the intra-chunk one; same strides),
  // chunk length and local window in 64-key blocks
  const __bf16* q_succ;
  const __bf16* q_inter;
  int32_t dca_cblk, dca_wblk;
  // Key split (template parameter SPLIT) for launches of few units (a unit: a query tile of one head, or of `pack`
  // heads).  The first n_whole units are walked whole; the walk of each of the others is cut into n_split ranges of
  // key-block distances, and the pieces write their unnormalised results (relative to their own references), which
  // k_attn_combine folds: part_o [n_split][n_units - n_whole][rows of a tile][D], part_ml the same with
  // (reference, sum).  With n_split = 1 every unit is whole.  See unit_of for the order of the units.
  // (first_piece: the whole units in front of it are another launch's.)
  int32_t n_split, n_units, n_whole, first_piece;
  float* part_o;
  float* part_ml;
  int32_t first_slot;   // BATCH: of the request's partial results
  // SPLIT: query heads of one KV group that share a tile (1, 2 or 4).  Chunks whose rows lie in one query block leave
  // half of a tile's waves (three quarters: at most 32 rows) without rows; these waves take further heads.
  // n_hs: tiles per KV group = ceil(group / pack)
  int32_t pack, n_hs;
  // SPLIT: eight queues of pieces, one per XCD (kQueueStride words apart; zero at the start of the launch)
  uint32_t* queue;
  const __bf16* k;
  const __bf16* v;
  __bf16* out;
  float* lse;
  int64_t q_stride_tok, q_stride_head, k_stride_tok, k_stride_head;
  int64_t v_stride_tok, v_stride_head, o_stride_tok, o_stride_head;
  const uint32_t* bm_a;  // block-diagonal bitmap per head
  const uint32_t* ent;   // key-block entry list per head (see BlockList); null (SPLIT only): every block, no list is made
  int64_t bm_stride;     // words per head, 0 = one bitmap shared by all heads (dense)
  int32_t bm_words;      // words of one bitmap row; its last two words: see build_list
  int64_t ent_stride;    // entries per head, 0 = one list shared by all heads (dense)
  int64_t ent_len;       // entries of one list (sentinel padding included)
  const int32_t* v_idx;  // null: no vertical phase (how many columns of a head: see build_list)
  // OWN: pieces of an uneven cut, 0: the even one stays.  (Here, because the fields behind it are read a tenth of a microsecond faster at
  // these places: without it, index sets of 700 rows of 8 heads at 9,000 keys 40.1 us -> 40.7, 20 rows of 4 at 2,000 12.15 -> 12.36.)
  int32_t* own_n;
  int32_t v_budget;
  int32_t n_q_heads, n_kv_heads, group;
  int32_t n_qtiles;
  // q_start is rounded down to a multiple of 64 and q_len grown by the same row_pad rows, so that
  // query blocks stay aligned to absolute positions; the first row_pad rows of the launch are
  // padding (nothing is loaded or stored for them).  q_rows is the caller's q_len.
  int64_t q_len, q_start;
  int32_t row_pad;
  int64_t q_rows;
  int64_t n_k;  // keys visible to the chunk
  // Dense attention of a single token with grouped queries that the decode kernel does not take (DCA, more than
  // 16 heads per group, a token in a small batch of longer requests): the G query heads of a KV group are the rows of one tile (so K and V are read once per
  // group, not once per head); all rows then stand at the same position, pos_in_block keys into the diagonal block.
  int32_t same_pos, pos_in_block;
  float scale_log2;  // softmax_scale * log2(e)
  // persistent launch: n_wg workgroups, workgroup b is member b / 8 of group b % 8 (the groups
  // follow the round-robin of workgroups over the 8 XCDs); in round r group g works on
  // group-round k = 8 r + g, one query tile per member.  The top n_full * members tiles of
  // every head go first, as (chunk of `members` consecutive tiles, head) rounds, latest chunks
  // first; the n_rem tiles per head that are left are packed, head after head, into the rounds
  // that follow, so that only the very last round can have idle members.
  int32_t n_wg, members, n_full, n_rem;
  // pace keeping: arrive[g][s] counts the members of group g that are done with key blocks
  // [s * sync_blocks, (s + 1) * sync_blocks) over all rounds so far; sync_blocks = 1 << sync_shift
  int32_t sync_blocks, sync_shift, n_sync;
  uint32_t* arrive;
  // sched[g][r]: the group-round that group g works on in its r-th round, -1 = none left
  // (written by k_attn_schedule from the lengths of the heads' block lists; n_gr entries per group)
  const int32_t* sched;
  int32_t n_gr;
  // Several requests in one launch (template parameter BATCH, always with SPLIT): the pieces of all
  // requests, one request after the other; a request's pointers, position and length come
  // from req[r], its piece and slot counts from plan[r], and replace the fields above (batch_view).
  // bm_a / ent hold one list per (request, head).  Requests beyond max_q_len / max_n_k
  // (the bounds the workspace was sized for) are skipped.
  const vs_request* req;
  const BatchPlan* plan;
  int32_t n_req, head_dim;
  int64_t max_q_len, max_n_k;
  int32_t skip_single;   // BATCH: single tokens are the decode kernel's
  // OWN: slots of partial results for an uneven cut of the cut units (own_cut), and what k_attn_pieces leaves of it beside the number of
  // pieces: the pieces, ranges and first slot of every cut unit.  (Behind everything else: a short kernel waits for each line of
  // its arguments.)
  int32_t own_slots;
  OwnPiece* own_pieces;
  int2* own_units;
};

constexpr int kMaxSplit = 128;                     // ranges of a unit at most
constexpr int kMinSteps = 2, kMinBatchSteps = 8;   // steps of a range at least, in a call and in a batch
constexpr double kPieceSteps = 4.0;                // what a piece costs beside its walk, in steps
constexpr double kAloneRate = 0.88;                // a step of a workgroup that has its compute unit to itself, against one of two
constexpr double kFoldSteps = 0.022;               // folding a row's piece, in steps
constexpr int kBatchSlots = 512, kShortSteps = 64;  // a batch of fewer steps per slot is cut into one piece per slot: 2 requests
                                                    // of 64 rows at 46K keys 134 us -> 107
constexpr int kMaxPieces = 2048, kBatchPieces = 1536;   // pieces with partial results: a call's, a batch's
constexpr int kMaxQueueUnits = 4096;               // beyond it only what whole rounds leave over is cut (see cut_rest); ranges that are asked for are made
constexpr int64_t kMaxAskedUnits = 1 << 23;        // all the same (128 M pieces of 33 KB and more: no workspace holds them)
constexpr int kPaceBlocks = 4096;                  // key blocks from which whole units of heads of 128 keep pace (see launch_attention)
constexpr int kShortList = 1024;                   // steps of a walk below which (by the budgets) heads of 64 over many keys are cut less finely
constexpr int kRun = 64;                           // workgroup slots of an XCD: members of a pace-keeping group
constexpr int kQueueStride = 16;                   // words between two queue counters: a cache line each
constexpr int kListBits = 28;                      // of a bitmap row's word that holds the length of the list (see build_list)
constexpr uint32_t kListMask = (1u << kListBits) - 1u;
constexpr int kTileRows = 64 * kAttnQBlocks;       // rows of a query tile, of a slot of partial results

// Query heads that share a tile, from the rows of the launch and the first one's place in its 64-block.  Rows of one query
// block fill two of a tile's four waves (two SIMDs of four), at most 32 rows one; with the heads side by side all four work,
// and K and V are copied once for them.  28 query / 4 KV heads: 64 rows at 1M keys 1,384 us -> 815 (with the finer cut and the
// order of the pieces, see attn_cut), 4 rows at 50K keys 100 -> 46, 22 requests of up to 64 rows and 38K keys (40 heads)
// 921 -> 308.  Heads without a group (or a second query block) have nothing to share.  Gathered columns are not shared: a tile
// walks those of its heads one after the other, so it takes as many heads as leave their steps (two per 64 columns, which
// take the masked path) below the n_blk of the key blocks; ranges are counted by these.  With four heads whatever the columns, 28 heads: 2 rows at 1,000
// keys, as many columns, 120 us, 55 so; at 300 keys 77 and 42.
__host__ __device__ __forceinline__ int heads_per_tile(int64_t rows, int row_pad, int group, int64_t n_blk, int64_t columns) {
  if (kAttnQBlocks != 2 || group < 2 || row_pad + rows > kBlock) return 1;
  int n = rows <= 32 && group > 2 ? 4 : 2;
  while (n > 1 && 2 * n * ((columns + 63) / 64) > n_blk) n >>= 1;
  return n;
}

// What a request of a batch is to the launch: false for one outside the stated bounds or with a null pointer, which is
// skipped (nothing of it is read or written).
struct BatchShape {
  bool dense, same_pos;
  int32_t row_pad, pack, n_hs, n_qtiles, n_units;
};
// (whatever the columns: the plan counts their steps and cuts the tiles that have many)
__device__ __forceinline__ int batch_pack(const vs_request& rq, int group) {
  return heads_per_tile(rq.q_len, (int)(rq.q_start % kBlock), group, 1, 0);
}
__device__ __forceinline__ bool batch_shape(const vs_request& rq, int group, int n_kv_heads, int64_t max_q_len, int64_t max_n_k,
                                            bool skip_single, int pack, BatchShape& b) {
  if (!rq.q || !rq.k || !rq.v || !rq.out) return false;
  if (rq.q_len < 1 || rq.q_len > max_q_len || rq.q_start < 0 || rq.q_start + rq.q_len > max_n_k) return false;
  if (skip_single && rq.q_len == 1) return false;
  b.dense = rq.s_idx == nullptr;
  if (!b.dense && (!rq.v_idx || !rq.v_cnt || !rq.s_cnt)) return false;
  b.row_pad = (int32_t)(rq.q_start % kBlock);
  // attention of one token: the G heads of a KV group are the rows of one tile
  b.same_pos = rq.q_len == 1 && group > 1 && b.dense;
  b.pack = b.same_pos ? 1 : pack;
  b.n_hs = b.same_pos ? 1 : (group + b.pack - 1) / b.pack;
  const int64_t rows = b.same_pos ? group : b.row_pad + rq.q_len;
  b.n_qtiles = (int32_t)((rows + kTileRows - 1) / kTileRows);
  b.n_units = b.n_qtiles * n_kv_heads * b.n_hs;
  return true;
}

// The arguments as request r of a batch sees them.  False: the request is skipped.
__device__ __forceinline__ bool batch_view(const AttnArgs& a0, int r, AttnArgs& a) {
  vs_request rq = a0.req[r];   // the same address in every lane: the fields are uniform
  rq.q = uniform64(rq.q); rq.k = uniform64(rq.k); rq.v = uniform64(rq.v); rq.out = uniform64(rq.out);
  rq.lse = uniform64(rq.lse); rq.v_idx = uniform64(rq.v_idx); rq.v_cnt = uniform64(rq.v_cnt);
  rq.s_idx = uniform64(rq.s_idx); rq.s_cnt = uniform64(rq.s_cnt);
  rq.q_start = uniform64(rq.q_start); rq.q_len = uniform64(rq.q_len);
  const BatchPlan pl = a0.plan[r];
  const int split_pack = __builtin_amdgcn_readfirstlane(pl.split_pack);
  BatchShape b;
  if (!batch_shape(rq, a0.group, a0.n_kv_heads, a0.max_q_len, a0.max_n_k, a0.skip_single, split_pack >> 16, b)) return false;
  a.q = (const __bf16*)rq.q; a.k = (const __bf16*)rq.k; a.v = (const __bf16*)rq.v;
  a.out = (__bf16*)rq.out; a.lse = rq.lse;
  a.v_idx = b.dense ? nullptr : rq.v_idx;
  a.row_pad = b.row_pad;
  a.q_start = rq.q_start - a.row_pad;
  a.q_len = rq.q_len + a.row_pad;
  a.q_rows = rq.q_len;
  a.n_k = rq.q_start + rq.q_len;
  a.bm_a = a0.bm_a + (int64_t)r * a0.n_q_heads * a0.bm_stride;
  a.ent = a0.ent + (int64_t)r * a0.n_q_heads * a0.ent_stride;
  a.n_split = split_pack & 0xFFFF;
  if (b.dense) a.ent_stride = a.bm_stride = 0;   // one list, the first head's
  a.first_slot = __builtin_amdgcn_readfirstlane(pl.slot);
  a.pack = b.pack; a.n_hs = b.n_hs; a.n_qtiles = b.n_qtiles; a.n_units = b.n_units;
  a.n_whole = a.n_split == 1 ? b.n_units : 0;
  a.first_piece = 0;
  if (b.same_pos) {
    a.q_stride_tok = a0.q_stride_head; a.q_stride_head = (int64_t)a0.group * a0.q_stride_head;
    a.o_stride_tok = a0.o_stride_head; a.o_stride_head = (int64_t)a0.group * a0.o_stride_head;
    a.n_q_heads = a0.n_kv_heads; a.group = 1;
    a.same_pos = 1; a.pos_in_block = a.row_pad;
    a.row_pad = 0; a.q_len = a0.group; a.q_rows = a0.group;
  }
  return true;
}

// Unit e of a launch: KV group, first head and query tile.  Consecutive units share K/V rows: runs of kRun consecutive
// tiles of one head, the latest first, heads inside (the order in which the pace-keeping kernel takes its rounds), then
// what is left of the heads, one after the other.
__device__ __forceinline__ void unit_of(const AttnArgs& a, int e, int& g, int& h0, int& qt) {
  const int n_run = a.n_qtiles / kRun, n_rem = a.n_qtiles - n_run * kRun, slots = a.n_q_heads / a.group * a.n_hs;
  int hs;
  if (e < n_run * kRun * slots) {
    const int run = e / kRun, c = run / slots;
    hs = run - c * slots;
    qt = n_rem + (n_run - c) * kRun - 1 - (e - run * kRun);
  } else {
    e -= n_run * kRun * slots;
    hs = e / n_rem;
    qt = n_rem - 1 - (e - hs * n_rem);
  }
  g = hs / a.n_hs;
  h0 = g * a.group + (hs - g * a.n_hs) * a.pack;
}

// Cut units that follow one another in that order and belong to one list (a run, or what runs leave of a head): segments.
__host__ __device__ __forceinline__ int cut_segment_of(int e, int n_qtiles, int lists) {
  const int n_run = n_qtiles / kRun, n_rem = n_qtiles - n_run * kRun, lead = n_run * lists * kRun;
  return e < lead ? e / kRun : n_run * lists + (n_rem ? (e - lead) / n_rem : 0);
}
// segment x of the cut units: its list, first unit and units (0: behind the last one)
__device__ __forceinline__ void cut_segment(const AttnArgs& a, int x, int& list, int& e0, int& cnt) {
  const int lists = a.n_q_heads / a.group * a.n_hs, n_run = a.n_qtiles / kRun, n_rem = a.n_qtiles - n_run * kRun;
  const int runs = n_run * lists, s = cut_segment_of(a.n_whole, a.n_qtiles, lists) + x;
  list = s < runs ? s % lists : s - runs;
  e0 = s < runs ? s * kRun : runs * kRun + (s - runs) * n_rem;
  const int end = e0 < a.n_units ? e0 + (s < runs ? kRun : n_rem) : e0;
  e0 = e0 < a.n_whole ? a.n_whole : e0;
  cnt = end - e0;
}
// Ranges by the lists' own lengths.  Heads differ in them (scattered slashes by a tenth, clustered ones by a factor of two), and with one
// range count for all a launch of one round waits for the heads with the longest lists.  Lane x of the calling wave (all lanes) gets the
// ranges n of each of the cnt units of segment x and the segment's first slot of partial results; pieces, most: of all, most ranges
// of a unit.  n follows the length, for up to four rounds of 512 pieces; most = 0 where the even cut is to stay: lists equally long
// (so that with everything selected the results are those of dense calls), or a gain of less than 5 % by this count.
// 28 heads, clustered slashes, even -> uneven: 200 rows at 500K keys 1,588 us -> 1,080, 333 at 100K 656 -> 518, 1,000 at 300K 2,584 ->
// 1,958, 2,000 at 150K 2,811 -> 2,390; lists that differ by a tenth or less within 1 %.  Finding the ranges takes 5 us where
// the even cut stays, up to 11 where it does not, and 2.5 to 4.5 of a call's time where that gains nothing: 1,000 rows of 8 heads at 200K keys 336 -> 338, the attention alone 95.8 -> 98.2, of 100 rows of 4
// heads at 300K with offsets side by side 30.2 -> 34.5; against 275 -> 203 for 300 clustered rows of those at 900K, 300 -> 206 for 2,000
// of 8 heads at 200K.  (A gain of four steps asked for on top of the 5 % keeps the even cut in these, too: equal distances hide from the
// count that all entries lie in one range.)
constexpr int kOwnRounds = 4, kOwnSegments = 64;
__device__ __forceinline__ void own_cut(const AttnArgs& a, int lane, int& n, int& cnt, int& slot, int& pieces, int& most) {
  int list, e0;
  cut_segment(a, lane, list, e0, cnt);
  int len = 0;
  if (cnt > 0) {
    const int h0 = list / a.n_hs * a.group + list % a.n_hs * a.pack;
    const uint32_t* const tail = a.bm_a + (int64_t)h0 * a.bm_stride + a.bm_words - 2;
    len = (int)(tail[0] & kListMask) + 2 * (int)((tail[1] + 63) >> 6);   // (a gathered tile takes as long as two: the masked path)
    len = len > 1 ? len : 1;
  }
  int mx = len, mn = cnt > 0 ? len : 1 << 30;
  float total = (float)cnt * (float)len;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int x = __shfl_xor(mx, d), y = __shfl_xor(mn, d);
    mx = x > mx ? x : mx;
    mn = y < mn ? y : mn;
    total += __shfl_xor(total, d);
  }
  n = 0;
  pieces = most = slot = 0;
  if (mx == mn) return;
  const int n_cut = a.n_units - a.n_whole;
  // a piece's time beside its walk, writing and folding it: as attn_cut counts them
  auto beside = [](int p) -> float {
    return (float)kPieceSteps * (float)((p + kBatchSlots - 1) / kBatchSlots) + 8.f * (float)p / (float)kBatchSlots;
  };
  const float share = total / (float)kBatchSlots;
  float best = 0.95f * ((float)mx / (float)a.n_split + beside(n_cut * a.n_split));
  for (int r = 1; r <= kOwnRounds && r * kBatchSlots <= a.own_slots; ++r) {
    if (r * kBatchSlots <= n_cut) continue;
    // (one each and the rest by length, rounded down: never more than the slots)
    int m = 1 + (int)((float)len * ((float)(r * kBatchSlots - n_cut) / total));
    m = m > kMaxSplit ? kMaxSplit : m;
    m = m > 1 + len / 8 ? 1 + len / 8 : m;
    float longest = cnt > 0 ? (float)len / (float)m : 0.f;
    int p = cnt * m;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      longest = fmaxf(longest, __shfl_xor(longest, d));
      p += __shfl_xor(p, d);
    }
    const float c = fminf((float)((p + kBatchSlots - 1) / kBatchSlots) * longest, share + 0.5f * longest) + beside(p);
    if (fmaxf(c, longest) < best) { best = fmaxf(c, longest); n = m; }
  }
  if (__builtin_amdgcn_readfirstlane(n) == 0) { n = 0; return; }
  most = cnt > 0 ? n : 1;
  int end = cnt * n;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int x = __shfl_xor(most, d), y = __shfl_up(end, d);
    most = x > most ? x : most;
    end += lane >= d ? y : 0;
  }
  slot = end - cnt * n;
  pieces = __builtin_amdgcn_readlane(end, 63);
  most = __builtin_amdgcn_readfirstlane(most);
}
__device__ __forceinline__ bool bm_test(const uint32_t* bm, int i) {
  return (bm[i >> 5] >> (i & 31)) & 1u;
}

// LDS bytes of one workgroup: K and V tiles (unpadded, chunk-swizzled), double-buffered, the
// gathered column indices of a vertical tile, and per-wave mask thresholds.
template <int D>
constexpr int attn_lds_bytes() { return 4 * 64 * D * 2 + 4 * 64 * 4 + 4 * kAttnQBlocks * 64; }

// Direct global -> LDS copy, 16 bytes per lane: lane L's bytes land at lds_addr + 16 L
// (lds_addr is wave-uniform and goes through M0).  Completion is tracked by vmcnt.
// N such copies from one scalar base with per-copy lane offsets; the LDS destinations are
// lds_addr, lds_addr + step, ...  (M0 is read when a copy issues, so it can move on at once;
// a write to M0 needs one wait state before the copy that uses it.)
// (lds_addr, sbase and step are the same in every lane; where the compiler cannot see that, the
// values are moved into scalar registers here: the instructions take them from there)
__device__ __forceinline__ void dma16x4(uint32_t lds_addr, const void* sbase, uint32_t o0, uint32_t o1,
                                        uint32_t o2, uint32_t o3, uint32_t step) {
  lds_addr = __builtin_amdgcn_readfirstlane(lds_addr);
  step = __builtin_amdgcn_readfirstlane(step);
  sbase = uniform64(sbase);
  asm volatile(
      "s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %5\n\t"
      "s_add_u32 m0, m0, %6\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %5\n\t"
      "s_add_u32 m0, m0, %6\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %3, %5\n\t"
      "s_add_u32 m0, m0, %6\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %4, %5"
      :: "s"(lds_addr), "v"(o0), "v"(o1), "v"(o2), "v"(o3), "s"(sbase), "s"(step) : "memory", "scc");
}
__device__ __forceinline__ void dma16x2(uint32_t lds_addr, const void* sbase, uint32_t o0, uint32_t o1,
                                        uint32_t step) {
  lds_addr = __builtin_amdgcn_readfirstlane(lds_addr);
  step = __builtin_amdgcn_readfirstlane(step);
  sbase = uniform64(sbase);
  asm volatile(
      "s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %3\n\t"
      "s_add_u32 m0, m0, %4\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3"
      :: "s"(lds_addr), "v"(o0), "v"(o1), "s"(sbase), "s"(step) : "memory", "scc");
}
__device__ __forceinline__ void dma16_lane_ptr(uint32_t lds_addr, const void* ptr) {
  lds_addr = __builtin_amdgcn_readfirstlane(lds_addr);
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
               :: "s"(lds_addr), "v"(ptr) : "memory");
}
__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return (uint32_t)(size_t)(const __attribute__((address_space(3))) char*)p;
}

}  // namespace vs
#include "vs_attn_short.h"
namespace vs {

constexpr int kHeadShift = 27;   // vertical tile of packed heads: (head << kHeadShift) | tile of 64 columns (a head has at most 2^25)
// OWN: the cut units may have ranges by the lengths of their lists.  (Instantiations of their own: with this decided in the others, dense
// calls of 20 to 500 rows took 0.15 to 0.5 us of 12 to 24 more.)
// TAIL: behind a pace-keeping walk in the same kernel, whose workgroups end at different times: the first piece, too, is taken from a
// queue.  args_at: where the arguments lie among the kernel's.
template <int D, int NQB, bool DCA, bool SPLIT, bool BATCH, bool OWN, bool TAIL = false>
__device__ __forceinline__ void attention_body(const AttnArgs& a0, const size_t args_at = 0) {
  static_assert(!BATCH || (SPLIT && !DCA), "several requests per launch ride on the key-split kernel");
  static_assert(!OWN || (SPLIT && !BATCH), "uneven ranges are those of cut units of a single call");
  static_assert(!TAIL || SPLIT, "pieces");
  constexpr int DCH = D / 8;           // 16-byte chunks per row
  constexpr int DSTEPS = D / 16;       // MFMA k-steps of QK^T
  constexpr int DB = D / 32;           // 32-row blocks of O^T
  constexpr int TILE = 64 * D;         // elements of one K or V tile in LDS (rows unpadded)
  constexpr int RPG = 512 / D;         // rows in one 1 KiB group (= one wave-wide copy)
  constexpr int NG = 64 / RPG;         // groups per tile
  constexpr int GPW = NG / (2 * NQB);  // groups per wave
  constexpr int R = 128 / D;           // rows per 256 bytes of LDS
  static_assert(NG % (2 * NQB) == 0, "tile must divide over the waves");
  // LDS layout.  Row r of a tile starts at r * D elements; its 16-byte chunk c is stored in
  // slot c ^ f(r) for K and c ^ g(r) for V, which spreads the MFMA operand reads over all
  // banks without padding (the copy engine writes 1 KiB contiguously per instruction):
  //   f(r) = (r / R) % DCH                      16 consecutive keys of one d-chunk (K reads)
  //   g(r) = (((r / R) & 3) << 2) & (DCH - 1)   4 keys x 4 d-chunks (transposing V reads)

  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  __bf16* const Ks = (__bf16*)smem_raw;               // [2][TILE]
  __bf16* const Vs = Ks + 2 * TILE;                   // [2][TILE]
  int32_t* const vidx_s = (int32_t*)(Vs + 2 * TILE);  // [4][64]
  uint8_t* const need_s = (uint8_t*)(vidx_s + 4 * 64);  // [waves][64], private to each wave
  static_assert(2 * (2 * NQB) * 64 <= 4 * kAttnQBlocks * 64, "need_s and dcak_s share the bytes after vidx_s");
  uint8_t* const dcak_s = need_s + 2 * NQB * 64;        // [waves][64], DCA pattern code of a tile's keys
  const uint32_t ks_addr = lds_address(Ks), vs_addr = lds_address(Vs);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave index, known uniform
  const int hh = lane >> 5;

  // The arguments, for what comes after the walk: read from memory there.  (Read through a0 they are loaded once, in front of the
  // rounds, and sit in vector registers' lanes during the walk: there are about a hundred scalar registers for twice as many values.)
  auto late_args = [&]() -> const AttnArgs& {
    uint64_t p = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr() + args_at;
    asm volatile("" : "+s"(p));
    return *(const AttnArgs*)(const __attribute__((address_space(4))) AttnArgs*)p;
  };
  // ---- persistent workgroup: one (query tile, head) per round ------------------------------
  // The `members` workgroups of a group take consecutive query tiles of ONE head, so they walk
  // the same entry list, shifted by two key blocks per tile, at the same pace; the arrive
  // counters below keep the group inside a window of a few sync segments, small enough for
  // the XCD's L2, so that a K/V block is fetched from memory once per group and round.
  // Waiting is bounded and only shapes the timing: results never depend on it.
  //
  // SPLIT: no pace keeping.  The pieces lie in eight queues, `members` consecutive ones in each in turn; a workgroup
  // takes the piece of its own place, then from its XCD's queue (the pieces there share K/V rows in the L2), then from
  // the queue with the most left.  The results do not depend on who takes what.
  const int grp = blockIdx.x & 7, member = blockIdx.x >> 3;
  const int n_full_gr = a0.n_full * a0.n_q_heads;   // full rounds: latest chunks first, heads inside
  const int n_gr = a0.n_gr;
  uint32_t* const arr = a0.arrive + (int64_t)grp * a0.n_sync;
  const int s_glob_top = (int)((a0.n_k - 1) / 64) >> a0.sync_shift;  // highest sync segment of the chunk
  int n_pieces = 0;
  if constexpr (BATCH) n_pieces = __builtin_amdgcn_readfirstlane(a0.plan[a0.n_req].first);
  else if constexpr (SPLIT) n_pieces = a0.n_whole - a0.first_piece + (a0.n_units - a0.n_whole) * a0.n_split;
  if constexpr (OWN) {
    const int own = __builtin_amdgcn_readfirstlane(*a0.own_n);
    if (own > 0) n_pieces = a0.n_whole - a0.first_piece + own;
  }
  int q_grp = grp, q_pos = member;   // SPLIT: the queue and the place in it of the next piece
  // The next piece; q_pos = -1: there is none.  It is asked for when the one before it is done: asked for at the start of that, to have the
  // answer at hand, it waited for its workgroup where others had nothing left to do (28 heads: 5,084 rows at 45K keys 3,219 us, 2,998 so,
  // 8,000 dense ones at 20K 1,914 and 1,758; 34 requests of up to 16 rows 100 and 81).
  auto next_piece = [&]() {
    const AttnArgs& z0 = late_args();
    const int lead = TAIL ? 0 : z0.members;   // of a queue, that go to whom they lie at
    int* const next_s = (int*)vidx_s;
    if (tid < 64) {
      uint32_t first = 0;
      if (lane == 0) first = atomicAdd(&z0.queue[grp * kQueueStride], 1u);
      int at = (int)__builtin_amdgcn_readfirstlane(first) + lead, from = grp;
      auto left_in = [&](int x) -> int {   // pieces of queue x: whole runs of `members`, and the run that the last piece ends in
        const int runs = n_pieces / z0.members, tail = n_pieces - runs * z0.members;
        return ((runs - x + 7) >> 3) * z0.members + ((runs & 7) == x ? tail : 0);
      };
      while (at >= left_in(from)) {
        // the own queue is empty: the one with the most left.  A queue only ever grows emptier, so this ends
        const int x = lane & 7;
        const int seen = (int)__hip_atomic_load(&z0.queue[x * kQueueStride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + lead;
        int best = left_in(x) - seen > 0 ? ((left_in(x) - seen) << 3) | x : 0;
#pragma unroll
        for (int d = 1; d < 8; d <<= 1) { const int y = __shfl_xor(best, d); best = y > best ? y : best; }
        best = __builtin_amdgcn_readfirstlane(best);
        if (best == 0) { at = -1; break; }
        from = best & 7;
        uint32_t got = 0;
        if (lane == 0) got = atomicAdd(&z0.queue[from * kQueueStride], 1u);
        at = (int)__builtin_amdgcn_readfirstlane(got) + lead;
      }
      if (tid == 0) { next_s[0] = at; next_s[1] = from; }
    }
    __syncthreads();   // (also: the LDS tiles are reused by the next piece)
    q_pos = __builtin_amdgcn_readfirstlane(next_s[0]);
    q_grp = __builtin_amdgcn_readfirstlane(next_s[1]);
    __syncthreads();   // the next piece writes column indices there
  };
  if constexpr (TAIL) {
    next_piece();
    if (q_pos < 0) return;
  }
  for (int rnd = 0; SPLIT || rnd < n_gr; ++rnd) {
  int gr = 0, u = 0;
  if constexpr (SPLIT) {
    u = ((q_pos / a0.members) * 8 + q_grp) * a0.members + q_pos % a0.members;
    // (pieces that the host cannot count: fewer than workgroups are dealt evenly over the XCDs, as launch_attention does)
    if (!TAIL && (BATCH || OWN) && n_pieces < (int)gridDim.x) {
      const int each = (n_pieces + 7) >> 3;
      u = member < each ? grp * each + member : n_pieces;
    }
  } else {
    gr = __builtin_amdgcn_readfirstlane(a0.sched[grp * n_gr + rnd]);
    if (gr < 0) break;
  }
  // this round's view of the arguments: the kernel's own, or (BATCH) those of the unit's request
  AttnArgs a_req;
  if constexpr (BATCH) a_req = a0;
  const AttnArgs& a = BATCH ? a_req : a0;
  int g, h, qt, sp = 0, slot = 0, n_sp = 1, own = -1;   // own: piece of an uneven cut
  bool whole = true, none = false;   // none: no tile for this workgroup in this round
  if constexpr (SPLIT) {
    none = u >= n_pieces;
    if constexpr (BATCH) {
      if (!none) {
        const int r = batch_find<&BatchPlan::first>(a0.plan, a0.n_req, u);
        u -= __builtin_amdgcn_readfirstlane(a0.plan[r].first);
        none = !batch_view(a0, r, a_req);
      }
    }
    if constexpr (!BATCH) u += a0.first_piece;
    int e = u;
    whole = u < a.n_whole;
    if (!whole && !none) {
      const int v = u - a.n_whole, n = a.n_units - a.n_whole;
      if (OWN && __builtin_amdgcn_readfirstlane(*a.own_n) > 0) {
        own = v;
        const OwnPiece* const o = a.own_pieces + v;
        e = __builtin_amdgcn_readfirstlane(o->unit);
        sp = __builtin_amdgcn_readfirstlane(o->sp);
        n_sp = __builtin_amdgcn_readfirstlane(o->n_sp);
        slot = __builtin_amdgcn_readfirstlane(o->slot);
      } else {
        if (OWN) n_sp = a.n_split;
        sp = v / n;
        e = a.n_whole + v - sp * n;
        slot = BATCH ? v + a.first_slot : v;
      }
      if (OWN) whole = n_sp == 1;
    }
    g = h = qt = 0;
    if (!none) unit_of(a, e, g, h, qt);
  } else {
    if (gr < n_full_gr) {
      h = gr % a.n_q_heads;
      qt = a.n_rem + (a.n_full - 1 - gr / a.n_q_heads) * a.members + (a.members - 1 - member);
    } else {  // packed rounds: unit u = (head, tile below n_rem), tiles descending inside a head
      const int v = (gr - n_full_gr) * a.members + member;
      h = v / a.n_rem;
      qt = a.n_rem - 1 - v % a.n_rem;
      if (h >= a.n_q_heads) { h = 0; none = true; }
    }
    g = h / a.group;
  }
  // This wave's rows: query block t of the tile, 32 rows from block row il0; with packed heads the one query block,
  // the rows from its first live one, and head h + th (whose bit in an entry's mask is th)
  const int pack = SPLIT ? a.pack : 1;
  int t = wv >> 1, th = 0, il0 = (wv & 1) << 5;
  if (SPLIT && pack > 1) {
    t = 0;
    th = pack == 4 ? wv : wv >> 1;
    il0 = a.row_pad + (pack == 4 ? 0 : il0);
  }
  const int mbit = SPLIT && pack > 1 ? th : t;
  const bool head_ok = !SPLIT || (h - g * a.group) + th < a.group;
  const int hw = head_ok ? h + th : h;             // this wave's head
  const int il = il0 + (lane & 31) < 64 ? il0 + (lane & 31) : 63;   // row inside the query block (rows behind it: not stored)
  const int64_t n_k = a.n_k;
  const uint32_t expected = (uint32_t)(rnd + 1) * (uint32_t)a.members;
  // marks key segments seg_done - 1, ..., s_new done for this member, then holds the workgroup
  // back (wave 0 polls, the others meet it at the step barrier) until the whole group is done
  // with segment s_new + 2
  int seg_done = s_glob_top + 1;
  bool patient = true;  // a wait that ran out (group not co-resident?) ends the waiting for this tile
  auto enter_segment = [&](int s_new, bool wait) {
    if constexpr (SPLIT) return;
    if (s_new >= seg_done - 1) return;  // still in the segment entered last
    if (wv == 0) {
      for (int sg = seg_done - 1 - lane; sg > s_new; sg -= 64) atomicAdd(&arr[sg], 1u);
      if (wait && patient && s_new + 2 <= s_glob_top) {
        int spins = 0;
        while (__hip_atomic_load(&arr[s_new + 2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < expected &&
               spins < 2048) {
          __builtin_amdgcn_s_sleep(16);
          ++spins;
        }
        patient = spins < 2048;
      }
    }
    seg_done = s_new + 1;
  };
  if (!SPLIT && none) {
    enter_segment(-1, false);
    continue;
  }
  if (!none) {
  const int64_t row0 = (int64_t)qt * (64 * NQB);
  const int row = (int)row0 + 64 * t + il0 + (lane & 31);
  const int m0 = (int)(a.q_start / 64) + qt * NQB;  // absolute index of query block t = 0
  const bool wave_valid = head_ok && row0 + 64 * t + il0 < a.q_len;
  const int64_t rows_in_tile = (a.q_len - row0) < 64 * NQB ? (a.q_len - row0) : 64 * NQB;
  const int64_t last_pos = a.same_pos ? n_k - 1 : a.q_start + row0 + rows_in_tile - 1;

  const uint32_t* bmA = a.bm_a + (int64_t)hw * a.bm_stride;
  const int seg_shift = __builtin_amdgcn_readfirstlane((int)(bmA[a.bm_words - 2] >> kListBits));  // sparser list, longer sync segments
  const uint32_t* ent_h = a.ent + (int64_t)(SPLIT ? g * a.n_hs + (h - g * a.group) / pack : h) * a.ent_stride;
  const int32_t* vidx_h = a.v_idx ? a.v_idx + (int64_t)h * a.v_budget : nullptr;
  // columns to gather of head h, with packed heads those of head h + i in lane i
  const int vcnt_l = a.v_idx ? (int)a.bm_a[(int64_t)(SPLIT ? h + (lane < pack && h - g * a.group + lane < a.group ? lane : 0) : h) * a.bm_stride + a.bm_words - 1] : 0;
  const int vcnt = __builtin_amdgcn_readfirstlane(vcnt_l);
  const int n_vt = (vcnt + 63) >> 6;
  const int cc_last = m0 + NQB - 1;  // entry cc stands for key block m0 + (NQB - 1) - cc >= 0

  const __bf16* kbase = a.k + (int64_t)g * a.k_stride_head;
  const __bf16* vbase = a.v + (int64_t)g * a.v_stride_head;

  // ---- Q^T operand: lane (i = lane%32, hh) holds Q[i][16 st + 8 hh .. +7] ----------------
  // With DCA the operand is one of three rotations of the same rows; q_var says which one the
  // registers hold (the walk goes from the query block's own keys backwards, so it changes
  // at most a few times per tile).
  bf16x8 qreg[DSTEPS];
  int q_var = 0;
  auto load_q = [&](int var) {
    const __bf16* qb = a.q;
    if constexpr (DCA) {
      if (var == 1) qb = a.q_succ;
      if (var == 2) qb = a.q_inter;
    }
    int rc = row - a.row_pad;  // the caller's row (clamped: padding and tail rows load a valid one)
    rc = rc < 0 ? 0 : (rc < (int)a.q_rows ? rc : (int)a.q_rows - 1);
    const __bf16* qp = qb + (int64_t)rc * a.q_stride_tok + (int64_t)hw * a.q_stride_head + 8 * hh;
#pragma unroll
    for (int st = 0; st < DSTEPS; ++st) qreg[st] = *(const bf16x8*)(qp + 16 * st);
    q_var = var;
  };
  load_q(0);

  f32x16 oacc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int x = 0; x < 16; ++x) oacc[db][x] = 0.f;
  // ---- softmax state of this wave's rows, and the tile whose PV contraction is still owed ----
  // The V^T P^T product of a tile runs one step after its K Q^T product (see the main loop), so
  // between two steps a wave carries the tile's probabilities as four bf16 MFMA operands and
  // their row sum.
  // Probabilities are 2^(score - m_o) with ONE reference m_o per row for accumulators, row sum
  // and pending tile alike.  Any reference gives the same softmax; it only has to keep the
  // numbers in range.  m_o is the true maximum of the row's first tile and is raised (with a
  // rescale, on the exact path only) when a score outruns it by more than 2^64, so the
  // steady-state path never touches the accumulators except through the MFMAs.
  float l_run = 0.f;
  float m_o = -INFINITY;  // scaled reference (log2 domain)
  bool have_max = false;  // every row of this wave has a finite m_o (uniform)
  bool pend = false;      // uniform
  bf16x8 pp[4];           // P^T operands of the pending tile: keys 16 u .. 16 u + 15 (in MFMA k order)
  float pend_ps = 0.f;
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int x = 0; x < 8; ++x) pp[u][x] = (__bf16)0.f;

  // ---- tile iterator (uniform over the workgroup, kept in scalar registers) -----------------
  // kind 0: slash tile, idx = cc, mask = query blocks that use it; kind 1: vertical tile,
  // idx = vt; kind 2: end.  Entries are fetched 64 at a time (one per lane), one batch ahead.
  // With a key split this workgroup walks the entries with cc in [cc_lo, cc_end] (of `ranges` of equal distances, or an uneven
  // cut's) and every `ranges`-th vertical tile; the first entry is searched for with 64 probes at a time (the list ascends
  // in cc and ends in sentinels): three loads in a row for 16K entries, 14 by bisection.
  int cc_end = cc_last, ei0 = 0;
  const int ranges = OWN ? n_sp : a.n_split, vstep = SPLIT && !whole ? ranges : 1;
  int vlin = sp - vstep;
  if (SPLIT && !whole) {
    const int per = (cc_last + ranges) / ranges;  // ceil((cc_last + 1) / ranges)
    int cc_lo = sp * per;
    cc_end = cc_lo + per - 1 < cc_last ? cc_lo + per - 1 : cc_last;
    if (OWN && own >= 0) {
      cc_lo = __builtin_amdgcn_readfirstlane(a.own_pieces[own].cc_lo);
      cc_end = __builtin_amdgcn_readfirstlane(a.own_pieces[own].cc_hi);
    }
    int lo = 0, hi = (int)a.ent_len - 1;  // the last entry is a sentinel: an answer always exists
    if (!BATCH && !a.ent) lo = hi = pack > 1 ? (cc_lo > NQB - 1 ? cc_lo - (NQB - 1) : 0) : cc_lo;
    while (lo < hi) {
      const int step = (hi - lo + 63) >> 6, x = lo + lane * step;
      const int below = __popcll(__ballot((int)(ent_h[x < hi ? x : hi] >> 4) < cc_lo));   // (never at hi)
      if (below == 0) break;
      hi = lo + below * step < hi ? lo + below * step : hi;
      lo += (below - 1) * step + 1;
    }
    ei0 = lo;
  }
  // entries at .. at + 63, one per lane: of the list, or (see build_list) of all blocks, which ends with the walk and not with sentinels
  auto entries = [&](int at) -> uint32_t {
    if (SPLIT && !BATCH && !a.ent) {
      const uint32_t i = (uint32_t)(at + lane);
      if (pack > 1) return ((i + NQB - 1) << 4) | 15u;
      return (i << 4) | (i < NQB - 1 ? ((1u << NQB) - 1u) & (((1u << NQB) - 1u) << (NQB - 1 - i)) : (1u << NQB) - 1u);
    }
    return ent_h[at + lane];
  };
  uint32_t ecache = entries(ei0 & ~63), ecache_nx = entries((ei0 & ~63) + 64);
  int ei = ei0 - 1;
  // Columns of vertical tiles go into a ring of four in LDS when the tile is found, two steps before its rows are copied:
  // slot (ring + n) & 3 for the tile n steps from now, written by the first wave, read behind the barrier of the step.
  // (Looked up when the rows were copied, K and then V, they cost two trips to memory in every such step: 4 sparse requests of
  // up to 200 rows and 4,671 keys 152 -> 116 us, 109 rows at 3,336 keys 64 -> 50, both with the search below.)
  int ring = -2;
  auto advance = [&](int& kind, int& idx, int& mask) {
    int k2 = kind, i2 = idx, m2 = 0;
    if (k2 == 0) {
      ++ei;
      if (__builtin_expect((ei & 63) == 0 && ei > ei0, 0)) {
        ecache = ecache_nx;
        ecache_nx = entries((ei & ~63) + 64);
      }
      const uint32_t e = __builtin_amdgcn_readlane(ecache, ei & 63);
      const int cc = (int)(e >> 4);
      if (cc <= cc_end) {
        i2 = cc; m2 = (int)(e & 15u);
        enter_segment((cc_last - cc) >> (a.sync_shift + seg_shift), true);
      } else {
        k2 = 1; i2 = sp - vstep;
        enter_segment(-1, false);  // the slash walk is over
      }
    }
    if (k2 == 1 && SPLIT && pack > 1) {
      // the tiles of the packed heads one after the other: idx = (head, tile of its columns).  The one query block of
      // the launch ends at the last key, so that no tile lies behind it
      vlin += vstep;
      int x = vlin, hd = 0;
      for (; hd < pack && h - g * a.group + hd < a.group; ++hd) {
        const int nt = (int)(__builtin_amdgcn_readlane(vcnt_l, hd) + 63) >> 6;
        if (x < nt) break;
        x -= nt;
      }
      if (hd < pack && h - g * a.group + hd < a.group) {
        i2 = (hd << kHeadShift) | x; m2 = 1 << hd;
        const int pos = 64 * x + lane;
        const int col = pos < __builtin_amdgcn_readlane(vcnt_l, hd) ? vidx_h[(int64_t)hd * a.v_budget + pos] : 0;
        if (wv == 0) vidx_s[((ring + 2) & 3) * 64 + lane] = col;
      } else { k2 = 2; i2 = 0; }
    } else if (k2 == 1) {
      const int vt = i2 + vstep;
      bool more = vt < n_vt;
      if (more) {
        const int col = 64 * vt + lane < vcnt ? vidx_h[64 * vt + lane] : 0;
        more = (int64_t)__builtin_amdgcn_readfirstlane(col) <= last_pos;
        if (wv == 0) vidx_s[((ring + 2) & 3) * 64 + lane] = col;
      }
      if (more) i2 = vt; else { k2 = 2; i2 = 0; }
    }
    // the descriptor is uniform by construction; say so, so that it lives in scalar registers
    kind = __builtin_amdgcn_readfirstlane(k2);
    idx = __builtin_amdgcn_readfirstlane(i2);
    mask = __builtin_amdgcn_readfirstlane(m2);
  };
  // key index that row r of a slash tile comes from (general path)
  auto src_row = [&](int idx, int r) -> int64_t {
    int64_t j = (int64_t)(m0 - (idx - (NQB - 1))) * 64 + r;
    return j < n_k ? j : n_k - 1;
  };

  // ---- staging: global -> LDS copies, GPW groups of RPG rows per wave for K and for V --------
  // wave wv copies groups q = e * (2 NQB) + wv, e = 0..GPW-1; with this interleaving the
  // swizzle of a lane's row does not depend on e, so one 32-bit offset per lane serves all
  // its copies and the e-dependent part stays in scalar registers.
  constexpr int WAVES = 2 * NQB;
  const int lr = lane / DCH, lc = lane % DCH;  // this lane's row inside a group, and its LDS slot
  const int r0 = wv * RPG + lr;                // its row in the group e = 0
  const int kch = lc ^ ((r0 / R) % DCH);       // d-chunk it fetches for K (after the swizzle)
  const int vch = lc ^ ((((r0 / R) & 3) << 2) & (DCH - 1));  // ... and for V
  static_assert((WAVES * RPG / R) % DCH == 0 && (WAVES * RPG / R) % 4 == 0, "swizzle must not depend on e");
  static_assert(GPW == 1 || GPW == 2 || GPW == 4, "copies of a tile per wave");
  uint32_t koff[GPW], voff[GPW];  // byte offset of this lane's 16 bytes in copy e of a tile
#pragma unroll
  for (int e = 0; e < GPW; ++e) {
    koff[e] = (uint32_t)((e * WAVES * RPG + r0) * a.k_stride_tok * 2 + kch * 16);
    voff[e] = (uint32_t)((e * WAVES * RPG + r0) * a.v_stride_tok * 2 + vch * 16);
  }
  auto issue_k = [&](int kind, int idx, int buf, int slot) {
    const uint32_t kdst = ks_addr + (uint32_t)(buf * TILE * 2 + wv * 1024);
    bool fast = false;
    if (kind == 0) {
      const int64_t j0 = (int64_t)(m0 - (idx - (NQB - 1))) * 64;
      if (__builtin_expect(j0 + 64 <= n_k, 1)) {  // whole block in range: uniform bases + one per-lane 32-bit offset
        fast = true;
        const char* kt = (const char*)kbase + j0 * a.k_stride_tok * 2;
        if constexpr (GPW == 4) dma16x4(kdst, kt, koff[0], koff[1], koff[2], koff[3], WAVES * 1024);
        else if constexpr (GPW == 2) dma16x2(kdst, kt, koff[0], koff[1], WAVES * 1024);
        else dma16_lane_ptr(kdst, kt + koff[0]);
      }
    }
    if (__builtin_expect(!fast, 0)) {
#pragma unroll
      for (int e = 0; e < GPW; ++e) {
        const int64_t j = kind == 1 ? (int64_t)vidx_s[slot * 64 + e * WAVES * RPG + r0] : src_row(idx, e * WAVES * RPG + r0);
        dma16_lane_ptr(kdst + e * WAVES * 1024, kbase + j * a.k_stride_tok + kch * 8);
      }
    }
  };
  auto issue_v = [&](int kind, int idx, int buf, int slot) {
    const uint32_t vdst = vs_addr + (uint32_t)(buf * TILE * 2 + wv * 1024);
    bool fast = false;
    if (kind == 0) {
      const int64_t j0 = (int64_t)(m0 - (idx - (NQB - 1))) * 64;
      if (__builtin_expect(j0 + 64 <= n_k, 1)) {
        fast = true;
        const char* vt = (const char*)vbase + j0 * a.v_stride_tok * 2;
        if constexpr (GPW == 4) dma16x4(vdst, vt, voff[0], voff[1], voff[2], voff[3], WAVES * 1024);
        else if constexpr (GPW == 2) dma16x2(vdst, vt, voff[0], voff[1], WAVES * 1024);
        else dma16_lane_ptr(vdst, vt + voff[0]);
      }
    }
    if (__builtin_expect(!fast, 0)) {
#pragma unroll
      for (int e = 0; e < GPW; ++e) {
        const int64_t j = kind == 1 ? (int64_t)vidx_s[slot * 64 + e * WAVES * RPG + r0] : src_row(idx, e * WAVES * RPG + r0);
        dma16_lane_ptr(vdst + e * WAVES * 1024, vbase + j * a.v_stride_tok + vch * 8);
      }
    }
  };
  auto wait_copies = [&]() { __builtin_amdgcn_s_waitcnt(0x0F70); };  // vmcnt(0)

  // ---- per-lane LDS element offsets of the MFMA operands -------------------------------------
  // K rows as A operand of S^T = K Q^T: lane (j = lane%32, hh) reads d-chunk 2 st + hh of row j
  int k_ofs[DSTEPS];
  {
    const int y = hh ^ (((lane & 31) / R) % DCH);
#pragma unroll
    for (int st = 0; st < DSTEPS; ++st) k_ofs[st] = (lane & 31) * D + ((2 * st) ^ y) * 8;
  }
  // V^T operand through the transposing LDS read: inside each 16-lane group, lane L supplies
  // the address of V[J0 + L/4][D0 + 4 (L%4) .. +3] and receives V[J0 .. J0+3][D0 + L];
  // D0 = 32 db + 16 * (group & 1), J0 = (multiple of 8) + 4 hh.
  int v_ofs[DB];
  {
    const int rl = ((lane & 15) >> 2) + 4 * hh;
    const int gl = (((rl / R) & 3) << 2) & (DCH - 1);
    const int ul = 2 * ((lane >> 4) & 1) + ((lane >> 1) & 1);
#pragma unroll
    for (int db = 0; db < DB; ++db) v_ofs[db] = rl * D + (((4 * db + ul) ^ gl) * 8) + 4 * (lane & 1);
  }

  auto k_load = [&](const __bf16* kb, int jb, int st) -> bf16x8 {
    return *(const bf16x8*)&kb[k_ofs[st] + 32 * jb * D];
  };
  auto v_load = [&](const __bf16* vb, int jb, int tt, int db) -> bf16x8 {
    typedef bf16x4 __attribute__((address_space(3))) * lds_b4;
    const __bf16* p0 = &vb[v_ofs[db] + (32 * jb + 16 * tt) * D];
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_b4)(p0));
    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_b4)(p0 + 8 * D));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  };
  auto qk_step = [&](f32x16& acc, const __bf16* kb, int jb, int st) {
    const bf16x8 ka = *(const bf16x8*)&kb[k_ofs[st] + 32 * jb * D];
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qreg[st], acc, 0, 0, 0);
  };
  auto to_bf16 = [&](const f32x16& sv, int tt) -> bf16x8 {
    f32x8 pf;
#pragma unroll
    for (int x = 0; x < 8; ++x) pf[x] = sv[8 * tt + x];
    return __builtin_convertvector(pf, bf16x8);
  };
  auto block_max = [&](const f32x16& sv) -> float {
    float mx = sv[0];
#pragma unroll
    for (int x = 1; x < 16; ++x) mx = fmaxf(mx, sv[x]);
    return mx;
  };
  // sv <- exp2(sv * scale_log2 - m_ref); returns this lane's sum of the 16 probabilities
  auto exp_block = [&](f32x16& sv, float m_ref) -> float {
    float ps = 0.f;
#pragma unroll
    for (int x = 0; x < 16; ++x) {
      const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(sv[x], a.scale_log2, -m_ref));
      sv[x] = p;
      ps += p;
    }
    return ps;
  };

  // ---- per-step building blocks ----------------------------------------------------------------
  const float c = a.scale_log2;
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
  typedef __attribute__((ext_vector_type(2))) float f32x2;
  constexpr float kTooLarge = 1.8446744e19f;  // 2^64: a probability above it means the reference is stale
  // probabilities of score pair (x, x + 1) of sv relative to ref, rounded to bf16 into operand
  // P0 (x < 8) or P1; the row sum takes the unrounded values (it also feeds the lse output)
  auto exp_pair = [&](const f32x16& sv, int x, float ref, bf16x8& P0, bf16x8& P1, float& ps) {
    f32x2 pf;
    pf[0] = __builtin_amdgcn_exp2f(__builtin_fmaf(sv[x], c, -ref));
    pf[1] = __builtin_amdgcn_exp2f(__builtin_fmaf(sv[x + 1], c, -ref));
    const bf16x2 pk = __builtin_convertvector(pf, bf16x2);
    ps += pf[0] + pf[1];
    bf16x8& P = x < 8 ? P0 : P1;
    P[x & 7] = pk[0];
    P[(x & 7) + 1] = pk[1];
  };
  constexpr int NM = DSTEPS;  // MFMAs of one 32-key half of K Q^T, and of one half of V^T P^T
  static_assert(2 * DB == DSTEPS, "both contractions of a half take the same number of MFMAs");
  // V fragment u (0 .. 2 NM - 1) of the pending tile: half u / NM, k-step tt, output block db
  auto v_frag = [&](const __bf16* vbp, int u) -> bf16x8 { return v_load(vbp, u / NM, (u % NM) / DB, u % DB); };

  // V^T P^T of the pending tile alone (this wave has no K Q^T to pair it with in this step)
  auto drain = [&](const __bf16* vbp) {
    constexpr int VPF = 3, VNB = VPF + 1;
    bf16x8 vf[VNB];
#pragma unroll
    for (int j = 0; j < VPF; ++j) vf[j] = v_frag(vbp, j);
#pragma unroll
    for (int u = 0; u < 2 * NM; ++u) {
      if (u + VPF < 2 * NM) vf[(u + VPF) % VNB] = v_frag(vbp, u + VPF);
      oacc[u % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[u % VNB], pp[u / DB], oacc[u % DB], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    l_run += pend_ps;
    pend = false;
  };

  // K Q^T of a masked tile, of the first tile of a row block, or of a tile whose scores
  // outran the reference: true maximum first, then the exponentials.  Nothing may be pending
  // (the accumulators must be up to date when the reference moves).  Leaves the tile pending.
  // offset of this row's position inside its 64-key block (the last key of the diagonal block it
  // may use); packed decode: all rows stand at the same position
  const int il_diag = a.same_pos ? a.pos_in_block : il;
  // DCA: first key block of the chunk that holds this wave's query block
  const int dca_cs = DCA ? ((m0 + t) / a.dca_cblk) * a.dca_cblk : 0;
  int need_var = 0;       // DCA: rotation this wave's tile needs; 3 = it differs inside the tile (codes in dcak_s)
  uint32_t dca_need = 0;  //      need_var == 3: bit v set iff some usable element needs rotation v
  bool qsw = false;       //      the registers hold another rotation than the tile needs
  auto qk_exact = [&](const __bf16* kb, bool diag, bool vert, auto&& apply_mask) {
    f32x16 s0, s1;
#pragma unroll
    for (int x = 0; x < 16; ++x) { s0[x] = 0.f; s1[x] = 0.f; }
    if (DCA && need_var == 3) {
      // one product per rotation that occurs in the tile; an element takes the product of its
      // own pattern.  Code of key r: 100 = intra-chunk; otherwise a threshold thr: rows
      // il < thr are inside the local window (successive-chunk), the others inter-chunk.
#pragma unroll
      for (int var = 0; var < 3; ++var) {
        if (!((dca_need >> var) & 1u)) continue;
        if (q_var != var) load_q(var);
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) {
          f32x16 tt;
#pragma unroll
          for (int x = 0; x < 16; ++x) tt[x] = 0.f;
#pragma unroll
          for (int st = 0; st < DSTEPS; ++st) qk_step(tt, kb, jb, st);
#pragma unroll
          for (int xq = 0; xq < 4; ++xq) {
            const uint32_t cd = *(const uint32_t*)&dcak_s[wv * 64 + 32 * jb + 8 * xq + 4 * hh];
#pragma unroll
            for (int x = 0; x < 4; ++x) {
              const int code = (int)((cd >> (8 * x)) & 255u);
              const int ev = code == 100 ? 0 : (il_diag < code ? 1 : 2);
              if (ev == var) {
                if (jb == 0) s0[4 * xq + x] = tt[4 * xq + x];
                else s1[4 * xq + x] = tt[4 * xq + x];
              }
            }
          }
        }
      }
    } else {
#pragma unroll
      for (int st = 0; st < DSTEPS; ++st) qk_step(s0, kb, 0, st);
#pragma unroll
      for (int st = 0; st < DSTEPS; ++st) qk_step(s1, kb, 1, st);
    }
    if (diag || vert) {
      apply_mask(s0, 0);
      apply_mask(s1, 1);
    }
    float mx = fmaxf(block_max(s0), block_max(s1));
    mx = fmaxf(mx, __shfl_xor(mx, 32)) * c;
    if (!have_max || __any(mx > m_o + 64.f)) {
      const float m_new = fmaxf(m_o, mx);
      const float alpha = m_new == m_o ? 1.f : __builtin_amdgcn_exp2f(m_o - m_new);
      m_o = m_new;
      l_run *= alpha;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int x = 0; x < 16; ++x) oacc[db][x] *= alpha;
      have_max = !__any(m_o == -INFINITY);
    }
    const float m_use = (m_o == -INFINITY) ? 0.f : m_o;
    float ps = 0.f;
#pragma unroll
    for (int x = 0; x < 16; x += 2) exp_pair(s0, x, m_use, pp[0], pp[1], ps);
#pragma unroll
    for (int x = 0; x < 16; x += 2) exp_pair(s1, x, m_use, pp[2], pp[3], ps);
    pend_ps = ps;
    pend = true;
  };

  // K Q^T of an unmasked tile with nothing pending: S(keys 0..31), then S(keys 32..63) with the
  // exponentials of the first half between its MFMAs.  Returns false if a score outran the
  // reference (the caller then redoes the tile on the exact path).
  auto qk_fast = [&](const __bf16* kb) -> bool {
    constexpr int PF = 3, NB = PF + 1;
    bf16x8 kf[NB];
    f32x16 sa, sn;
#pragma unroll
    for (int x = 0; x < 16; ++x) { sa[x] = 0.f; sn[x] = 0.f; }
#pragma unroll
    for (int j = 0; j < PF; ++j) kf[j] = k_load(kb, j / NM, j % NM);
#pragma unroll
    for (int st = 0; st < NM; ++st) {
      const int j = st + PF;
      kf[j % NB] = k_load(kb, j / NM, j % NM);
      sa = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[st % NB], qreg[st], sa, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    float ps = 0.f;
#pragma unroll
    for (int st = 0; st < NM; ++st) {
      const int j = NM + st + PF;
      if (j < 2 * NM) kf[j % NB] = k_load(kb, 1, j - NM);
      sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[(NM + st) % NB], qreg[st], sn, 0, 0, 0);
#pragma unroll
      for (int x = (16 / NM) * st; x < (16 / NM) * (st + 1); x += 2) exp_pair(sa, x, m_o, pp[0], pp[1], ps);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int x = 0; x < 16; x += 2) exp_pair(sn, x, m_o, pp[2], pp[3], ps);
    if (__builtin_expect(__any(!(ps < kTooLarge)), 0)) return false;
    pend_ps = ps;
    pend = true;
    return true;
  };

  // The steady state: K Q^T of this tile and V^T P^T of the previous one in one instruction
  // stream, so that most MFMAs have a share of the softmax arithmetic next to them:
  //   A  NM MFMAs      QK(keys 0..31)
  //   B  3 NM / 2      QK(keys 32..63) with a quarter of PV(prev) mixed in | exp of keys 0..31
  //   C  3 NM / 2      the rest of PV(prev)                               | exp of keys 32..63
  // LDS operands are fetched PF MFMAs ahead; the scheduling fences pin the interleaving.
  // Returns false if a score outran the reference; the previous tile is folded in either way.
  auto fused = [&](const __bf16* kb, const __bf16* vbp, auto&& launch) -> bool {
    constexpr int PF = 3, NB = PF + 1;
    constexpr int NBQ = NM / 2;  // PV MFMAs mixed into phase B
    // MFMA n of the step: which operand it takes from LDS
    auto is_k = [&](int n) -> bool { return n < NM || (n < NM + 3 * NBQ && (n - NM) % 3 != 2); };
    auto k_index = [&](int n) -> int { return n < NM ? n : NM + 2 * ((n - NM) / 3) + (n - NM) % 3; };  // jb * NM + st
    auto v_index = [&](int n) -> int { return n < NM + 3 * NBQ ? (n - NM) / 3 : n - NM - 2 * NBQ; };
    auto frag = [&](int n) -> bf16x8 {
      if (is_k(n)) return k_load(kb, k_index(n) / NM, k_index(n) % NM);
      return v_frag(vbp, v_index(n));
    };
    bf16x8 fq[NB];
    f32x16 sa, sn;
#pragma unroll
    for (int x = 0; x < 16; ++x) { sa[x] = 0.f; sn[x] = 0.f; }
#pragma unroll
    for (int j = 0; j < PF; ++j) fq[j] = frag(j);
    // the first operands are on their way from LDS while the copies are launched
    __builtin_amdgcn_sched_barrier(0);
    launch();
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(2);  // this wave's MFMA stream goes before the other workgroup's bookkeeping
    bf16x8 q0, q1;  // the second half's operands replace pp[0], pp[1], which are spent by then
    float ps = 0.f;
    int xa = 0, xb = 0;  // next score pair of each half (compile-time after unrolling)
#pragma unroll
    for (int n = 0; n < 4 * NM; ++n) {
      if (n + PF < 4 * NM) fq[(n + PF) % NB] = frag(n + PF);
      if (is_k(n)) {
        const int ki = k_index(n);
        if (ki < NM) sa = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fq[n % NB], qreg[ki], sa, 0, 0, 0);
        else sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fq[n % NB], qreg[ki - NM], sn, 0, 0, 0);
      } else {
        const int u = v_index(n);
        oacc[u % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fq[n % NB], pp[u / DB], oacc[u % DB], 0, 0, 0);
      }
      if (n >= NM && n < NM + 3 * NBQ) {
        const int hi = 16 * (n - NM + 1) / (3 * NBQ);
        for (; xa + 2 <= hi; xa += 2) exp_pair(sa, xa, m_o, q0, q1, ps);
      } else if (n >= NM + 3 * NBQ) {
        const int hi = 16 * (n - NM - 3 * NBQ + 1) / (3 * NBQ);
        for (; xb + 2 <= hi; xb += 2) exp_pair(sn, xb, m_o, pp[0], pp[1], ps);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_s_setprio(0);
    l_run += pend_ps;
    pend = false;
    if (__builtin_expect(__any(!(ps < kTooLarge)), 0)) return false;
    pp[2] = pp[0]; pp[3] = pp[1]; pp[0] = q0; pp[1] = q1;
    pend_ps = ps;
    pend = true;
    return true;
  };

  // ---- prologue: K of tile 0 -> LDS buffer 0 ----------------------------------------------------
  int cur_kind = 0, cur_idx = -1, cur_mask = 0;
  advance(cur_kind, cur_idx, cur_mask);
  int nxt_kind = cur_kind, nxt_idx = cur_idx, nxt_mask = cur_mask;
  if (cur_kind != 2) {
    if (cur_kind == 1) __syncthreads();   // (a piece without a slash tile: its columns were found just now)
    issue_k(cur_kind, cur_idx, 0, 0);
    ring = -1;
    advance(nxt_kind, nxt_idx, nxt_mask);
  }
  ring = 0;
  wait_copies();
  __syncthreads();
  int buf = 0;

  // Step i multiplies K of tile i (LDS buffer i % 2) with Q and V of tile i - 1 (buffer
  // (i - 1) % 2) with its probabilities.  The copies of K(i + 1) and V(i) into the two free
  // buffers run under this arithmetic; one barrier per step.  One extra step after the last
  // tile drains the pipeline.
  bool last = false, part = false, diag = false, vert = false;
  const __bf16* kb = Ks;
  const __bf16* vbp = Vs;
  // element x of block jb is key r = 32 jb + 8 (x/4) + 4 hh + (x%4) of the tile
  auto apply_mask = [&](f32x16& sv, int jb) {
    if (diag) {
#pragma unroll
      for (int x = 0; x < 16; ++x) {
        const int r = 32 * jb + 8 * (x >> 2) + 4 * hh + (x & 3);
        if (r > il_diag) sv[x] = -INFINITY;
      }
    } else {
#pragma unroll
      for (int xq = 0; xq < 4; ++xq) {
        const uint32_t nd = *(const uint32_t*)&need_s[wv * 64 + 32 * jb + 8 * xq + 4 * hh];
#pragma unroll
        for (int x = 0; x < 4; ++x)
          if (il < (int)((nd >> (8 * x)) & 255u)) sv[4 * xq + x] = -INFINITY;
      }
    }
  };
  // start of a step: find out whether this wave takes part in tile i and with which element
  // mask.  A masked tile gives every key r of the tile a threshold need[r]:
  // row il of the query block may use it iff il >= need[r] (64 = never).  Slash tile on the
  // block's own diagonal: need[r] = r.  Vertical tile: 0 for a column of an earlier, uncovered
  // key block; the column's offset inside the block when it lies in the query block's own key
  // block; 64 when it is out of range, in a later block, or already covered by a computed
  // diagonal.
  auto classify = [&]() {
    last = cur_kind == 2;
    kb = Ks + buf * TILE;
    vbp = Vs + (buf ^ 1) * TILE;
    part = wave_valid && !last;
    diag = false;
    bool usable = false;  // vertical tile: this lane's key can be used by some row of the block
    if (__builtin_expect(cur_kind == 0, 1)) {
      part = part && ((cur_mask >> mbit) & 1);
      diag = cur_idx - (NQB - 1) + t == 0;  // block diagonal 0 of (query block t, this key block)
    } else if (!last) {
      int pos = 64 * cur_idx + lane, n_cols = vcnt;
      if (SPLIT && pack > 1) {
        const int hd = cur_idx >> kHeadShift;
        pos = 64 * (cur_idx & ((1 << kHeadShift) - 1)) + lane;
        n_cols = __builtin_amdgcn_readlane(vcnt_l, hd);
        part = part && hd == th;
      }
      const int j = vidx_s[(ring & 3) * 64 + lane];
      const int ad = (m0 + t) - (j >> 6);
      int need = 64;
      if (pos < n_cols && ad >= 0 && !bm_test(bmA, ad)) need = ad == 0 ? (j & 63) : 0;
      need_s[wv * 64 + lane] = (uint8_t)need;
      usable = need < 64;
      part = part && __ballot(usable) != 0;
    }
    vert = cur_kind == 1;
    if constexpr (DCA) {
      // which rotation of Q meets this tile's keys (section 5.1, DCA paragraph): keys of the
      // query block's own chunk the intra-chunk one; keys of the chunk before it, closer than
      // the local window, the successive-chunk one; all others the inter-chunk one
      qsw = false;
      if (part) {
        if (cur_kind == 0) {
          const int dblk = cur_idx - (NQB - 1) + t;  // block distance, >= 0 for a tile this wave takes
          const int cb = m0 + t - dblk;               // the key block
          if (cb >= dca_cs) need_var = 0;
          else if (cb >= dca_cs - a.dca_cblk && dblk < a.dca_wblk) need_var = 1;
          else if (cb >= dca_cs - a.dca_cblk && dblk == a.dca_wblk) {
            // the window ends inside this block: distance 64 dblk + il - r < window iff il < r
            need_var = 3;
            dca_need = 6u;
            dcak_s[wv * 64 + lane] = (uint8_t)lane;
          } else need_var = 2;
        } else {
          const int j = vidx_s[(ring & 3) * 64 + lane];
          const int cb = j >> 6;
          int code = 0;
          if (cb >= dca_cs) code = 100;
          else if (cb >= dca_cs - a.dca_cblk) {
            const int thr = 64 * a.dca_wblk - (64 * (m0 + t) - j);  // il < thr: inside the window
            code = thr < 0 ? 0 : (thr > 64 ? 64 : thr);
          }
          dcak_s[wv * 64 + lane] = (uint8_t)code;
          dca_need = (__ballot(usable && code == 100) != 0 ? 1u : 0u) |
                     (__ballot(usable && code != 100 && code > 0) != 0 ? 2u : 0u) |
                     (__ballot(usable && code < 64) != 0 ? 4u : 0u);
          need_var = 3;
        }
        qsw = need_var != q_var;
        if (qsw && cur_kind == 0) {
          // a slash tile that needs another rotation takes the path of the masked tiles, with
          // a mask that lets every row use every key
          vert = true;
          need_s[wv * 64 + lane] = 0;
        }
      }
    }
  };
  // copies of K(i + 1) and V(i) into the buffers that step i - 1 used last
  auto launch_copies = [&]() {
    if (!last) {
      if (nxt_kind != 2) issue_k(nxt_kind, nxt_idx, buf ^ 1, (ring + 1) & 3);
      issue_v(cur_kind, cur_idx, buf, ring & 3);
    }
  };
  auto end_step = [&]() {
    int nn_kind = nxt_kind, nn_idx = nxt_idx, nn_mask = nxt_mask;
    if (nxt_kind != 2) advance(nn_kind, nn_idx, nn_mask);
    wait_copies();
    __syncthreads();
    cur_kind = nxt_kind; cur_idx = nxt_idx; cur_mask = nxt_mask;
    nxt_kind = nn_kind; nxt_idx = nn_idx; nxt_mask = nn_mask;
    buf ^= 1;
    ++ring;
  };

  for (;;) {
    classify();
    // steady state: runs of steps in which this wave multiplies tile i and folds in tile i - 1
    while (__builtin_expect(pend && part && !(diag || vert || !have_max), 1)) {
      if (__builtin_expect(!fused(kb, vbp, launch_copies), 0)) qk_exact(kb, diag, vert, apply_mask);
      end_step();
      classify();
    }
    launch_copies();
    if (pend) drain(vbp);
    bool exact = diag || vert || !have_max;
    if constexpr (DCA) {
      if (part && qsw && need_var < 3) load_q(need_var);
    }
    if (part && !exact) exact = !qk_fast(kb);
    if (__builtin_expect(part && exact, 0)) qk_exact(kb, diag, vert, apply_mask);
    if (last) break;
    end_step();
  }

  // ---- normalise and store ------------------------------------------------------------------
  const AttnArgs& z0 = late_args();
  const AttnArgs& z = BATCH ? a : z0;
  const float l_tot = l_run + __shfl_xor(l_run, 32);
  const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
  if (SPLIT && !whole) {
    // this piece's share of the row: accumulators and row sum relative to the reference m_o
    const int64_t ro = row - z.row_pad;
    if (head_ok && ro >= 0 && ro < z.q_rows) {
      const int64_t pr = (int64_t)slot * kTileRows + 32 * wv + (lane & 31);
      float* op = z0.part_o + pr * D;
      float* mlp = z0.part_ml + pr * 2;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int vq = 0; vq < 4; ++vq) {
          f32x4 o4;
#pragma unroll
          for (int x = 0; x < 4; ++x) o4[x] = oacc[db][4 * vq + x];
          *(f32x4*)(op + 32 * db + 8 * vq + 4 * hh) = o4;
        }
      if (hh == 0) {
        mlp[0] = m_o;
        mlp[1] = l_tot;
      }
    }
  } else
  if (head_ok && row >= z.row_pad && row < z.q_len) {
    const int64_t ro = row - z.row_pad;
    __bf16* op = z.out + ro * z.o_stride_tok + (int64_t)hw * z.o_stride_head;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int vq = 0; vq < 4; ++vq) {
        f32x4 o4;
#pragma unroll
        for (int x = 0; x < 4; ++x) o4[x] = oacc[db][4 * vq + x] * inv;
        *(bf16x4*)(op + 32 * db + 8 * vq + 4 * hh) = __builtin_convertvector(o4, bf16x4);
      }
    if (z.lse && hh == 0)
      z.lse[(int64_t)hw * z.q_rows + ro] =
          l_tot > 0.f ? (m_o + __builtin_amdgcn_logf(l_tot)) * kLn2 : -INFINITY;
  }
  enter_segment(-1, false);  // (a tile whose walk ended early has marked nothing yet)
  }  // !none
  if constexpr (SPLIT) {
    if (!TAIL && n_pieces <= (int)gridDim.x) break;
    next_piece();
    if (q_pos < 0) break;
  } else {
    __syncthreads();   // the LDS tiles are reused by the next round
  }
  }  // rounds
}
template <int D, int NQB, bool DCA, bool SPLIT, bool BATCH = false>
__global__ __launch_bounds__(128 * NQB, 2) void k_attention(const AttnArgs a) { attention_body<D, NQB, DCA, SPLIT, BATCH, false>(a); }
// Whole units that keep pace, and then the pieces of the others, near ones (the longest) first: in one kernel, so that the workgroups
// whose rounds end early take more of them.  In two launches, the second as long as its longest piece, 28 heads: 11,109 clustered rows at
// 500K keys (lists between 920 and 2,120 blocks: rounds of a group 5 % above the mean) 17.3 ms, 15.9 so; 3,000 at 600K 7.4 and 5.6.
struct PacedArgs {
  AttnArgs whole, cut;
};
template <int D, int NQB, bool DCA>
__global__ __launch_bounds__(128 * NQB, 2) void k_attention_paced(const PacedArgs a) {
  attention_body<D, NQB, DCA, false, false, false>(a.whole);
  __syncthreads();
  attention_body<D, NQB, DCA, true, false, false, true>(a.cut, offsetof(PacedArgs, cut));
}
// A batch of single tokens and longer requests.  Tokens wait for memory, tiles for the matrix cores, so they share the compute units: the
// first workgroups, one on each (b and b + 256 lie on the same), walk the tokens, in half the LDS that k_decode takes, before they take
// pieces; the others take pieces from the start.  Six launches (two for lists, two walks, two folds) become three.  8 requests of 1 to 64 rows and
// 262,144 keys, dense and sparse, 1,210 us -> 1,130 (tokens by themselves 387, 424 in half the LDS; pieces 840); 22 dense ones of up to 64 rows and 38K keys,
// 40 heads, 419 -> 391, 34 of up to 16 rows and 1,100 keys 102 -> 81, 5 sparse ones of 51K keys 474 -> 411, 30 of up to 64 rows and 60K
// keys, 8 heads of 64, 131 -> 104.
struct MixedArgs {
  DecodeArgs tokens;
  AttnArgs rows;
};
template <int D, int NQB>
__global__ __launch_bounds__(128 * NQB, 2) void k_attention_mixed(const MixedArgs a) {
  static_assert(kDecThreads == 128 * NQB && decode_lds_bytes<D>() / 2 <= attn_lds_bytes<D>(), "one launch serves both");
  const int n_wg = a.tokens.shares < (int)gridDim.x ? a.tokens.shares : (int)gridDim.x;
  if ((int)blockIdx.x < n_wg) {
    int64_t mine;
    bool uneven;
    const int64_t T = decode_total<int4>(a.tokens, mine, uneven);
    if (D == 128 && a.tokens.side == 2 && T >= kDecSideBlocks && !uneven) decode_body<D, D == 128 ? 2 : 1, false, int4, true>(a.tokens, T / 2, mine, n_wg);
    else decode_body<D, 1, false, int4, true>(a.tokens, T, mine, n_wg);
    __syncthreads();
  }
  attention_body<D, NQB, false, true, true, false, true>(a.rows, offsetof(MixedArgs, rows));
}
template <int D, int NQB, bool DCA>
__global__ __launch_bounds__(128 * NQB, 2) void k_attention_own(const AttnArgs a) { attention_body<D, NQB, DCA, true, false, true>(a); }

// ---------------------------------------------------------------------------------------------
// Block list of one head from its selected slash offsets.
// Offset o crosses, inside a 64-aligned query block, the key blocks of diagonals floor(o/64)
// and, when o is not a multiple of 64, floor(o/64) + 1: these set the bitmap A.  The entry
// list then holds every cc for which A has a bit in [cc - (NQB-1), cc], with the per-query-
// block mask, in ascending order, followed by sentinels up to the end of the row.
// With packed heads (pack > 1) a list is that of a tile of `pack` heads with one query block: the union of their
// diagonals a, as cc = a + NQB - 1, with a mask bit per head that has the diagonal.
// List x0 is blockIdx.x, the part of a dense list blockIdx.y (the x axis takes any number of heads, y 65,535 workgroups).
// With req != null the launch builds one list per (request, head), blockIdx = (h, 1 + r):
// offsets, their count, the number of key blocks and "dense" (no offsets given) come from the
// request; a request that the attention kernel skips gets no list, and where it packs heads only as many as it
// has tiles.  The first workgroup of a batch writes its plan (write_plan), the lists follow.  The first workgroup also
// clears the n_zero words at `zero` (the attention launch's counters).
//
// A sparse list is one workgroup's (part 0) and bound by latency and instructions, not bytes (6,096 offsets of a head
// in, 16K bits and up to 64 KB of entries out).  Diagonals are collected as bytes in LDS (collect_flags): 28 heads, 20,000 keys
// 8 us -> 6, four heads per list, 300,000 keys, 30 -> 14, the lists of 32 requests 36 -> 22.  Entries are written 64 diagonals at a time
// with a lane per diagonal, so that the stores of a wave are contiguous.  A dense list needs no collecting and
// is cut into kBlDensePart entries per workgroup.
// ---------------------------------------------------------------------------------------------
constexpr int kBlThreads = 1024;
constexpr int kBlWin = 16384 + 64;  // diagonals of packed heads in LDS at a time (1M keys and what a bitmap has behind them; of one head
                                    // four times as many)
// Groups of 64 diagonals of a single call's lists up to which their bitmaps are made by ballots.  In instantiations of their own, because
// short calls wait for the instructions.  Calls of 4 heads with 256 offsets each, ballots and lanes: 2,500 keys 19.8 us and 20.2, 100,000
// (25 groups of four heads) 35.6 and 36.0, 300,000 (74) 34.4 and 34.2, 1M (245) 39.9 and 36.9.
constexpr int kBlBallots = 64;
constexpr int kBlDensePart = 4096;  // entries of a dense list per workgroup
constexpr int kListGroups = 4096;   // workgroups for the lists of a batch, about
struct ListArgs {
  const int32_t* s_idx;
  const int32_t* s_cnt;
  const int32_t* v_cnt;   // null: nobody gathers columns
  int32_t s_budget, dense, n_blk, n_words, ent_stride;
  uint32_t* bm_a;
  uint32_t* ent;
  int32_t n_heads, group, pack;
  uint32_t* zero;
  int32_t n_zero;
  // a batch
  const vs_request* req;
  BatchPlan* plan;
  int32_t n_req, skip_single, pieces;
  int64_t max_q_len, max_n_k;
};
// Steps (64-key blocks, columns at twice their number: they take the masked path) that a tile of the request walks, for the
// plan only: a list is taken to scatter.
__device__ __forceinline__ int64_t batch_steps(const vs_request& rq, const BatchShape& b) {
  const int64_t n_blk = (rq.q_start + rq.q_len + kBlock - 1) / kBlock;
  if (b.dense) return n_blk;
  const int64_t listed = 2 * (int64_t)rq.s_cnt[0] + 1;
  return (listed < n_blk ? listed : n_blk) + 2 * b.pack * ((rq.v_cnt[0] + 63) / 64);
}
// Ranges that equally long units are best cut into: rounds of kBatchSlots pieces.  Not the cut of attn_cut: all units or none are cut,
// in ranges of at least kMinBatchSteps (the caller sees to that), and the terms for a piece alone on its compute unit and for the serial
// part of the fold, fitted to single calls, are not counted.
__device__ int best_split(int64_t units, int64_t steps, int64_t most_pieces) {
  int best = 1;
  float best_cost = 0.f;
  for (int n = 1; n <= kMaxSplit && n <= steps; ++n) {
    const int64_t pieces = units * n;
    if (n > 1 && pieces > most_pieces) break;
    float cost = (float)((pieces + kBatchSlots - 1) / kBatchSlots) * ((float)steps / (float)n + (float)kPieceSteps);
    if (n > 1) cost += 3.f + 8.f * (float)pieces / (float)kBatchSlots;
    if (n == 1 || cost < best_cost) { best = n; best_cost = cost; }
  }
  return best;
}
// Ranges per unit so that all pieces of a batch come out about equally long and there are a.pieces of them: the requests
// differ in length, and a workgroup takes the next piece when it is done with one.  Rounded down, so that the split units
// have at most a.pieces pieces (slots of partial results).  The units of a single request are equally long: best_split says
// how they are cut (2,500 rows at 20,000 keys, 20 heads: 400 units whole 528 us, in three ranges each 613).
__device__ void write_plan(const ListArgs& a, int64_t* scan) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  constexpr int NW = kBlThreads / 64;
  auto look = [&](int r, BatchShape& b, int64_t& steps) -> bool {
    const vs_request rq = a.req[r];
    if (!batch_shape(rq, a.group, a.n_heads / a.group, a.max_q_len, a.max_n_k, a.skip_single, batch_pack(rq, a.group), b)) return false;
    steps = batch_steps(rq, b);
    return true;
  };
  BatchShape b;
  int64_t steps = 0, sum = 0;
  bool taken = false;   // of the request this thread looked at last (the only one of up to kBlThreads requests)
  for (int r = tid; r < a.n_req; r += kBlThreads) {
    taken = look(r, b, steps);
    if (taken) sum += b.n_units * steps;
  }
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) sum += __shfl_xor((long long)sum, d);
  if (lane == 0) scan[wv] = sum;
  __syncthreads();
  int64_t total = 0;
  for (int w = 0; w < NW; ++w) total += scan[w];
  __syncthreads();
  // (about three pieces per workgroup slot, one where they would come out short)
  const int64_t target = total < (int64_t)kBatchSlots * kShortSteps && a.pieces > kBatchSlots ? kBatchSlots : a.pieces;
  int64_t before = 0;   // pieces, from bit 32 on slots, from bit 48 on cut units (at most a.pieces of both)
  for (int r0 = 0; r0 < a.n_req; r0 += kBlThreads) {
    const int r = r0 + tid;
    int n_split = 0;
    int64_t mine = 0;
    if (a.n_req > kBlThreads) taken = r < a.n_req && look(r, b, steps);
    if (taken) {
      int64_t n = steps * target / total;
      if (a.n_req == 1) n = best_split(b.n_units, steps, a.pieces);
      if (n > steps / kMinBatchSteps) n = steps / kMinBatchSteps;
      n_split = n < 1 ? 1 : (n > kMaxSplit ? kMaxSplit : (int)n);
      const int64_t pieces = (int64_t)b.n_units * n_split;
      mine = pieces | (n_split > 1 ? pieces << 32 | (int64_t)b.n_units << 48 : 0);
    }
    int64_t inc = mine;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int64_t y = __shfl_up((long long)inc, d);
      if (lane >= d) inc += y;
    }
    if (lane == 63) scan[wv] = inc;
    __syncthreads();
    int64_t all = 0;
    for (int w = 0; w < NW; ++w) {
      if (w < wv) inc += scan[w];
      all += scan[w];
    }
    inc += before - mine;
    if (r < a.n_req) {
      a.plan[r].first = (int32_t)inc;
      a.plan[r].split_pack = n_split | (taken ? b.pack << 16 : 0);
      a.plan[r].slot = (int32_t)(inc >> 32) & 0xFFFF;
      a.plan[r].cut = (int32_t)(inc >> 48);
    }
    before += all;
    __syncthreads();
  }
  if (tid == 0) {
    a.plan[a.n_req].first = (int32_t)before;
    a.plan[a.n_req].split_pack = 0;
    a.plan[a.n_req].slot = (int32_t)(before >> 32) & 0xFFFF;
    a.plan[a.n_req].cut = (int32_t)(before >> 48);
  }
}
// List x0; false: nothing to be done for it or the ones behind it.  flags: kBlFlags bytes of LDS.
constexpr int kBlFlags = 16 + 4 * kBlWin + 16;
template <int NQB, bool BATCH, bool WIDE>
__device__ __forceinline__ bool build_list(const ListArgs& a, int x0, uint8_t* flags) {
  constexpr int NW = kBlThreads / 64;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int part = BATCH ? 0 : blockIdx.y, n_parts = BATCH ? 1 : gridDim.y;
  const int r = (int)blockIdx.y - 1;   // (of a batch, whose first workgroup is the plan's)
  const int n_words = a.n_words, ent_stride = a.ent_stride;
  int dense = a.dense, n_blk = a.n_blk, pack = a.pack, n_hs = (a.group + pack - 1) / pack;
  const int32_t* s_idx = a.s_idx;
  const int32_t* s_cnt = a.s_cnt;
  const int32_t* v_cnt = a.v_cnt;
  uint32_t* bm_a = a.bm_a;
  if constexpr (BATCH) {
    const vs_request rq = a.req[r];
    BatchShape b;
    if (!batch_shape(rq, a.group, a.n_heads / a.group, a.max_q_len, a.max_n_k, a.skip_single, batch_pack(rq, a.group), b)) return false;
    pack = b.pack;
    n_hs = b.n_hs;
    dense = b.dense;
    s_idx = rq.s_idx; s_cnt = rq.s_cnt; v_cnt = rq.v_cnt;
    n_blk = (int)((rq.q_start + rq.q_len + kBlock - 1) / kBlock);
    bm_a += (int64_t)r * a.n_heads * n_words;
    if (x0 >= (b.dense ? 1 : a.n_heads / a.group * n_hs)) return false;   // (a dense request has one list for all heads)
  }
  uint32_t* const E = a.ent + ((BATCH ? (int64_t)r * a.n_heads : 0) + x0) * ent_stride;
  // the first head of list x0, and how many heads it has
  const int grp = dense && !BATCH ? 0 : x0 / n_hs, h0 = dense && !BATCH ? 0 : grp * a.group + (x0 - grp * n_hs) * pack;
  const int n_in = grp * a.group + a.group - h0 < pack ? grp * a.group + a.group - h0 : pack;
  uint32_t* const A = bm_a + (int64_t)h0 * n_words;
  // The last two words of the bitmap row lie beyond every diagonal.  One holds the length of the list (the head's share of the work) and,
  // from bit kListBits on, how sparse it is: sync segments of this head are 2^shift times the base size, so that a segment holds about
  // as many listed key blocks as it would in a dense list.  The other holds the columns to gather: none where the head has every
  // diagonal (6,096 scattered offsets give all of them up to some 64K keys), because all their rows are walked.  28 heads, 4,096 rows
  // from the first on 296 us -> 250, 5,000 of 12,000 keys 827 -> 775; 32 requests of up to 64 rows and 20,000 keys 353 -> 285.
  const uint32_t cols = v_cnt ? (uint32_t)v_cnt[h0 + (tid < n_in ? tid : 0)] : 0u;   // (on its way from here; thread p writes head p's tail)
  auto write_tail = [&](int p, uint32_t n_list, int shift, bool full) {
    uint32_t* const row = A + (int64_t)p * n_words;
    row[n_words - 1] = full ? 0u : cols;
    row[n_words - 2] = n_list | (uint32_t)shift << kListBits;
  };
  if (dense && pack > 1) {
    for (int i = part * kBlDensePart + tid; i < ent_stride && (i < (part + 1) * kBlDensePart || n_parts == part + 1);
         i += kBlThreads)
      E[i] = i < n_blk ? ((uint32_t)(i + NQB - 1) << 4) | 15u : kEntSentinel;
    // (no bitmap: a dense walk has no columns that ask it)
    if (part == 0 && tid == 0) write_tail(0, (uint32_t)n_blk, 0, true);
    return true;
  }
  if (dense) {
    const int n_list = n_blk + NQB - 1, all = (1 << NQB) - 1;
    for (int i = part * kBlDensePart + tid; i < ent_stride && (i < (part + 1) * kBlDensePart || n_parts == part + 1);
         i += kBlThreads) {
      uint32_t e = kEntSentinel;
      if (i < n_list) {   // mask bit t = diagonal i - (NQB - 1) + t exists
        int mask = all;
        if (i < NQB - 1) mask &= all << (NQB - 1 - i);
        if (i >= n_blk) mask &= all >> (i - n_blk + 1);
        e = ((uint32_t)i << 4) | (uint32_t)mask;
      }
      E[i] = e;
    }
    if (part == 0) {
      for (int w = tid; w < n_words - 2; w += kBlThreads) {
        const int lo = w * 32;
        A[w] = lo + 32 <= n_blk ? ~0u : (lo < n_blk ? (1u << (n_blk - lo)) - 1u : 0u);
      }
      if (tid == 0) write_tail(0, (uint32_t)n_list, 0, true);
    }
    return true;
  }
  if (part != 0) return false;

  // A byte per diagonal of the window (of four heads side by side with pack > 1) from f on; behind it what lies outside, in front of it the
  // last diagonal before it.  Every wave has consecutive groups of 64 diagonals.  It writes their bitmaps and counts their entries,
  // and then writes the entries with a lane per diagonal.  The former by ballots of a lane per diagonal too, or, WIDE, with eight
  // diagonals of four heads, or 16 of one, per lane (see kBlBallots).
  static_assert(NQB == 2, "an entry has the diagonals of two query blocks");
  static_assert(kBlWin % 64 == 0, "whole groups");
  __shared__ uint32_t wsum[NW], missing_s;   // (a bit per head that lacks a diagonal)
  uint32_t running = 0, before = 0, missing = 0;
  if (tid == 0) missing_s = 0u;
  const int shift = pack > 1 ? 2 : 0, win = pack > 1 ? kBlWin : 4 * kBlWin;
  for (int b0 = 0; b0 < 32 * (n_words - 2); b0 += win) {
    const int bits = 32 * (n_words - 2) - b0, n_grp = ((bits < win ? bits : win) + 63) >> 6;
    uint8_t* const f = flags + 16;
    for (int x = tid; x < n_grp << (2 + shift); x += kBlThreads) ((u32x4*)f)[x] = u32x4{0u, 0u, 0u, 0u};
    if (tid == 0) f[-1] = (uint8_t)before;
    __syncthreads();
    const int n_in_win = n_blk - b0 < win ? (n_blk > b0 ? n_blk - b0 : 0) : win;
    collect_flags<kBlThreads, 8>(f, shift, b0, n_in_win, win, s_idx + (int64_t)h0 * a.s_budget, s_cnt + h0, a.s_budget, n_in);
    __syncthreads();
    // the mask of a diagonal's entry: the heads that have it, or, of one head, bit t: diagonal b0 + x - 1 + t
    auto mask_of = [&](int x) -> uint32_t {
      if (pack > 1) return (((const uint32_t*)f)[x] * 0x01020408u >> 24) & 15u;   // (bytes of 0 and 1 to bits)
      return (uint32_t)f[x - 1] | (uint32_t)f[x] << 1;
    };
    const int each = (n_grp + NW - 1) / NW, g0 = wv * each < n_grp ? wv * each : n_grp, g1 = g0 + each < n_grp ? g0 + each : n_grp;
    uint32_t c = 0;
    if constexpr (!WIDE)
      for (int grp = g0; grp < g1; ++grp) {
        const uint32_t mask = mask_of(64 * grp + lane), own = pack > 1 ? mask : mask >> 1;
        c += __popcll(__ballot(mask != 0u));
        if (b0 + 64 * grp + lane < n_blk) missing |= ~own & (pack > 1 ? 15u : 1u);
        // lanes 2 p, 2 p + 1 write the words of head p
        uint64_t bits_p = __ballot(own & 1u);
        if (pack > 1)
#pragma unroll
          for (int p = 1; p < 4; ++p) {
            const uint64_t b = __ballot((mask >> p) & 1u);
            bits_p = (lane >> 1) == p ? b : bits_p;
          }
        const int w = (b0 >> 5) + 2 * grp + (lane & 1);
        if (lane < 2 * n_in && w < n_words - 2) A[(int64_t)(lane >> 1) * n_words + w] = (uint32_t)(bits_p >> (32 * (lane & 1)));
      }
    auto add_up = [&](uint32_t mine) {   // mine: at most 16
#pragma unroll
      for (int b = 0; b < 5; ++b) c += (uint32_t)__popcll(__ballot((mine >> b) & 1u)) << b;
    };
    // diagonals from d on that exist, of n
    auto existing = [&](int d, int n) -> uint32_t { return d + n <= n_blk ? (1u << n) - 1u : (d < n_blk ? (1u << (n_blk - d)) - 1u : 0u); };
    if constexpr (!WIDE) {
    } else if (pack > 1) {
      for (int x0 = 8 * g0; x0 < 8 * g1; x0 += 64) {
        const int x = x0 + lane;
        uint32_t n = 0;
        if (x < 8 * g1) {
          const u32x4 lo = ((const u32x4*)f)[2 * x], hi = ((const u32x4*)f)[2 * x + 1];
          const uint32_t v = lo[0] | lo[1] << 1 | lo[2] << 2 | lo[3] << 3 | hi[0] << 4 | hi[1] << 5 | hi[2] << 6 | hi[3] << 7;   // (a byte per head)
          const uint32_t want = existing(b0 + 8 * x, 8);
#pragma unroll
          for (int p = 0; p < 4; ++p) {
            const uint32_t v_p = (v >> (8 * p)) & 0xFFu;
            if (p < n_in && b0 + 8 * x < 32 * (n_words - 2)) ((uint8_t*)(A + (int64_t)p * n_words))[(b0 >> 3) + x] = (uint8_t)v_p;
            missing |= v_p != want ? 1u << p : 0u;
          }
          n = __popc((v | v >> 8 | v >> 16 | v >> 24) & 0xFFu);
        }
        add_up(n);
      }
    } else {
      for (int x0 = 4 * g0; x0 < 4 * g1; x0 += 64) {
        const int x = x0 + lane;
        uint32_t n = 0;
        if (x < 4 * g1) {
          const u32x4 q = ((const u32x4*)f)[x];
          uint32_t v = 0;
#pragma unroll
          for (int y = 0; y < 4; ++y) v |= ((q[y] * 0x01020408u >> 24) & 15u) << (4 * y);
          if (b0 + 16 * x < 32 * (n_words - 2)) ((uint16_t*)A)[(b0 >> 4) + x] = (uint16_t)v;
          missing |= v != existing(b0 + 16 * x, 16) ? 1u : 0u;
          n = __popc((v | v << 1 | f[16 * x - 1]) & 0xFFFFu);
        }
        add_up(n);
      }
    }
    if (lane == 0) wsum[wv] = c;
    uint32_t lacks = 0;
#pragma unroll
    for (int p = 0; p < 4; ++p) lacks |= __ballot((missing >> p) & 1u) ? 1u << p : 0u;
    if (lane == 0) atomicOr(&missing_s, lacks);
    before = pack > 1 ? 0u : f[win - 1];
    __syncthreads();
    uint32_t pos = running;
    for (int x = 0; x < NW; ++x) {
      if (x < wv) pos += wsum[x];
      running += wsum[x];
    }
    for (int grp = g0; grp < g1; ++grp) {
      const uint32_t mask = mask_of(64 * grp + lane);
      const uint64_t m = __ballot(mask != 0u);
      if (mask)
        E[pos + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] =
            (uint32_t)(b0 + 64 * grp + lane + (pack > 1 ? NQB - 1 : 0)) << 4 | mask;
      pos += __popcll(m);
    }
    __syncthreads();   // wsum and flags are rewritten by the next window
  }
  for (int i = running + tid; i < ent_stride; i += kBlThreads) E[i] = kEntSentinel;
  if (pack > 1) {
    if (tid < n_in) write_tail(tid, running, 0, !(missing_s >> tid & 1u));
  } else if (tid == 0) {
    int sft = 0;
    while (sft < 4 && ((uint32_t)n_blk >> (sft + 1)) >= (running > 0 ? running : 1u)) ++sft;
    write_tail(0, running, sft, missing_s == 0u);
  }
  return true;
}
template <int NQB, bool BATCH, bool WIDE>
__device__ __forceinline__ void build_lists(const ListArgs& a, uint8_t* flags) {
  if (blockIdx.x == 0 && blockIdx.y == 0)
    for (int x = threadIdx.x; x < a.n_zero; x += kBlThreads) a.zero[x] = 0u;
  if constexpr (BATCH) {
    __shared__ int64_t scan[kBlThreads / 64];
    if (blockIdx.y == 0) {
      if (blockIdx.x == 0) write_plan(a, scan);
      return;
    }
    for (int x0 = blockIdx.x; x0 < a.n_heads; x0 += gridDim.x) {
      if (!build_list<NQB, true, WIDE>(a, x0, flags)) return;   // (the same for all threads)
      __syncthreads();   // its LDS is the next list's
    }
  } else {
    build_list<NQB, false, WIDE>(a, blockIdx.x, flags);
  }
}
template <int NQB, bool BATCH, bool WIDE = false>
__global__ __launch_bounds__(kBlThreads) void k_build_blocklist(const ListArgs a) {
  __shared__ __attribute__((aligned(16))) uint8_t flags[kBlFlags];
  build_lists<NQB, BATCH, WIDE>(a, flags);
}
// The lists of a batch (20 of 1,200 us when they came one after the other), and behind them, blockIdx.y from 1 + n_req on, those of its single tokens.
struct MixedListArgs {
  ListArgs rows;
  DecodeArgs tokens;
};
template <int NQB>
__global__ __launch_bounds__(kBlThreads) void k_mixed_lists(const MixedListArgs a) {
  static_assert(kBlThreads == kDecListThreads, "one launch serves both");
  constexpr int kTokenBytes = 64 << 10;
  __shared__ __attribute__((aligned(16))) uint8_t flags[kBlFlags > kTokenBytes + 16 ? kBlFlags : kTokenBytes + 16];
  const int r = (int)blockIdx.y - 1 - a.rows.n_req;
  if (r < 0) {
    build_lists<NQB, true, false>(a.rows, flags);
    return;
  }
  for (int g = blockIdx.x; g < a.tokens.n_kv_heads; g += gridDim.x) {
    decode_lists<int4, kTokenBytes>(a.tokens, g, r, flags);
    __syncthreads();   // its LDS is the next list's
  }
}

// Issued-tile accounting, one workgroup per head: for every query block of the chunk, the
// number of slash tiles (computed diagonals a <= m) and of vertical tiles (groups of 64
// gathered columns with at least one usable column).  This is the work that the head's own sets ask for, and what k_attention
// executes where a tile is one head's; tiles that heads share, and single tokens, walk the union of their heads' lists.
__global__ __launch_bounds__(256) void k_count_tiles(const int32_t* v_idx, const int32_t* v_cnt,
                                                    int32_t v_budget, const uint32_t* bm_a,
                                                    int n_words, int64_t q_start, int64_t q_len,
                                                    int64_t* tiles) {
  const int h = blockIdx.x;
  const uint32_t* A = bm_a + (int64_t)h * n_words;
  const int32_t* vi = v_idx + (int64_t)h * v_budget;
  const int vcnt = v_cnt[h];
  const int n_vt = (vcnt + 63) >> 6;
  const int mb0 = (int)(q_start / 64), n_qb = (int)((q_len + 63) / 64);
  __shared__ unsigned long long acc[2];
  if (threadIdx.x < 2) acc[threadIdx.x] = 0;
  __syncthreads();
  unsigned long long ns = 0, nv = 0;
  for (int qb = threadIdx.x; qb < n_qb; qb += blockDim.x) {
    const int m = mb0 + qb;
    for (int w = 0; w <= (m >> 5); ++w) {
      uint32_t x = A[w];
      if (w == (m >> 5) && (m & 31) != 31) x &= (2u << (m & 31)) - 1u;
      ns += __popc(x);
    }
    const int64_t rows = (q_len - 64ll * qb) < 64 ? (q_len - 64ll * qb) : 64;
    const int64_t lastp = q_start + 64ll * qb + rows - 1;
    for (int vt = 0; vt < n_vt; ++vt) {
      bool any = false;
      for (int r = 0; r < 64 && 64 * vt + r < vcnt; ++r) {
        const int j = vi[64 * vt + r];
        const int ad = m - (j >> 6);
        if (j <= lastp && ad >= 0 && !((A[ad >> 5] >> (ad & 31)) & 1u)) { any = true; break; }
      }
      nv += any;
    }
  }
  atomicAdd(&acc[0], ns);
  atomicAdd(&acc[1], nv);
  __syncthreads();
  if (threadIdx.x < 2) tiles[2 * h + threadIdx.x] = (int64_t)acc[threadIdx.x];
}

// ---------------------------------------------------------------------------------------------
// Pace keeping of the persistent launch: key blocks per sync segment.  The members of a group
// (one XCD) may be at most two segments apart, so about three segments of K and V (64 KiB per
// block at D = 128) are live in the caches at a time.  0 = automatic: 64 blocks at D = 128
// (measured best for full lists; sparse lists scale it up per head, see k_build_blocklist).
// (The tuning switches are process-wide atomics: a size query and the call it is for must see the
// same values; a call under a setting that needs more workspace than it was given is refused by
// the size check of the entry point.)
static std::atomic<int> g_sync_blocks{0};
void set_attn_segment_blocks(int blocks) { g_sync_blocks.store(blocks < 0 ? 0 : blocks, std::memory_order_relaxed); }
static int attn_sync_blocks(const vs_params& p) {
  const int forced = g_sync_blocks.load(std::memory_order_relaxed);
  if (forced > 0) {   // a power of two (rounded down): the kernel finds a block's segment with a shift
    int sb = 1;
    while (sb * 2 <= forced) sb *= 2;
    return sb;
  }
  const int per_block = kBlock * p.head_dim * 2 * 2;  // K and V of one KV head
  int sb = 1;
  while (sb * 2 * 3 * per_block <= (6 << 20)) sb *= 2;
  return sb;
}
static size_t attn_counter_bytes(const vs_params& p) {
  const int64_t n_blk = ceil_div(p.q_start + p.q_len, kBlock);
  const size_t queues = 8 * kQueueStride * sizeof(uint32_t);   // of the key-split kernel, in front
  return queues + align_up((size_t)8 * (size_t)ceil_div(n_blk, attn_sync_blocks(p)) * sizeof(uint32_t), 256);
}
// the schedule: 8 rows of at most Hq x (query tiles) group-rounds
static size_t attn_sched_bytes(const vs_params& p) {
  const size_t rounds = (size_t)p.n_q_heads * (size_t)ceil_div(p.q_len + p.q_start % kBlock, (int64_t)64 * kAttnQBlocks);
  return align_up(8 * rounds * sizeof(int32_t), 256);
}

// Key split of short chunks, and of what is left of longer ones when their units do not fill the chip evenly: a launch
// has 512 workgroup slots (256 compute units x 2; fixed, so that workspace sizes do not depend on the device).
static std::atomic<int> g_key_split{0};  // 0: automatic, 1: never, n: n ranges (still at least 16 key blocks each)
void set_attn_key_split(int n) { g_key_split.store(n < 0 ? 0 : (n > 16 ? 16 : n), std::memory_order_relaxed); }
// dense attention of one token with grouped queries: the heads of a KV group share a tile
bool attn_packed_decode(const vs_params& p, bool dense) {
  return dense && p.q_len == 1 && p.n_q_heads > p.n_kv_heads && p.n_q_heads / p.n_kv_heads <= 64 * kAttnQBlocks;
}
// How a launch is cut: queue false = the pace-keeping kernel, every unit whole (where that is asked for, and of few key blocks); else
// pieces in queues, before which attn_paced lets whole units keep pace.  Units rarely fill whole rounds
// of the 512 slots: what is left over is cut so finely that it takes a fraction of a round (28 heads; before, at most 16
// ranges and only below 256 units): 5,084 rows at 45K keys, 2.2 rounds, 4.06 -> 3.13 ms; 850 rows at 758K, 0.4 rounds in two
// ranges, 10.5 -> 8.9; 8,192 rows at 400K, 3.5 rounds, 39.5 -> 35.9; 2,400 rows at 100K 4.94 -> 3.13.  The count of rounds below
// finds the ranges of launches below a round and of short walks; the rest of longer ones is cut as finely as partial results allow.
struct AttnCut {
  bool queue;
  int32_t pack, n_hs, n_qtiles, n_units, n_whole, n_split;
  int32_t own_slots;   // slots for ranges by the lists' lengths (own_cut; 0: even ranges only)
  double steps;        // what it should take, in steps (automatic cuts)
  int64_t slots() const {
    const int64_t even = n_split > 1 ? (int64_t)(n_units - n_whole) * n_split : 0;
    return even > own_slots ? even : own_slots;
  }
};
// Few heads of 64 over many keys, with units for two whole rounds or more and at most 128 over: with index sets the whole units keep pace all the
// same, by the lists' lengths.  The queues know nothing of these, so the longest may begin last.  Clustered lists, in the queues and keeping pace:
// 8 heads, 16,512 rows at 300,032 keys (lists of 232 to 465 blocks, 8 units over) 1,300 us and 1,075, 17,536 rows (72 over) 1,297 and 1,171, 24,704 (8) 1,227 and
// 1,173; 4 heads without groups, 32,896 rows at 400,000 918 and 779.  Not for more: 18,944 rows (160 over) 1,302 and 1,282, of lists that are alike 845 and 925;
// 16 heads, 12,416 rows at 400,000 (16 over) 1,184 and 1,476.  Where lists are alike it loses: 4 heads of a group, 32,768 rows at 700,032 keys 436 and 494 (487 while
// heads of 64 kept pace everywhere), scattered ones of 8 heads 3,258 and 3,362.  Nor for dense calls, whose units are alike: 10,830 and 11,140.
static bool attn_few_over(const vs_params& p, int64_t units) {
  return p.head_dim == 64 && p.n_q_heads <= 8 && ceil_div(p.q_start + p.q_len, kBlock) >= kPaceBlocks && units > 1024 && units % 512 != 0 &&
         units % 512 <= 128;
}
static AttnCut attn_cut_as(const vs_params& p, bool dense, bool least, int forced) {
  const bool one = attn_packed_decode(p, dense);
  const int group = p.n_q_heads / p.n_kv_heads, row_pad = (int)(p.q_start % kBlock);
  const int64_t n_blk = ceil_div(p.q_start + p.q_len, kBlock);
  AttnCut c = {};
  const int64_t columns = dense ? 0 : (p.vertical_budget < p.q_start + p.q_len ? p.vertical_budget : p.q_start + p.q_len);
  c.pack = one || forced == 1 ? 1 : heads_per_tile(p.q_len, row_pad, group, n_blk, columns);
  c.n_hs = one ? 1 : (int)ceil_div(group, c.pack);
  const int64_t n_qtiles = ceil_div(one ? group : p.q_len + row_pad, (int64_t)kTileRows);
  const int64_t units = n_qtiles * p.n_kv_heads * c.n_hs;
  c.n_split = 1;
  const int64_t slots = 512;
  const bool long_walk = p.head_dim == 128 && n_blk >= kPaceBlocks;   // whole units keep pace
  // What whole rounds leave over in up to kMaxPieces ranges, of full rounds the last one: a workgroup takes the next piece when it is done with
  // one, and whole units end as differently as lists are long, rows far from the first key and XCDs fast (workgroups of full rounds
  // ended 2 to 2.5 % before the last one on average).  32,768 rows, full rounds whole and so: 28 heads at 1M keys 225.9 ms and 221.4; 40 heads at
  // 262,144 146.7 and 142.3; 16,384 rows of 28 at 16,384 dense 2,165 us and 1,766, clustered at 50K 7,562 and 7,046.  Full rounds of more than
  // kMaxQueueUnits units that do not keep pace stay whole and come out of the queues: 28 heads at 65,536 dense 20.98 ms keeping pace, 20.33 so,
  // clustered 16.21 and 15.12.  With their last round cut, too, the dense ones would take 19.57; they are not
  // because calls of this size have always done without room for partial results (0.24 MB, and 137 then) and are held to it.  No
  // measurement draws the line at kMaxQueueUnits.
  // Walks that the budgets make short (heads of 64, 256K keys and more) in half as many: the partial results take as much of the caches and of the time
  // as they save.  4 heads with 256 offsets, clustered: 30,000 rows at 700,000 keys 418, 610, 661 us (three sets of keys), 401, 602, 660 so; 32,768 rows at 1M 484,
  // 639, 671 and 483, 627, 664 (482, 611, 674 whole); with 700 offsets, 8 heads, 15,000 rows at 500,000 1,443, 1,014, 1,090 and 1,544, 1,019, 1,142.
  const auto cut_rest = [&](int64_t rest) {
    const int64_t listed = dense ? n_blk : 2 * (int64_t)p.slash_budget + 1 + 2 * ((columns + 63) / 64);
    const bool short_lists = p.head_dim == 64 && n_blk >= kPaceBlocks && listed < kShortList;
    int64_t n = (short_lists ? kMaxPieces / 2 : kMaxPieces) / rest;
    n = n < n_blk / 16 ? n : n_blk / 16;
    c.queue = true;
    c.n_qtiles = (int32_t)n_qtiles;
    c.n_units = (int32_t)units;
    c.n_whole = (int32_t)(units - rest);
    c.n_split = (int32_t)(n < kMaxSplit ? n : kMaxSplit);
  };
  const bool fine = forced == 0 && !least && c.pack == 1 && n_blk >= 64 && units > slots && units < kMaxAskedUnits;
  if (fine && (units > kMaxQueueUnits || units % slots == 0)) {
    if (units % slots != 0 || units <= kMaxQueueUnits || long_walk) {
      cut_rest(units % slots ? units % slots : slots);
    } else {
      c.queue = true;
      c.n_qtiles = (int32_t)n_qtiles;
      c.n_units = c.n_whole = (int32_t)units;
    }
    return c;
  }
  if (forced == 1 || units > (forced > 1 ? kMaxAskedUnits : kMaxQueueUnits)) return c;
  c.n_qtiles = (int32_t)n_qtiles;
  c.n_units = (int32_t)units;
  c.n_whole = 0;
  if (forced > 1) {
    c.n_split = (int)(forced < n_blk / 16 ? forced : n_blk / 16);
    c.queue = c.n_split > 1;
    if (!c.queue) { c.pack = 1; c.n_hs = group; c.n_split = 1; }
    return c;
  }
  // Steps of a whole walk: all key blocks, with index sets too (so that the cut is the same as without them, and with every
  // offset selected the results are, unless many columns put fewer heads into a tile)
  const double steps = (double)n_blk;
  // Rounds of 512 pieces, in steps.  A piece costs kPieceSteps beside its walk; writing and folding partial results
  // costs about eight steps per 512 pieces and kFoldSteps per piece of a row, and the second launch three.  Ranges of two
  // steps where that is the least: short calls wait for their longest piece.  With eight at least, 12 rows of 28 heads at 956
  // keys 27.1 us -> 16.2 with two, 8 rows at 19,695 31.5 -> 28.5, 185 rows of 8 heads at 9,060 27.5 -> 25.1, 32 rows at 2,048 with
  // index sets 58.4 -> 52.3; over 100 calls of 2 to 3,000 rows below 60,000 keys 4.7 % less, the slowest 2.7 % more.
  double best = -1.0;
  // whole rounds kept: all, all but one, none
  const int64_t full = units / slots * slots, keep[3] = {full, full - slots, 0};
  for (int x = 0; x < 3; ++x) {
    const int64_t whole = keep[x];
    if (x > 0 && (whole < 0 || whole == keep[x - 1])) continue;
    const int64_t rest = units - whole;
    for (int64_t n = 1; n <= kMaxSplit; ++n) {
      if (n > 1 && (rest == 0 || rest * n > kMaxPieces || steps / (double)n < kMinSteps)) break;
      const int64_t pieces = rest * n;
      double cost = (double)(whole / slots) * (steps + kPieceSteps) +
                    (2 * pieces <= slots ? kAloneRate : 1.0) * (double)ceil_div(pieces, slots) * (steps / (double)n + kPieceSteps);
      if (n > 1) cost += 3.0 + kFoldSteps * (double)n + 8.0 * (double)pieces / (double)slots;
      if (best < 0 || cost < best) {
        best = c.steps = cost;
        c.n_whole = (int32_t)whole;
        c.n_split = (int32_t)n;
      }
    }
  }
  if (c.n_split == 1) c.n_whole = c.n_units;
  c.queue = units <= slots || best < 0.97 * (double)ceil_div(units, slots) * (steps + kPieceSteps);
  if (!c.queue) { c.pack = 1; c.n_hs = group; c.n_split = 1; }
  // Partial rounds, too, are cut finely where the count above would not.  Long walks, 28 heads, 512, 1,024 and 2,048 pieces at most: 8,192 rows
  // at 400K keys 35.2 ms, 34.5, 34.1, with DCA 36.6, 35.8, 35.3; 6,822 rows at 858K (2.95 rounds) 50.2 whole, 48.7.  Shorter ones: 13,307 rows
  // at 31K keys 4,850 us whole, 4,300; 4,096 clustered ones at 8,192 521 and 430; 3,128 of 40 heads at 63K in a few ranges 4,116, 4,043.
  // Below 1,024 key blocks the ranges that the count makes are as good (40 calls: 2 % either way), and smaller; and ranges of one
  // round go, with index sets, by the lists' lengths where no whole units keep pace before them.
  const bool one_round = c.n_split > 1 && (c.n_units - c.n_whole) * (int64_t)c.n_split <= slots && n_blk >= 64 * (int64_t)c.n_split;
  if (fine && units % slots != 0 && (c.n_split == 1 || long_walk || attn_few_over(p, units) || (n_blk >= 1024 && !one_round))) {
    cut_rest(units % slots);
    return c;
  }
  // Uneven ranges where pieces are long enough for a launch that finds them (5 to 11 us; a range of 64 blocks takes 120, less where lists
  // are short); whole units below a round, which need the fold then as well, from 1,024 blocks on.  Not with one query tile: even ranges
  // of the heads of a KV group lie at the same keys, which the XCD's L2 reads once for them (64 rows at 1M keys, lists that differ by 8 %:
  // 2,024 us, 2,101 uneven).  Nor where the even cut has several rounds: a slot takes the next piece when it is done, and the far
  // pieces, which come last, are the short ones (11,109 clustered rows at 500K keys 16.9 ms, 17.2 uneven).
  if (c.queue && !dense && n_qtiles > 1 && n_blk >= 64 * (int64_t)c.n_split && (c.n_split > 1 || n_blk >= 1024) &&
      (c.n_units - (c.n_split > 1 ? c.n_whole : 0)) * (int64_t)c.n_split <= slots) {
    if (c.n_split == 1) c.n_whole = 0;   // (units fit a round)
    const int lists = p.n_kv_heads * c.n_hs;
    if (cut_segment_of(c.n_units - 1, c.n_qtiles, lists) - cut_segment_of(c.n_whole, c.n_qtiles, lists) < kOwnSegments) {
      const int64_t rounds = ceil_div(8 * (int64_t)(c.n_units - c.n_whole), slots);   // about eight pieces of a unit
      c.own_slots = (int32_t)(slots * (rounds < kOwnRounds ? rounds : kOwnRounds));
    } else if (c.n_split == 1) {
      c.n_whole = c.n_units;
    }
  }
  return c;
}
// least: without uneven and without the finest ranges, whose partial results are most of the workspace (28 heads of 128: 2,000 rows at
// 150,000 keys 137 MB of it, 0.3 without; 8,192 rows at 400,000 keys 134 MB and 35)
static AttnCut attn_cut(const vs_params& p, bool dense, bool least = false) {
  AttnCut c = attn_cut_as(p, dense, least, g_key_split.load(std::memory_order_relaxed));
  if (least && c.own_slots) {
    c.own_slots = 0;
    if (c.n_split == 1) c.n_whole = c.n_units;
  }
  return c;
}
// Partial results of the cut units: a tile's rows for every range.
size_t attn_split_bytes(const vs_params& p, bool dense, bool least) {
  const AttnCut c = attn_cut(p, dense, least);
  if (!c.queue || c.slots() == 0) return 0;
  const size_t rows = (size_t)c.slots() * kTileRows, own = c.own_slots ? 256 + kMaxPieces * (sizeof(int2) + sizeof(OwnPiece)) : 0;
  return align_up(rows * p.head_dim * sizeof(float), 256) + align_up(rows * 2 * sizeof(float), 256) + own;
}
// counters, schedule
size_t attn_sync_bytes(const vs_params& p) { return attn_counter_bytes(p) + attn_sched_bytes(p); }

// out = sum_s O_s 2^(m_s - M) / sum_s l_s 2^(m_s - M), M = max_s m_s; D / 4 lanes per row of a tile,
// pieces folded in ascending order (fixed, so the result is run-to-run identical).
// One workgroup folds 1024 / D rows of a unit at a time; those of a batch, whose cut units only the device knows, take the next
// ones until none are left (a grid for as many units as there may be: 26 us for 1,500 requests none of which was cut, 4 now),
// and up to four of a unit in a row where there are more than workgroups, because finding them takes as long as folding a few
// pieces.  Bound by latency: a row's lanes read a reference and a sum each (all pieces' at once) while the first eight accumulators are
// under way, and the weights go around through the LDS.  (Every lane reading all references, and after them everything again,
// eight pieces at a time: 5 to 10 us for 40 to 60 pieces of a row, 3 to 6 so.)
template <int D>
constexpr int combine_parts() { return kTileRows / (1024 / D); }   // per unit
constexpr int kCombineGrid = 2048;   // workgroups for a batch at most
// n_wg: workgroups that share in it
template <int D, bool BATCH, bool OWN>
__device__ __forceinline__ void attn_fold(const AttnArgs& a0, const int n_wg) {
  constexpr int LR = D / 4;            // lanes per row
  constexpr int WPU = combine_parts<D>();
  __shared__ __attribute__((aligned(16))) float w_s[256 / LR][kMaxSplit];
  const int d = 4 * (threadIdx.x % LR);
  const int n_tasks = (BATCH ? __builtin_amdgcn_readfirstlane(a0.plan[a0.n_req].cut) : a0.n_units - a0.n_whole) * WPU;
  int run = 1;   // consecutive parts of a unit
  while (BATCH && run < 4 && n_tasks > run * n_wg) run *= 2;
  for (int task = blockIdx.x * run; task < n_tasks; task += n_wg * run) {
  int e = task / WPU;
  AttnArgs a = a0;
  if constexpr (BATCH) {
    const int r = batch_find<&BatchPlan::cut>(a0.plan, a0.n_req, e);
    e -= __builtin_amdgcn_readfirstlane(a0.plan[r].cut);
    if (!batch_view(a0, r, a)) continue;
  }
  const int n_fold = a.n_units - a.n_whole;
  if (e >= n_fold) continue;
  int g, h, qt;
  unit_of(a, a.n_whole + e, g, h, qt);
  int n_sp = a.n_split, slot0 = BATCH ? e + a.first_slot : e, slot_step = n_fold;
  if constexpr (OWN) {
    if (__builtin_amdgcn_readfirstlane(*a.own_n) > 0) {
      const int2 own = a.own_units[e];
      n_sp = __builtin_amdgcn_readfirstlane(own.x);
      slot0 = __builtin_amdgcn_readfirstlane(own.y);
      slot_step = 1;
    }
    if (n_sp == 1) continue;   // (its walk was whole)
  }
  for (int part = task % WPU; part < task % WPU + run; ++part) {
  // (the row of the tile as k_attention deals them out)
  const int lrow = part * (1024 / D) + threadIdx.x / LR;
  const int wv = lrow >> 5;
  int t = wv >> 1, th = 0, il0 = (wv & 1) << 5;
  if (a.pack > 1) {
    t = 0;
    th = a.pack == 4 ? wv : wv >> 1;
    il0 = a.row_pad + (a.pack == 4 ? 0 : il0);
  }
  const int64_t row = (int64_t)qt * kTileRows + 64 * t + il0 + (lrow & 31) - a.row_pad;
  if (row < 0 || row >= a.q_rows || h - g * a.group + th >= a.group) continue;
  const int hw = h + th;
  const int64_t at = (int64_t)slot0 * kTileRows, step = (int64_t)slot_step * kTileRows;
  constexpr int U = 8, NB = kMaxSplit / LR;   // pieces whose accumulators are under way together; references per lane
  const float* const po = a.part_o + at * D + (lrow * D + d);   // (at: the same in every lane)
  f32x4 o[U];
  auto fetch = [&](int sp) {
#pragma unroll
    for (int u = 0; u < U; ++u) o[u] = *(const f32x4*)(po + step * (sp + u < n_sp ? sp + u : n_sp - 1) * D);
  };
  fetch(0);
  // lane x of the row: pieces x, LR + x, ...; their weights wait in LDS (a row's lanes are of one wave)
  const int lr = threadIdx.x % LR;
  float* const ws = &w_s[threadIdx.x / LR][0];
  float m[NB], l[NB], M = -INFINITY, L = 0.f;
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    m[b] = -INFINITY;
    l[b] = 0.f;
    if (b * LR < n_sp && b * LR + lr < n_sp) {
      const float2 ml = *(const float2*)(a.part_ml + 2 * (at + lrow + step * (b * LR + lr)));
      m[b] = ml.x;
      l[b] = ml.y;
    }
    M = fmaxf(M, m[b]);
  }
#pragma unroll
  for (int x = 1; x < LR; x <<= 1) M = fmaxf(M, __shfl_xor(M, x));
  const float M0 = M == -INFINITY ? 0.f : M;
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const float w = __builtin_amdgcn_exp2f(m[b] - M0);   // (a piece without live keys: weight 0, and zeros in its slot)
    L += l[b] * w;
    if (b * LR < n_sp) ws[b * LR + lr] = w;         // (0 behind the last piece)
  }
#pragma unroll
  for (int x = 1; x < LR; x <<= 1) L += __shfl_xor(L, x);
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma clang loop unroll(disable)
  for (int sp = 0; sp < n_sp; sp += U) {
    if (sp > 0) fetch(sp);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float w = ws[sp + u];
#pragma unroll
      for (int x = 0; x < 4; ++x) acc[x] += o[u][x] * w;
    }
  }
  const float inv = L > 0.f ? 1.0f / L : 0.f;
#pragma unroll
  for (int x = 0; x < 4; ++x) acc[x] *= inv;
  *(bf16x4*)(a.out + row * a.o_stride_tok + (int64_t)hw * a.o_stride_head + d) = __builtin_convertvector(acc, bf16x4);
  if (a.lse && d == 0)
    a.lse[(int64_t)hw * a.q_rows + row] = L > 0.f ? (M + __builtin_amdgcn_logf(L)) * kLn2 : -INFINITY;
  }  // parts
  }  // tasks
}
template <int D, bool BATCH = false, bool OWN = false>
__global__ __launch_bounds__(256) void k_attn_combine(const AttnArgs a) { attn_fold<D, BATCH, OWN>(a, gridDim.x); }
// The folds of a batch, the first n_rows workgroups those of its longer requests, then one per request and head those of its tokens.
template <int D>
__global__ __launch_bounds__(256) void k_mixed_combine(const MixedArgs a, const int n_rows) {
  if ((int)blockIdx.x < n_rows) {
    attn_fold<D, true, false>(a.rows, n_rows);
    return;
  }
  const int x = (int)blockIdx.x - n_rows, r = x / a.tokens.n_q_heads;
  decode_fold<D, 4, D == 128 ? 0 : 1, int4>(a.tokens, x - r * a.tokens.n_q_heads, r);
}

// The pieces of an uneven cut (own_cut), one workgroup.  They lie in `most` slices, one after the other: in slice z those of the segments
// in turn whose range falls into it, about z n / most of a unit's ranges lie before it.  So pieces that are walked at the same time read
// the same part of the cache, as with the even cut.  A range holds as many entries as the others of its unit: of equal distances
// the near ones have twice the entries of the far ones where slashes are clustered.  (In the attention kernel itself, 2 us of every
// workgroup, the code spilled 31 registers of the walk.)
__global__ __launch_bounds__(1024) void k_attn_pieces(const AttnArgs a) {
  __shared__ int32_t n_s[kOwnSegments], cnt_s[kOwnSegments], e0_s[kOwnSegments], slot_s[kOwnSegments], pieces_s, most_s;
  __shared__ int32_t reach_s[kMaxPieces], table[kMaxPieces];   // of a cut unit: entries up to its last block; of a piece: unit, range
  const int tid = threadIdx.x, lists = a.n_q_heads / a.group * a.n_hs, seg0 = cut_segment_of(a.n_whole, a.n_qtiles, lists);
  if (tid < 64) {
    int n, cnt, slot, pieces, most, list, e0;
    own_cut(a, tid, n, cnt, slot, pieces, most);
    cut_segment(a, tid, list, e0, cnt);
    n_s[tid] = n; cnt_s[tid] = cnt; e0_s[tid] = e0; slot_s[tid] = slot;
    if (tid == 0) { pieces_s = pieces; most_s = most; *a.own_n = pieces; }
  }
  __syncthreads();
  const int pieces = pieces_s, most = most_s, n_cut = a.n_units - a.n_whole;
  if (pieces == 0) return;
  const int n_seg = cut_segment_of(a.n_units - 1, a.n_qtiles, lists) - seg0 + 1;
  auto list_of = [&](int e, int& cc_last) -> const uint32_t* {
    int g, h, qt;
    unit_of(a, e, g, h, qt);
    cc_last = (int)(a.q_start / 64) + qt * kAttnQBlocks + kAttnQBlocks - 1;
    return a.ent + (int64_t)(g * a.n_hs + (h - g * a.group) / a.pack) * a.ent_stride;
  };
  for (int j = tid; j < n_cut; j += 1024) {
    const int e = a.n_whole + j, x = cut_segment_of(e, a.n_qtiles, lists) - seg0;
    a.own_units[j] = make_int2(n_s[x], slot_s[x] + (e - e0_s[x]) * n_s[x]);
    int cc_last;
    const uint32_t* const ent = list_of(e, cc_last);
    int lo = 0, hi = (int)a.ent_len - 1;   // the last entry is a sentinel
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if ((int)(ent[mid] >> 4) <= cc_last) lo = mid + 1;
      else hi = mid;
    }
    reach_s[j] = lo;
  }
  // (about z n / most, sometimes one more than its whole part; what the places need is that it is 0 at 0, n at `most` and rises by 0 or 1
  // from slice to slice, which holds for every n <= most <= 128, and as far as most^2 < 65536)
  static_assert(kMaxSplit * kMaxSplit < 65536, "the quotient below");
  auto before = [&](int z, int n) -> int { return (z * n * ((65535 + most) / most)) >> 16; };
  for (int t = tid; t < n_seg * most; t += 1024) {
    const int sp = t / n_seg, x = t - sp * n_seg, n = n_s[x];
    if (sp >= n) continue;
    int z = sp * most / n;
    while (before(z + 1, n) <= sp) ++z;
    while (before(z, n) > sp) --z;
    int at = 0;
    for (int y = 0; y < n_seg; ++y) at += cnt_s[y] * (y < x ? before(z + 1, n_s[y]) : before(z, n_s[y]));
    for (int i = 0; i < cnt_s[x]; ++i) table[at + i] = (e0_s[x] - a.n_whole + i) | sp << 16;
  }
  __syncthreads();
  for (int v = tid; v < pieces; v += 1024) {
    const int j = table[v] & 0xFFFF, sp = table[v] >> 16, e = a.n_whole + j, x = cut_segment_of(e, a.n_qtiles, lists) - seg0, n = n_s[x];
    int cc_last;
    const uint32_t* const ent = list_of(e, cc_last);
    const int all = reach_s[j], each = (all + n - 1) / n, from = sp * each, to = from + each < all ? from + each : all;
    OwnPiece o = {};
    o.unit = e; o.sp = sp; o.n_sp = n;
    o.slot = slot_s[x] + (e - e0_s[x]) * n + sp;
    o.cc_lo = from < to ? (int)(ent[from] >> 4) : 0;
    o.cc_hi = from < to ? (int)(ent[to - 1] >> 4) : -1;
    a.own_pieces[v] = o;
  }
}

// Which group takes which group-round.  Heads differ in the length of their block lists (by a
// factor of almost two in the 1M workloads), so dealing the rounds out in turn leaves some
// groups idle at the end.  The rounds are weighed (list length x number of key blocks the
// tiles can reach), sorted, and given one by one to the group with the least work so far; a
// group works through its rounds in that (descending) order.  One workgroup; only the timing
// of the attention launch depends on the result.
constexpr int kSchedMax = 8192;  // rounds the sort is done for (beyond it: dealt out in turn)
static std::atomic<int> g_sched_in_turn{0};
void set_attn_schedule_in_turn(int on) { g_sched_in_turn.store(on ? 1 : 0, std::memory_order_relaxed); }
__global__ __launch_bounds__(1024) void k_attn_schedule(const AttnArgs a, int32_t* sched, int in_turn) {
  __shared__ float w[kSchedMax];
  __shared__ uint16_t order[kSchedMax];
  __shared__ float avg_ent;
  const int tid = threadIdx.x, n_gr = a.n_gr;
  if (n_gr > kSchedMax || in_turn) {
    for (int x = tid; x < 8 * n_gr; x += 1024) {
      const int g = x / n_gr, r = x - g * n_gr;
      sched[x] = r * 8 + g < n_gr ? r * 8 + g : -1;
    }
    return;
  }
  if (tid < 64) {
    uint64_t sum = 0;
    for (int h = tid; h < a.n_q_heads; h += 64) sum += a.bm_a[(int64_t)h * a.bm_stride + a.bm_words - 2] & kListMask;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) sum += __shfl_xor((unsigned long long)sum, d);
    if (tid == 0) avg_ent = (float)((double)sum / a.n_q_heads);
  }
  __syncthreads();
  const int n_full_gr = a.n_full * a.n_q_heads;
  const int mb = (int)(a.q_start / 64);
  for (int gr = tid; gr < n_gr; gr += 1024) {
    float ent, reach;
    if (gr < n_full_gr) {
      const int h = gr % a.n_q_heads, c = a.n_full - 1 - gr / a.n_q_heads;
      ent = (float)(a.bm_a[(int64_t)h * a.bm_stride + a.bm_words - 2] & kListMask);
      reach = (float)(mb + 2 * (a.n_rem + c * a.members + a.members / 2) + 2);  // key blocks before the chunk's middle tile
    } else {
      ent = avg_ent;  // leftover tiles of several heads
      reach = (float)(mb + a.n_rem + 2);
    }
    w[gr] = ent * reach;
  }
  __syncthreads();
  for (int gr = tid; gr < n_gr; gr += 1024) {
    const float mine = w[gr];
    int rank = 0;
    for (int j = 0; j < n_gr; ++j) rank += (w[j] > mine || (w[j] == mine && j < gr)) ? 1 : 0;
    order[rank] = (uint16_t)gr;
  }
  __syncthreads();
  // Lane g (and g + 8, ...) of the first wave keeps the load of group g.  A group's key is its load's float
  // image (loads are >= 0, so the images are ordered like them) with the group in the low three bits: the
  // least loaded group is three lane exchanges away.  The 64 next rounds wait in registers.  (One thread
  // walking eight loads in memory took 0.65 us per round, 104 us for the 160 rounds of a 40-head chunk, now 26.)
  if (tid < 64) {
    const int g = tid & 7;
    float load = 0.f;
    int cnt = 0;
    for (int i0 = 0; i0 < n_gr; i0 += 64) {
      const int mine = i0 + tid < n_gr ? (int)order[i0 + tid] : 0;
      const float wmine = w[mine];
      for (int i = 0; i < 64 && i0 + i < n_gr; ++i) {
        const uint32_t key = (__float_as_uint(load) & ~7u) | (uint32_t)g;
        auto least = [](uint32_t x, uint32_t y) { return x < y ? x : y; };
        uint32_t m = least(key, (uint32_t)__builtin_amdgcn_mov_dpp((int)key, 0xB1, 0xF, 0xF, true));  // lane ^ 1
        m = least(m, (uint32_t)__builtin_amdgcn_mov_dpp((int)m, 0x4E, 0xF, 0xF, true));               // lane ^ 2
        m = least(m, (uint32_t)__builtin_amdgcn_mov_dpp((int)m, 0x141, 0xF, 0xF, true));              // the other four of eight
        const int gr = __builtin_amdgcn_readlane(mine, i);
        const float wt = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(wmine), i));
        if (key == m) {
          if (tid < 8) sched[g * n_gr + cnt] = gr;
          ++cnt;
          load += wt;
        }
      }
    }
    if (tid < 8)
      for (int r = cnt; r < n_gr; ++r) sched[g * n_gr + r] = -1;
  }
}

// Per-device set-up, done once for each device a launch is made on (with that device current):
// its number of compute units, and the opt-in of every attention instantiation to more than
// 64 KiB of LDS per workgroup (a function attribute, held per device by the runtime).
constexpr int kMaxDevices = 64;
static hipError_t attn_device_setup(int* n_cu_out) {
  static std::mutex mu;
  static int cu_of[kMaxDevices] = {0};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (cu_of[dev] == 0) {
    constexpr int NQB = kAttnQBlocks;
    int cu = 0;
    e = hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    if (cu < 1) return hipErrorInvalidDevice;
    constexpr int lds128 = attn_lds_bytes<128>(), lds64 = attn_lds_bytes<64>();
    const struct { const void* kernel; int lds; } fns[] = {
        {reinterpret_cast<const void*>(&k_attention<128, NQB, false, false>), lds128},
        {reinterpret_cast<const void*>(&k_attention<64, NQB, false, false>), lds64},
        {reinterpret_cast<const void*>(&k_attention<128, NQB, true, false>), lds128},
        {reinterpret_cast<const void*>(&k_attention<64, NQB, true, false>), lds64},
        {reinterpret_cast<const void*>(&k_attention<128, NQB, false, true>), lds128},
        {reinterpret_cast<const void*>(&k_attention<64, NQB, false, true>), lds64},
        {reinterpret_cast<const void*>(&k_attention<128, NQB, true, true>), lds128},
        {reinterpret_cast<const void*>(&k_attention<64, NQB, true, true>), lds64},
        {reinterpret_cast<const void*>(&k_attention<128, NQB, false, true, true>), lds128},
        {reinterpret_cast<const void*>(&k_attention<64, NQB, false, true, true>), lds64},
        {reinterpret_cast<const void*>(&k_attention_own<128, NQB, false>), lds128},
        {reinterpret_cast<const void*>(&k_attention_own<64, NQB, false>), lds64},
        {reinterpret_cast<const void*>(&k_attention_own<128, NQB, true>), lds128},
        {reinterpret_cast<const void*>(&k_attention_own<64, NQB, true>), lds64},
        {reinterpret_cast<const void*>(&k_attention_paced<128, NQB, false>), lds128},
        {reinterpret_cast<const void*>(&k_attention_paced<128, NQB, true>), lds128},
        {reinterpret_cast<const void*>(&k_attention_paced<64, NQB, false>), lds64},
        {reinterpret_cast<const void*>(&k_attention_paced<64, NQB, true>), lds64},
        {reinterpret_cast<const void*>(&k_attention_mixed<128, NQB>), lds128},
        {reinterpret_cast<const void*>(&k_attention_mixed<64, NQB>), lds64},
        {reinterpret_cast<const void*>(&k_attn_short<128, false>), short_lds_bytes<128>()},
        {reinterpret_cast<const void*>(&k_attn_short<64, false>), short_lds_bytes<64>()},
        {reinterpret_cast<const void*>(&k_attn_short<128, true>), short_lds_bytes<128>()},
        {reinterpret_cast<const void*>(&k_attn_short<64, true>), short_lds_bytes<64>()},
        {reinterpret_cast<const void*>(&k_attn_short<128, true, true>), short_lds_bytes<128>()},
        {reinterpret_cast<const void*>(&k_attn_short<64, true, true>), short_lds_bytes<64>()}};
    for (const auto& f : fns) {
      e = hipFuncSetAttribute(f.kernel, hipFuncAttributeMaxDynamicSharedMemorySize, f.lds);
      if (e != hipSuccess) return e;
    }
    cu_of[dev] = cu;
  }
  *n_cu_out = cu_of[dev];
  return hipSuccess;
}

// Resident workgroups per XCD: two fit a compute unit
static int attn_members(int n_cu) {
  const int members = ((4 / kAttnQBlocks) * n_cu) / 8;
  return members < 1 ? 1 : members;
}
// Whole units of a cut launch that keep pace, before the pieces of the others in the same launch (see launch_attention).
static bool attn_paced(const AttnCut& c, const vs_params& p, bool dense, int members) {
  return c.queue && c.n_split > 1 && c.n_whole > 0 && !c.own_slots && c.pack == 1 && members == kRun &&
         ceil_div(p.q_start + p.q_len, kBlock) >= kPaceBlocks && (p.head_dim == 128 || (!dense && attn_few_over(p, c.n_units)));
}
// Dense launches of no more pieces than workgroups need neither a list (every block is in it) nor cleared counters (nobody takes
// a second piece): the list builder is not launched.  34 rows of 28 heads at 11,126 keys 34.5 us -> 31.3, the fold's share
// of it included; rows of 2 to 391 at 600 to 50,000 keys gain 2 to 11 %.
static bool attn_listless(const vs_params& p, bool dense, const AttnCut& c, int members) {
  return dense && c.queue && !attn_paced(c, p, dense, members) &&
         c.n_whole + (int64_t)(c.n_units - c.n_whole) * c.n_split <= 8 * (int64_t)members;
}

// Offsets of a tile's heads that a workgroup looks through by itself; beyond, it reads the bitmaps of k_build_blocklist.  The launch against the offsets,
// 28 heads of 128 and 16 to 32 rows: 16,384 offsets 31.7 us with lists and 27.2 without, 32,768 46.0 and 41.7, 64,000 43.4 and 43.2, 80,000 53.3 and 54.6, 131,072 71.5
// and 76.8 (and 72.9 in k_attention with lists); 17,000 of 8 heads of 64 30.4 and 26.6.
constexpr int64_t kShortOffsets = 65536;
static bool attn_short_listed(const vs_params& p, const AttnCut& c) {
  const int64_t n_k = p.q_start + p.q_len;
  return c.pack * (p.slash_budget < n_k ? p.slash_budget : n_k) > kShortOffsets;
}
// Ranges per unit of a call that k_attn_short takes (0: it does not): at most one workgroup per compute unit, and where it takes less
// time than the ranges of `c`, by two sums fitted (in us) to both kernels over 120 dense calls of 2 to 3,000 rows and 512 to 32,000 keys
// (they are off by 2.7 and 5 % on average, 10 and 13 at most, those of attn_cut by 5 and 7; what they choose is 0.2 % behind the
// faster one, at most 1 % slower than before, and on average 16 % faster for heads of 64 and 10 for 128).  With index sets there is a
// launch less besides (4.5 us), which the choice leaves out, so that with every offset selected a call goes the way of the dense one (where columns
// do not have it put fewer heads into a tile, see heads_per_tile).
static int attn_short(const vs_params& p, bool dense, bool dca, const AttnCut& c) {
  const int64_t n_blk = ceil_div(p.q_start + p.q_len, kBlock);
  if (dca || !c.queue || c.own_slots || attn_packed_decode(p, dense) || n_blk > kShortBlocks || c.n_qtiles >= kRun || c.n_units > 256) return 0;
  if (g_key_split.load(std::memory_order_relaxed) != 0 || (c.n_split > 1 && c.n_whole > 0)) return 0;
  // (with lists, too, only where it is the dense call's way)
  if (!dense && attn_short_listed(p, c) && c.pack != heads_per_tile(p.q_len, (int)(p.q_start % kBlock), p.n_q_heads / p.n_kv_heads, n_blk, 0)) return 0;
  const bool wide = p.head_dim == 128;
  double least = wide ? 1.6 + 1.28 * c.steps : 3.8 + 1.03 * c.steps;
  int best = 0;
  for (int n = 1; n <= c.n_split && n * c.n_units <= 256; ++n) {   // (no more ranges than before: the workspace is as large)
    const int64_t range = ceil_div(n_blk + 1, n);
    if (range > kShortRange) continue;
    const double full = n * c.n_units / 256.0, steps = (double)ceil_div(range, kShortSets);
    double cost = wide ? 5.5 + (1.06 + 0.82 * full) * steps + 3.2 * full : 4.2 + (1.15 + 0.14 * full) * steps + 2.5 * full;
    if (n > 1) cost += wide ? 4.7 : 4.2 + 0.09 * n;
    if (cost < least) { best = n; least = cost; }
  }
  return best;
}
// One list per head, or per tile of packed heads (one for all heads when dense); attn: for the attention launch with the
// counters at sync_ws, which are cleared on the way (null: for k_count_tiles, which packs nothing and has none to clear).
hipError_t launch_build_blocklist(const vs_params& p, const int32_t* s_idx, const int32_t* s_cnt,
                                  const int32_t* v_cnt, bool dense, bool dca, const BlockList& bl, void* sync_ws, hipStream_t st) {
  const int64_t n_k = p.q_start + p.q_len;
  AttnCut c = {};
  if (sync_ws) {
    c = attn_cut(p, dense);
    int n_cu = 0;
    const hipError_t e = attn_device_setup(&n_cu);
    if (e != hipSuccess) return e;
    if ((attn_short(p, dense, dca, c) && (dense || !attn_short_listed(p, c))) || attn_listless(p, dense, c, attn_members(n_cu))) return hipSuccess;
  }
  ListArgs a = {};
  a.s_idx = s_idx; a.s_cnt = s_cnt; a.v_cnt = v_cnt; a.s_budget = p.slash_budget;
  a.dense = dense;
  a.n_blk = (int)ceil_div(n_k, kBlock);
  a.n_words = (int)bl.words; a.ent_stride = (int)bl.ent_stride;
  a.bm_a = bl.bm_a; a.ent = bl.ent;
  a.n_heads = p.n_q_heads; a.group = p.n_q_heads / p.n_kv_heads;
  a.pack = c.queue ? c.pack : 1;
  a.zero = (uint32_t*)sync_ws;
  a.n_zero = sync_ws ? (int)(attn_counter_bytes(p) / sizeof(uint32_t)) : 0;
  const unsigned parts = dense ? (unsigned)ceil_div(bl.ent_stride, kBlDensePart) : 1u;
  const unsigned lists = dense ? 1u : (unsigned)(p.n_kv_heads * ceil_div(a.group, a.pack));
  if (!dense && a.n_blk > 64 * kBlBallots)
    hipLaunchKernelGGL((k_build_blocklist<kAttnQBlocks, false, true>), dim3(lists, parts), dim3(kBlThreads), 0, st, a);
  else
    hipLaunchKernelGGL((k_build_blocklist<kAttnQBlocks, false>), dim3(lists, parts), dim3(kBlThreads), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_attention(const vs_params& p, const void* q, const DcaArgs* dca, const void* k, const void* v,
                            const IndexSets& sets, bool dense,
                            const BlockList& bl, void* out, float* lse, void* sync_ws, void* split_ws, bool least,
                            hipStream_t st) {
  constexpr int NQB = kAttnQBlocks;
  if (!sync_ws) return hipErrorInvalidValue;
  AttnArgs a;
  a.q = (const __bf16*)q; a.k = (const __bf16*)k; a.v = (const __bf16*)v;
  a.q_succ = dca ? (const __bf16*)dca->q_succ : nullptr;
  a.q_inter = dca ? (const __bf16*)dca->q_inter : nullptr;
  a.dca_cblk = dca ? (int32_t)(dca->chunk / kBlock) : 0;
  a.dca_wblk = dca ? (int32_t)(dca->window / kBlock) : 0;
  a.out = (__bf16*)out; a.lse = lse;
  a.q_stride_tok = p.q_stride_tok; a.q_stride_head = p.q_stride_head;
  a.k_stride_tok = p.k_stride_tok; a.k_stride_head = p.k_stride_head;
  a.v_stride_tok = p.v_stride_tok; a.v_stride_head = p.v_stride_head;
  a.o_stride_tok = p.o_stride_tok; a.o_stride_head = p.o_stride_head;
  a.bm_a = bl.bm_a; a.ent = bl.ent;
  a.bm_stride = dense ? 0 : bl.words;
  a.bm_words = (int32_t)bl.words;
  a.ent_stride = dense ? 0 : bl.ent_stride;
  a.ent_len = bl.ent_stride;
  a.v_idx = dense ? nullptr : sets.v_idx;
  a.v_budget = p.vertical_budget;
  a.n_q_heads = p.n_q_heads; a.n_kv_heads = p.n_kv_heads; a.group = p.n_q_heads / p.n_kv_heads;
  a.row_pad = (int32_t)(p.q_start % kBlock);
  a.q_start = p.q_start - a.row_pad;
  a.q_len = p.q_len + a.row_pad;
  a.q_rows = p.q_len;
  a.n_k = p.q_start + p.q_len;
  a.same_pos = 0; a.pos_in_block = 0;
  if (attn_packed_decode(p, dense)) {
    // rows = the G heads of a KV group, "heads" = the KV heads: the strides say so
    const int G = p.n_q_heads / p.n_kv_heads;
    a.q_stride_tok = p.q_stride_head; a.q_stride_head = (int64_t)G * p.q_stride_head;
    a.o_stride_tok = p.o_stride_head; a.o_stride_head = (int64_t)G * p.o_stride_head;
    a.n_q_heads = p.n_kv_heads; a.group = 1;
    a.same_pos = 1; a.pos_in_block = a.row_pad;
    a.row_pad = 0; a.q_len = G; a.q_rows = G;   // lse [Hkv][G] is the caller's [Hq][1]
  }
  a.n_qtiles = (int)ceil_div(a.q_len, 64 * NQB);
  a.scale_log2 = p.softmax_scale * kLog2e;
  const AttnCut cut = attn_cut(p, dense, least);
  a.pack = cut.pack; a.n_hs = cut.n_hs;
  a.n_units = cut.n_units; a.n_whole = cut.n_whole;
  // two workgroups fit a compute unit; one persistent workgroup per slot, in 8 groups
  int n_cu = 0;
  {
    const hipError_t e = attn_device_setup(&n_cu);
    if (e != hipSuccess) return e;
  }
  const int members = attn_members(n_cu);
  if (attn_listless(p, dense, cut, members)) a.ent = nullptr;
  a.n_split = cut.n_split;
  a.part_o = a.part_ml = nullptr;
  a.own_slots = cut.own_slots;
  a.own_n = nullptr; a.own_units = nullptr; a.own_pieces = nullptr;
  if (cut.queue && cut.slots() > 0) {
    if (!split_ws) return hipErrorInvalidValue;
    const size_t rows = (size_t)cut.slots() * kTileRows;
    a.part_o = (float*)split_ws;
    a.part_ml = (float*)((char*)split_ws + align_up(rows * p.head_dim * sizeof(float), 256));
    a.own_n = (int32_t*)((char*)a.part_ml + align_up(rows * 2 * sizeof(float), 256));
    a.own_units = (int2*)(a.own_n + 64);
    a.own_pieces = (OwnPiece*)(a.own_units + kMaxPieces);
  }
  a.queue = (uint32_t*)sync_ws;
  a.sync_blocks = attn_sync_blocks(p);
  a.sync_shift = 0;
  while ((1 << (a.sync_shift + 1)) <= a.sync_blocks) ++a.sync_shift;
  a.n_sync = (int)ceil_div(ceil_div(p.q_start + p.q_len, kBlock), a.sync_blocks);
  a.arrive = (uint32_t*)sync_ws + 8 * kQueueStride;
  int32_t* const sched = (int32_t*)((char*)sync_ws + attn_counter_bytes(p));
  a.sched = sched;
#define VS_ATTN_LAUNCH(DD, DCA_, SPLIT_) \
  hipLaunchKernelGGL((k_attention<DD, NQB, DCA_, SPLIT_>), dim3((unsigned)a.n_wg), dim3(128 * NQB), attn_lds_bytes<DD>(), st, a)
  // `units` whole units keeping pace: the arguments and the schedule
  auto keep_pace = [&](int64_t units) {
    a.members = members;
    if (units < 8 * (int64_t)members) a.members = (int)ceil_div(units, 8);  // small launches: no idle workgroups
    a.n_wg = 8 * a.members;
    a.n_full = a.n_qtiles / a.members;
    a.n_rem = a.n_qtiles - a.n_full * a.members;
    const int64_t rounds = (int64_t)a.n_full * a.n_q_heads + ceil_div((int64_t)a.n_rem * a.n_q_heads, a.members);
    a.n_gr = (int)(ceil_div(units, a.members) < rounds ? ceil_div(units, a.members) : rounds);
    hipLaunchKernelGGL(k_attn_schedule, dim3(1), dim3(1024), 0, st, a, sched, g_sched_in_turn.load(std::memory_order_relaxed));
  };
  const auto fold = [&]() {
    const dim3 cgrid((unsigned)((int64_t)(a.n_units - a.n_whole) * (p.head_dim == 128 ? combine_parts<128>() : combine_parts<64>())));
    const auto go = [&](auto&& kernel) { hipLaunchKernelGGL(kernel, cgrid, dim3(256), 0, st, a); };
    if (a.own_slots) { if (p.head_dim == 128) go(k_attn_combine<128, false, true>); else go(k_attn_combine<64, false, true>); }
    else { if (p.head_dim == 128) go(k_attn_combine<128>); else go(k_attn_combine<64>); }
  };
  a.first_piece = 0;
  if (const int ranges = attn_short(p, dense, dca != nullptr, cut)) {
    a.n_split = ranges;
    a.n_whole = ranges > 1 ? 0 : a.n_units;
    ShortArgs b;
    b.q = a.q; b.k = a.k; b.v = a.v; b.out = a.out; b.lse = lse; b.part_o = a.part_o; b.part_ml = a.part_ml;
    b.q_stride_head = a.q_stride_head; b.k_stride_head = a.k_stride_head; b.v_stride_head = a.v_stride_head; b.o_stride_head = a.o_stride_head;
    b.q_stride_tok = (int32_t)a.q_stride_tok; b.k_stride_tok = (int32_t)a.k_stride_tok;
    b.v_stride_tok = (int32_t)a.v_stride_tok; b.o_stride_tok = (int32_t)a.o_stride_tok;
    b.n_units = a.n_units; b.n_qtiles = a.n_qtiles; b.n_hs = a.n_hs; b.n_split = a.n_split;
    b.n_pieces = a.n_units * a.n_split; b.each = (int32_t)ceil_div(b.n_pieces, 8);
    b.by_units = short_magic((uint32_t)b.n_units); b.by_qtiles = short_magic((uint32_t)b.n_qtiles);
    b.by_hs = short_magic((uint32_t)b.n_hs); b.by_split = short_magic((uint32_t)b.n_split);
    b.pack = a.pack; b.group = a.group; b.row_pad = a.row_pad; b.q_rows = (int32_t)a.q_rows; b.m_first = (int32_t)(a.q_start / kBlock);
    b.n_k = (int32_t)a.n_k; b.scale_log2 = a.scale_log2;
    b.v_idx = sets.v_idx; b.v_cnt = sets.v_cnt; b.s_idx = sets.s_idx; b.s_cnt = sets.s_cnt;
    b.v_budget = p.vertical_budget; b.s_budget = p.slash_budget;
    b.bm = a.bm_a; b.bm_words = a.bm_words;
    const bool listed = attn_short_listed(p, cut);
    const dim3 grid((unsigned)(8 * b.each));
    const auto go = [&](auto&& kernel, int lds) { hipLaunchKernelGGL(kernel, grid, dim3(kShortThreads), lds, st, b); };
    if (p.head_dim == 128) {
      if (dense) go(k_attn_short<128, false>, short_lds_bytes<128>());
      else if (listed) go(k_attn_short<128, true, true>, short_lds_bytes<128>());
      else go(k_attn_short<128, true>, short_lds_bytes<128>());
    } else {
      if (dense) go(k_attn_short<64, false>, short_lds_bytes<64>());
      else if (listed) go(k_attn_short<64, true, true>, short_lds_bytes<64>());
      else go(k_attn_short<64, true>, short_lds_bytes<64>());
    }
    if (a.n_split > 1) fold();
    return hipGetLastError();
  }
  if (!cut.queue) {
    keep_pace((int64_t)a.n_qtiles * a.n_q_heads);
    if (p.head_dim == 128) { if (dca) VS_ATTN_LAUNCH(128, true, false); else VS_ATTN_LAUNCH(128, false, false); }
    else { if (dca) VS_ATTN_LAUNCH(64, true, false); else VS_ATTN_LAUNCH(64, false, false); }
    return hipGetLastError();
  }
  // Long walks keep pace while they are whole (where the group of an XCD is as large as a run of units): 8,192 rows at 400K keys
  // 35.9 ms against 37.3 without, 9,500 clustered ones at 300K 12.8 against 14.0 (with the pieces in a launch of their own behind them,
  // 34.1 and 11.6 in the same).  Below 256K keys the caches hold what the members of a group are apart, and whole units come out of the
  // queues, too: 2,400 rows at 100K keys 3.44 ms against 3.52, 5,426 clustered ones at 33K 2.31 against 2.46.
  // Nor heads of 64, whose blocks are half as large, but for attn_few_over.  Against keeping pace (and fewer pieces) everywhere, attention alone: 8 heads, 19,083 rows at 300K
  // keys dense 4,095 us -> 3,719, scattered 4,064 -> 3,792, 9,000 clustered ones 762 -> 670, 15,000 at 500K 1,478 -> 1,268.  Whole rounds of clustered
  // lists are the exception, in whole chunks: 32,768 rows of 8 heads at 600K three sets of keys 2,659, 1,889, 2,064 -> 2,690, 1,950, 2,133 (the attention alone 2,487 -> 2,451, 1,708 ->
  // 1,681, 1,877 -> 1,851).
  // Not where heads share tiles: the pace-keeping kernel takes one head per unit, with one list per head.
  if (attn_paced(cut, p, dense, members)) {
    PacedArgs b;
    keep_pace(a.n_whole);
    b.whole = a;
    a.first_piece = a.n_whole;
    a.members = members;
    a.n_full = a.n_rem = a.n_gr = 0;
    b.cut = a;
    const dim3 grid((unsigned)a.n_wg), block(128 * NQB);
    const auto go = [&](auto&& kernel, int lds) { hipLaunchKernelGGL(kernel, grid, block, lds, st, b); };
    if (p.head_dim == 128) {
      if (dca) go(k_attention_paced<128, NQB, true>, attn_lds_bytes<128>());
      else go(k_attention_paced<128, NQB, false>, attn_lds_bytes<128>());
    } else {
      if (dca) go(k_attention_paced<64, NQB, true>, attn_lds_bytes<64>());
      else go(k_attention_paced<64, NQB, false>, attn_lds_bytes<64>());
    }
    fold();
    return hipGetLastError();
  }
  const int64_t pieces = a.n_whole + (int64_t)(a.n_units - a.n_whole) * a.n_split;
  a.members = pieces < 8 * (int64_t)members && !a.own_slots ? (int)ceil_div(pieces, 8) : members;
  a.n_wg = 8 * a.members;
  a.n_full = a.n_rem = a.n_gr = 0;
  if (a.own_slots) {
    hipLaunchKernelGGL(k_attn_pieces, dim3(1), dim3(1024), 0, st, a);
    const dim3 grid((unsigned)a.n_wg), block(128 * NQB);
    if (p.head_dim == 128) {
      if (dca) hipLaunchKernelGGL((k_attention_own<128, NQB, true>), grid, block, attn_lds_bytes<128>(), st, a);
      else hipLaunchKernelGGL((k_attention_own<128, NQB, false>), grid, block, attn_lds_bytes<128>(), st, a);
    } else {
      if (dca) hipLaunchKernelGGL((k_attention_own<64, NQB, true>), grid, block, attn_lds_bytes<64>(), st, a);
      else hipLaunchKernelGGL((k_attention_own<64, NQB, false>), grid, block, attn_lds_bytes<64>(), st, a);
    }
  } else if (p.head_dim == 128) {
    if (dca) VS_ATTN_LAUNCH(128, true, true); else VS_ATTN_LAUNCH(128, false, true);
  } else {
    if (dca) VS_ATTN_LAUNCH(64, true, true); else VS_ATTN_LAUNCH(64, false, true);
  }
#undef VS_ATTN_LAUNCH
  if (a.n_split > 1 || a.own_slots) fold();
  return hipGetLastError();
}

// ---- several requests per launch ----------------------------------------------------------------
// p.q_len is the longest request, p.q_start + p.q_len the most keys any request sees.  The host knows only these bounds;
// the plan is made on the device (write_plan).  About three pieces per workgroup slot: requests differ in what they cost,
// and a slot takes the next piece when it is done with one: 8 requests of 1 to 64 rows at 262,144 keys 870 us, with one range count
// for all and fixed places 1,850.
static int batch_pieces(const vs_params& p, int n_req) {
  const int64_t group = p.n_q_heads / p.n_kv_heads;
  const int64_t rows = p.q_len + kBlock - 1 > group ? p.q_len + kBlock - 1 : group;   // (single tokens: heads as rows)
  const int64_t units = (int64_t)n_req * p.n_q_heads * ceil_div(rows, (int64_t)kTileRows);
  const int64_t n_blk = ceil_div(p.q_start + p.q_len, kBlock) + 8 * ceil_div(p.vertical_budget, 64);
  int64_t n = n_blk / kMinBatchSteps;
  n = n < 1 ? 1 : (n > kMaxSplit ? kMaxSplit : n);
  return (int)(units * n < kBatchPieces ? units * n : kBatchPieces);
}
static size_t plan_bytes(int n_req) { return align_up((size_t)(n_req + 1) * sizeof(BatchPlan), 256); }
size_t attn_batch_bytes(const vs_params& p, int n_req) {
  const int64_t n_k = p.q_start + p.q_len;
  const size_t lists = (size_t)n_req * p.n_q_heads;
  const size_t rows = (size_t)batch_pieces(p, n_req) * kTileRows;
  return align_up(lists * (size_t)bitmap_words(n_k) * 4, 256) + align_up(lists * (size_t)entry_stride(n_k) * 4, 256) +
         align_up(rows * p.head_dim * sizeof(float), 256) + align_up(rows * 2 * sizeof(float), 256) +
         align_up(8 * kQueueStride * sizeof(uint32_t), 256) + plan_bytes(n_req);
}

hipError_t launch_attention_batch(const vs_params& p, const vs_request* req, int n_req, bool skip_single, void* tokens_ws, void* ws,
                                  hipStream_t st) {
  constexpr int NQB = kAttnQBlocks;
  const int64_t n_k = p.q_start + p.q_len;
  const size_t lists = (size_t)n_req * p.n_q_heads;
  const int64_t words = bitmap_words(n_k), ent_stride = entry_stride(n_k);
  const int pieces = batch_pieces(p, n_req);
  char* w = (char*)ws;
  auto take = [&](size_t bytes) { char* x = w; w += align_up(bytes, 256); return (void*)x; };
  AttnArgs a = {};
  a.bm_a = (uint32_t*)take(lists * (size_t)words * 4);
  a.ent = (uint32_t*)take(lists * (size_t)ent_stride * 4);
  a.part_o = (float*)take((size_t)pieces * kTileRows * p.head_dim * sizeof(float));
  a.part_ml = (float*)take((size_t)pieces * kTileRows * 2 * sizeof(float));
  a.queue = (uint32_t*)take(8 * kQueueStride * sizeof(uint32_t));
  BatchPlan* const plan = (BatchPlan*)take(plan_bytes(n_req));
  a.plan = plan;
  a.arrive = a.queue;   // unused by the key-split kernel; one valid word
  a.n_sync = 1; a.sync_blocks = 1 << 30; a.sync_shift = 30; a.sched = nullptr; a.n_gr = 0;
  a.q_stride_tok = p.q_stride_tok; a.q_stride_head = p.q_stride_head;
  a.k_stride_tok = p.k_stride_tok; a.k_stride_head = p.k_stride_head;
  a.v_stride_tok = p.v_stride_tok; a.v_stride_head = p.v_stride_head;
  a.o_stride_tok = p.o_stride_tok; a.o_stride_head = p.o_stride_head;
  a.bm_stride = words; a.bm_words = (int32_t)words;
  a.ent_stride = ent_stride; a.ent_len = ent_stride;
  a.v_budget = p.vertical_budget;
  a.n_q_heads = p.n_q_heads; a.n_kv_heads = p.n_kv_heads; a.group = p.n_q_heads / p.n_kv_heads;
  a.n_k = n_k;
  a.scale_log2 = p.softmax_scale * kLog2e;
  a.req = req; a.n_req = n_req; a.head_dim = p.head_dim;
  a.max_q_len = p.q_len; a.max_n_k = n_k;
  a.skip_single = skip_single;
  int n_cu = 0;
  hipError_t e = attn_device_setup(&n_cu);
  if (e != hipSuccess) return e;
  const int members = attn_members(n_cu);
  a.members = members; a.n_wg = 8 * members; a.n_full = 0; a.n_rem = 0;
  ListArgs l = {};
  l.s_budget = p.slash_budget;
  l.n_words = (int)words; l.ent_stride = (int)ent_stride;
  l.bm_a = (uint32_t*)a.bm_a; l.ent = (uint32_t*)a.ent;
  l.n_heads = p.n_q_heads; l.group = a.group; l.pack = 1;
  l.zero = a.queue; l.n_zero = 8 * kQueueStride;
  l.req = req; l.plan = plan; l.n_req = n_req; l.skip_single = skip_single; l.pieces = pieces;
  l.max_q_len = p.q_len; l.max_n_k = n_k;
  // (a few workgroups per request where they fill the chip: 24,000 of 1,024 threads that find nothing to do, for 1,500 dense
  // requests of 16 heads, took 187 us, 48 so)
  const int each = (int)ceil_div(kListGroups, n_req);
  const unsigned lists_x = (unsigned)(each < p.n_q_heads ? each : p.n_q_heads);
  MixedArgs m;
  if (tokens_ws) {
    m.tokens = decode_args(p, req, n_req, tokens_ws);
    m.rows = a;
    hipLaunchKernelGGL((k_mixed_lists<NQB>), dim3(lists_x, 2 * (unsigned)n_req + 1), dim3(kBlThreads), 0, st, MixedListArgs{l, m.tokens});
  } else {
    hipLaunchKernelGGL((k_build_blocklist<NQB, true>), dim3(lists_x, (unsigned)n_req + 1), dim3(kBlThreads), 0, st, l);
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;   // (what follows goes by the plan and the lists)
  const dim3 grid((unsigned)a.n_wg), block(128 * NQB);
  const int64_t parts = ceil_div(pieces, 2) * (p.head_dim == 128 ? combine_parts<128>() : combine_parts<64>());   // cut units: two pieces or more
  const unsigned folds = (unsigned)(parts < kCombineGrid ? parts : kCombineGrid);
  if (tokens_ws) {
    const dim3 cgrid(folds + (unsigned)n_req * (unsigned)p.n_q_heads);
    if (p.head_dim == 128) {
      hipLaunchKernelGGL((k_attention_mixed<128, NQB>), grid, block, attn_lds_bytes<128>(), st, m);
      hipLaunchKernelGGL(k_mixed_combine<128>, cgrid, dim3(256), 0, st, m, (int)folds);
    } else {
      hipLaunchKernelGGL((k_attention_mixed<64, NQB>), grid, block, attn_lds_bytes<64>(), st, m);
      hipLaunchKernelGGL(k_mixed_combine<64>, cgrid, dim3(256), 0, st, m, (int)folds);
    }
  } else if (p.head_dim == 128) {
    hipLaunchKernelGGL((k_attention<128, NQB, false, true, true>), grid, block, attn_lds_bytes<128>(), st, a);
    hipLaunchKernelGGL((k_attn_combine<128, true>), dim3(folds), dim3(256), 0, st, a);
  } else {
    hipLaunchKernelGGL((k_attention<64, NQB, false, true, true>), grid, block, attn_lds_bytes<64>(), st, a);
    hipLaunchKernelGGL((k_attn_combine<64, true>), dim3(folds), dim3(256), 0, st, a);
  }
  return hipGetLastError();
}

hipError_t launch_count_tiles(const vs_params& p, const int32_t* v_idx, const int32_t* v_cnt,
                              const BlockList& bl, int64_t* tiles, hipStream_t st) {
  hipLaunchKernelGGL(k_count_tiles, dim3(p.n_q_heads), dim3(256), 0, st, v_idx, v_cnt,
                     p.vertical_budget, bl.bm_a, (int)bl.words, p.q_start - p.q_start % kBlock,
                     p.q_len + p.q_start % kBlock, tiles);
  return hipGetLastError();
}

}  // namespace vs
