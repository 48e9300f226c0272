// Attention of single tokens (decode steps) against long caches, one request or many per launch, dense or with
// the index sets of the vertical-slash pattern (section 5.2, "Integrating with Chunked prefill": decoding of other
// requests goes on beside a long prefill).  bf16 MFMA with fp32 accumulation.
//
// Bound: the one read of the K and V rows; everything else is arranged around keeping that read going.
//  * The G <= 16 query heads of a KV group are the columns of 16x16x32 MFMA tiles (S^T = K Q^T, O^T = V^T P^T), so
//    K and V are read once per group.  A wave works alone on 32 keys at a time: it copies the rows global -> LDS into
//    its own two buffers (the next 32 keys are on their way while these are multiplied), waits for its own copies
//    only, and there is no barrier until the waves of the workgroup fold their results.  One workgroup of four waves
//    fills the LDS of a compute unit: 64 to 128 KB of copies in flight.  (Beside the tiles of longer requests, in
//    k_attention_mixed of vs_attn.hip, a wave has one buffer, for keys and values in turn, and a workgroup 64 KB.)
//  * Where there is much to read the waves take two neighbouring KV heads side by side, whose rows lie next to each other
//    (kDecSideBlocks).
//  * Work is cut into equal shares of 64-key blocks over all requests and KV heads (a share may start in the
//    middle of one and end in the middle of another), so caches of different lengths leave no workgroup idle.  Every
//    workgroup finds its share from the lengths alone.  Partial results are folded by k_decode_combine; a (request, KV
//    head) that lies in one share is finished on the spot.
//  * With index sets the tokens of a group walk the UNION of the heads' block lists (k_decode_lists; per entry the
//    heads whose own list has the diagonal: the scores of the others are -inf), then the gathered columns head by head.
// Measured on one MI355X, 28 query / 4 KV heads, head_dim 128, against the tile kernel of vs_attn.hip with the heads as rows of
// its 128-row tiles (copies of a step shared by four waves of which one multiplied, a barrier per step, one range count for a
// whole batch): one token at 5,003 keys 39 -> 10 us, at 1M keys 510 -> 361 (5.9 TB/s of K and V); 24 tokens at 2K to 64K keys
// 395 -> 215 (5.8 TB/s); 8 tokens with index sets at 262,144 keys 1,042 -> 770 (lists 252 -> 17 of it).
#include "vs_decode_walk.h"

namespace vs {

template <int D, typename Len>
__device__ __forceinline__ void decode_apart(const DecodeArgs& a) {
  int64_t mine;
  bool unused;
  const int64_t T = decode_total<Len>(a, mine, unused);
  decode_body<D, 1, false, Len>(a, T, mine, gridDim.x);
}
template <int D>
__global__ __launch_bounds__(kDecThreads, 2) void k_decode(const DecodeArgs a) { decode_apart<D, int4>(a); }
template <int D>
__global__ __launch_bounds__(kDecThreads, 2) void k_decode_least(const DecodeArgs a) { decode_apart<D, int2>(a); }
// A table whose bounds allow two neighbouring KV heads side by side: whether that pays, its requests say (see kDecSideBlocks).
__global__ __launch_bounds__(kDecThreads, 2) void k_decode_pairs(const DecodeArgs a) {
  int64_t mine;
  bool uneven;
  const int64_t T = decode_total<int4>(a, mine, uneven);
  if (T >= kDecSideBlocks && !uneven) decode_body<128, 2, false, int4>(a, T / 2, mine, gridDim.x);
  else decode_body<128, 1, false, int4>(a, T, mine, gridDim.x);
}
template <int D, int SIDE>
__global__ __launch_bounds__(kDecThreads, 2) void k_decode_one(const DecodeArgs a) { decode_body<D, SIDE, true, int4>(a, a.one_T, 0, gridDim.x); }

template <int D, int NW, int SIDE, typename Len = int4>
__global__ __launch_bounds__(64 * NW) void k_decode_combine(const DecodeArgs a) { decode_fold<D, NW, SIDE, Len>(a, blockIdx.x, blockIdx.y); }

template <typename Len>
__device__ __forceinline__ void decode_all_lists(const DecodeArgs& a) {
  __shared__ __attribute__((aligned(16))) uint8_t flags[kDecListBytes + 16];
  decode_lists<Len, kDecListBytes>(a, blockIdx.x, blockIdx.y, flags);
}
__global__ __launch_bounds__(kDecListThreads) void k_decode_lists(const DecodeArgs a) { decode_all_lists<int4>(a); }
__global__ __launch_bounds__(kDecListThreads) void k_decode_least_lists(const DecodeArgs a) { decode_all_lists<int2>(a); }

// ---------------------------------------------------------------------------------------------------
// the query heads of a KV group are the columns of one MFMA tile
bool decode_fits(const vs_params& p) { return p.n_q_heads / p.n_kv_heads <= 16; }

namespace {
constexpr int kDecShares = 256;   // at most: one workgroup fills the LDS of a compute unit
struct DecLayout {
  size_t part_ml, plan, len, ent, bm, total;
  int32_t words, ent_stride, shares;
  int32_t side;   // KV heads side by side, of a table at most
};
// table: requests from a table, with or without index sets; lists: with.  least: every KV head by itself, the columns of every head gathered
DecLayout dec_layout(const vs_params& p, int n_req, bool table, bool lists, bool least) {
  DecLayout l;
  const int64_t n_blk = ceil_div(p.q_start + p.q_len, (int64_t)kBlock);
  const bool side_by_side = p.k_stride_head == p.head_dim && p.v_stride_head == p.head_dim;
  l.side = !least && (table || !lists) && p.head_dim == 128 && p.n_kv_heads % 2 == 0 && side_by_side && (int64_t)n_req * p.n_kv_heads * n_blk >= kDecSideBlocks ? 2 : 1;
  const size_t G = (size_t)(p.n_q_heads / p.n_kv_heads), segs = (size_t)n_req * (p.n_kv_heads / l.side);
  const int64_t most = ceil_div((int64_t)segs * (n_blk + (lists ? (int64_t)G * ceil_div(p.vertical_budget, 64) : 0)), kDecMinBlocks / l.side);
  l.shares = (int32_t)(most < kDecShares ? most : kDecShares);
  l.words = (int32_t)ceil_div(n_blk, 32);
  l.ent_stride = (int32_t)n_blk;
  const size_t rows = ((size_t)l.shares + segs) * l.side * G;
  size_t off = align_up(rows * p.head_dim * sizeof(float), 256);
  l.part_ml = off; off += align_up(rows * 2 * sizeof(float), 256);
  l.plan = off; off += align_up((2 + (size_t)n_req) * sizeof(int64_t), 256);
  l.len = l.ent = l.bm = off;
  if (lists) {
    const size_t heads = (size_t)n_req * p.n_kv_heads;
    off += align_up(heads * (least ? sizeof(int2) : sizeof(int4)), 256);
    l.ent = off; off += align_up(heads * (size_t)l.ent_stride * sizeof(uint2), 256);
    l.bm = off; off += align_up((size_t)n_req * p.n_q_heads * (size_t)l.words * sizeof(uint32_t), 256);
  }
  l.total = off;
  return l;
}
}  // namespace

size_t decode_bytes(const vs_params& p, int n_req, bool table, bool lists, bool least) { return dec_layout(p, n_req, table, lists, least).total; }

static DecodeArgs dec_args(const vs_params& p, const DecLayout& l, const vs_request* one, const vs_request* req, int n_req, void* ws) {
  DecodeArgs a = {};
  if (one) a.one = *one;
  a.req = req; a.n_req = n_req;
  a.n_q_heads = p.n_q_heads; a.n_kv_heads = p.n_kv_heads; a.group = p.n_q_heads / p.n_kv_heads;
  a.q_stride_head = p.q_stride_head; a.o_stride_head = p.o_stride_head;
  a.k_stride_tok = p.k_stride_tok; a.k_stride_head = p.k_stride_head;
  a.v_stride_tok = p.v_stride_tok; a.v_stride_head = p.v_stride_head;
  a.scale_log2 = p.softmax_scale * kLog2e;
  a.v_budget = p.vertical_budget; a.s_budget = p.slash_budget;
  a.max_n_k = p.q_start + p.q_len;
  char* const w = (char*)ws;
  a.part_o = (float*)w;
  a.part_ml = (float*)(w + l.part_ml);
  a.plan = (int64_t*)(w + l.plan);
  a.len = w + l.len;
  a.ent = (uint2*)(w + l.ent);
  a.bm = (uint32_t*)(w + l.bm);
  a.words = l.words; a.ent_stride = l.ent_stride;
  a.shares = l.shares; a.side = l.side;
  return a;
}
static void launch_lists(const DecodeArgs& a, bool least, hipStream_t st) {
  const dim3 grid((unsigned)a.n_kv_heads, (unsigned)a.n_req);
  if (least) hipLaunchKernelGGL(k_decode_least_lists, grid, dim3(kDecListThreads), 0, st, a);
  else hipLaunchKernelGGL(k_decode_lists, grid, dim3(kDecListThreads), 0, st, a);
}
// the fold: by four waves, or by eight where a KV head lies in many shares
template <typename Four, typename Eight>
static void launch_fold(const DecodeArgs& a, Four&& four, Eight&& eight, hipStream_t st) {
  const dim3 grid((unsigned)a.n_q_heads, (unsigned)a.n_req);
  if (a.shares > 32 * (int64_t)a.n_req * (a.n_kv_heads / a.side)) hipLaunchKernelGGL(eight, grid, dim3(512), 0, st, a);
  else hipLaunchKernelGGL(four, grid, dim3(256), 0, st, a);
}

DecodeArgs decode_args(const vs_params& p, const vs_request* req, int n_req, void* ws) {
  return dec_args(p, dec_layout(p, n_req, true, true, false), nullptr, req, n_req, ws);
}

hipError_t launch_decode(const vs_params& p, const vs_request* one, const vs_request* req, int n_req, bool lists, bool least, void* ws,
                         hipStream_t st) {
  const DecLayout l = dec_layout(p, n_req, req != nullptr, lists, least);
  DecodeArgs a = dec_args(p, l, one, req, n_req, ws);
  const int n_seg = p.n_kv_heads / l.side;
  static DeviceOnce once;   // the opt-in to more than 64 KiB of LDS
  const hipError_t e = once.run([]() {
    const void* const fns[8] = {reinterpret_cast<const void*>(&k_decode<128>), reinterpret_cast<const void*>(&k_decode_pairs),
                                reinterpret_cast<const void*>(&k_decode_one<128, 1>), reinterpret_cast<const void*>(&k_decode_one<128, 2>),
                                reinterpret_cast<const void*>(&k_decode_least<128>), reinterpret_cast<const void*>(&k_decode<64>),
                                reinterpret_cast<const void*>(&k_decode_one<64, 1>), reinterpret_cast<const void*>(&k_decode_least<64>)};
    for (int i = 0; i < 8; ++i) {
      const hipError_t e1 = hipFuncSetAttribute(fns[i], hipFuncAttributeMaxDynamicSharedMemorySize,
                                                i < 5 ? decode_lds_bytes<128>() : decode_lds_bytes<64>());
      if (e1 != hipSuccess) return e1;
    }
    return hipSuccess;
  });
  if (e != hipSuccess) return e;
  if (lists) launch_lists(a, least, st);
  if (one && !lists) {   // as k_decode counts them
    a.one_T = ceil_div(one->q_start + one->q_len, (int64_t)kBlock) * n_seg;
    a.one_n = ceil_div(a.one_T, kDecMinBlocks / l.side);
    if (a.one_n > l.shares) a.one_n = l.shares;
  }
  const dim3 grid((unsigned)l.shares);
  const auto fold = [&](auto&& four, auto&& eight) { launch_fold(a, four, eight, st); };
  const auto walk = [&](auto&& kernel, int lds) { hipLaunchKernelGGL(kernel, grid, dim3(kDecThreads), lds, st, a); };
  constexpr int lds128 = decode_lds_bytes<128>(), lds64 = decode_lds_bytes<64>();
  if (l.side == 2) {
    if (a.one_T) {
      walk(k_decode_one<128, 2>, lds128);
      fold(k_decode_combine<128, 4, 2>, k_decode_combine<128, 8, 2>);
    } else {
      walk(k_decode_pairs, lds128);
      fold(k_decode_combine<128, 4, 0>, k_decode_combine<128, 8, 0>);
    }
  } else if (least && !a.one_T) {
    if (p.head_dim == 128) {
      walk(k_decode_least<128>, lds128);
      fold(k_decode_combine<128, 4, 1, int2>, k_decode_combine<128, 8, 1, int2>);
    } else {
      walk(k_decode_least<64>, lds64);
      fold(k_decode_combine<64, 4, 1, int2>, k_decode_combine<64, 8, 1, int2>);
    }
  } else if (p.head_dim == 128) {
    if (a.one_T) walk(k_decode_one<128, 1>, lds128); else walk(k_decode<128>, lds128);
    fold(k_decode_combine<128, 4, 1>, k_decode_combine<128, 8, 1>);
  } else {
    if (a.one_T) walk(k_decode_one<64, 1>, lds64); else walk(k_decode<64>, lds64);
    fold(k_decode_combine<64, 4, 1>, k_decode_combine<64, 8, 1>);
  }
  return hipGetLastError();
}

}  // namespace vs
