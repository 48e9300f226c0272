// Internal declarations shared by the HIP sources of libvs (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "../../include/vs.h"

namespace vs {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(8))) float f32x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

constexpr int kBlock = 64;            // B: edge of the computed slash blocks
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// a 64-bit value that is the same in every lane, moved into scalar registers
template <typename T>
__device__ __forceinline__ T uniform64(T x) {
  static_assert(sizeof(T) == 8, "uniform64 takes pointers and 64-bit integers");
  const uint64_t b = (uint64_t)x;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b), hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
  return (T)(((uint64_t)hi << 32) | lo);
}

// Set-up that a device needs once (function attributes are held per device by the runtime).
struct DeviceOnce {
  static constexpr int kMaxDevices = 64;
  std::mutex mu;
  bool done[kMaxDevices] = {false};
  template <typename F>
  hipError_t run(F&& set_up) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!done[dev]) {
      e = set_up();
      if (e != hipSuccess) return e;
      done[dev] = true;
    }
    return hipSuccess;
  }
};

static inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
static inline size_t align_up(size_t a, size_t b) { return (a + b - 1) / b * b; }

// ---- block list (built per head from the selected slash offsets) -----------------------
// A: bitmap, bit a set <=> block diagonal a is computed.
// ent: ascending list of key-block entries for a query tile of kAttnQBlocks query blocks:
//   entry = (cc << 4) | mask, cc = c + (kAttnQBlocks - 1); the tile whose first query block is
//   m0 uses key block m0 - c, and query block t of the tile takes part iff mask bit t is set
//   (diagonal c + t is in A).  The list is padded with sentinels (cc = 0x7FFFFFF) so that a
//   reader may fetch whole batches of 64 entries without bounds checks.
constexpr int kAttnQBlocks = 2;       // query blocks (of 64 rows) per attention workgroup
constexpr uint32_t kEntSentinel = 0x7FFFFFF0u;

// The block diagonals of lists of slash offsets as bytes in LDS: offset o computes diagonals floor(o / 64) and, where it is no multiple
// of 64, the next one, ceil(o / 64) in both cases.  Byte (ad - b0 << shift) + p is set for diagonal ad of list p of n_lists (at most
// 64); diagonals outside b0 .. b0 + n - 1 go to the byte of index n_win.  Rows of `budget` offsets at s_idx, s_cnt of each in use, in any
// order; called by a whole workgroup of THREADS.  Bytes, because all that is done to them is a store: an atomic OR into a word of bits,
// only for what an offset's neighbour does not set already, was 60 instructions per offset, 25 of the 29 us that the lists of seven heads
// with 6,096 offsets each took.  U groups of THREADS offsets are on their way at once, the first ones without waiting for the
// counts (what lies in a row behind its count is read and dropped).
template <int THREADS, int U>
__device__ __forceinline__ void collect_flags(uint8_t* flags, int shift, int b0, int n, int n_win, const int32_t* s_idx,
                                              const int32_t* s_cnt, int budget, int n_lists) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int cnts = s_cnt[lane < n_lists ? lane : 0];
  auto put = [&](int offset, bool in, int list) {
    const uint32_t x = (uint32_t)((offset >> 6) - b0), y = (uint32_t)(((offset + 63) >> 6) - b0);
    flags[((in && x < (uint32_t)n ? x : (uint32_t)n_win) << shift) + list] = 1;
    flags[((in && y < (uint32_t)n ? y : (uint32_t)n_win) << shift) + list] = 1;
  };
  if (n_lists == 1 && budget <= THREADS) {   // (the loop below is 0.8 us of instructions for it)
    const int o = s_idx[tid < budget ? tid : budget - 1];
    if (tid < __builtin_amdgcn_readfirstlane(cnts)) put(o, true, 0);
    return;
  }
  int p = 0, at = 0, most;   // list and place in it of the next group: the lists in turn
  do {
    int o[U], list[U], from[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      list[u] = p;
      from[u] = at;
      const int i = at + tid;
      o[u] = 0;
      if (at < budget) o[u] = s_idx[(int64_t)p * budget + (i < budget ? i : budget - 1)];
      if (++p == n_lists) { p = 0; at += THREADS; }
    }
    most = lane < n_lists ? cnts : 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int cnt = __builtin_amdgcn_readlane(cnts, list[u]);
      if (from[u] >= cnt) continue;
      put(o[u], from[u] + tid < cnt, list[u]);
    }
  } while (__ballot(most > at));
}

struct BlockList {
  uint32_t* bm_a;     // [heads][words]
  uint32_t* ent;      // [heads][ent_stride]
  int64_t words, ent_stride;
  int heads;          // n_q_heads, or 1 for the dense list shared by all heads
};
static inline int64_t bitmap_words(int64_t n_k) { return ceil_div(ceil_div(n_k, kBlock) + 8, 32) + 2; }
static inline int64_t entry_stride(int64_t n_k) {
  return ceil_div(ceil_div(n_k, kBlock) + kAttnQBlocks, 64) * 64 + 128;
}
static inline size_t blocklist_bytes(const vs_params& p, bool dense) {
  const size_t heads = dense ? 1 : (size_t)p.n_q_heads;
  const int64_t n_k = p.q_start + p.q_len;
  return align_up(heads * (size_t)bitmap_words(n_k) * 4, 256) + align_up(heads * (size_t)entry_stride(n_k) * 4, 256);
}
static inline BlockList blocklist_layout(const vs_params& p, bool dense, void* ws) {
  BlockList b;
  const int64_t n_k = p.q_start + p.q_len;
  b.heads = dense ? 1 : p.n_q_heads;
  b.words = bitmap_words(n_k);
  b.ent_stride = entry_stride(n_k);
  b.bm_a = (uint32_t*)ws;
  b.ent = (uint32_t*)((char*)ws + align_up((size_t)b.heads * (size_t)b.words * 4, 256));
  return b;
}

// ---- launchers (defined in the .hip files; all enqueue on `st`, return hipError_t) ------
hipError_t launch_build_blocklist(const vs_params& p, const int32_t* s_idx, const int32_t* s_cnt,
                                  const int32_t* v_cnt, bool dense, bool dca, const BlockList& bl, void* sync_ws, hipStream_t st);
// Dual Chunk Attention: the two other rotations of the chunk's queries (same strides as q),
// chunk length and local window in tokens (multiples of 64)
struct DcaArgs {
  const void* q_succ;
  const void* q_inter;
  int64_t chunk, window;
};
struct IndexSets {   // (nulls when dense)
  const int32_t* v_idx;
  const int32_t* v_cnt;
  const int32_t* s_idx;
  const int32_t* s_cnt;
};
// sync_ws: attn_sync_bytes(p) bytes: counters, cleared by launch_build_blocklist, and the schedule; split_ws:
// attn_split_bytes(p) bytes (may be null when that is 0); dca may be null
hipError_t launch_attention(const vs_params& p, const void* q, const DcaArgs* dca, const void* k, const void* v,
                            const IndexSets& sets, bool dense,
                            const BlockList& bl, void* out, float* lse, void* sync_ws, void* split_ws, bool least,
                            hipStream_t st);
// several requests in one launch (short chunks, decode steps): p.q_len = the longest request,
// p.q_start + p.q_len = the most keys any request sees; req is a device array
size_t attn_batch_bytes(const vs_params& p, int n_req);
// (skip_single: single tokens are the decode walk's; with tokens_ws, decode_bytes(p, n_req, true, true, false) of them, this launch has it)
hipError_t launch_attention_batch(const vs_params& p, const vs_request* req, int n_req, bool skip_single, void* tokens_ws, void* ws,
                                  hipStream_t st);
// single tokens, one request (`one`, by value; lists: it has index sets) or those of a table (req, device; lists = true)
bool decode_fits(const vs_params& p);
// (least: the smallest workspace, with which it is slower)
size_t decode_bytes(const vs_params& p, int n_req, bool table, bool lists, bool least);
hipError_t launch_decode(const vs_params& p, const vs_request* one, const vs_request* req, int n_req, bool lists, bool least, void* ws,
                         hipStream_t st);
size_t attn_sync_bytes(const vs_params& p);
// key split of short chunks: bytes of partial results
void set_attn_key_split(int n);
void set_attn_schedule_in_turn(int on);
size_t attn_split_bytes(const vs_params& p, bool dense, bool least);
void set_attn_segment_blocks(int blocks);
hipError_t launch_count_tiles(const vs_params& p, const int32_t* v_idx, const int32_t* v_cnt,
                              const BlockList& bl, int64_t* tiles, hipStream_t st);

size_t estimate_ws_bytes(const vs_params& p);
hipError_t launch_estimate(const vs_params& p, const void* q, const DcaArgs* dca, const void* k, float* vscore,
                           float* sscore, float* lse_lastq, void* ws, hipStream_t st);

// (least: the smallest workspace that a call takes)
size_t select_ws_bytes(const vs_params& p, bool least);
// ws with fewer bytes than that: another route (slower for long rows); 4,736 bytes per row at least
hipError_t launch_select(const vs_params& p, const float* vscore, const float* sscore,
                         const int32_t* v_budget_h, const int32_t* s_budget_h,
                         int32_t* v_idx, int32_t* v_cnt, int32_t* s_idx, int32_t* s_cnt,
                         void* ws, size_t ws_bytes, hipStream_t st);
// the selection's scratch in a file-scope device array (callers that cannot allocate): the most query heads
// of such a call, a limit of its interface, and the array on the current device
constexpr int kSelStaticMaxHeads = 128;
hipError_t select_static_scratch(void** ptr_out, size_t* bytes_out);
hipError_t launch_recall(const vs_params& p, const float* lse_sparse, const float* lse_full, float* recall,
                         hipStream_t st);
hipError_t launch_refine(const vs_params& p, const float* recall, float threshold, int32_t dv, int32_t ds,
                         int32_t* v_budget, int32_t* s_budget, int32_t* changed, hipStream_t st);

}  // namespace vs
