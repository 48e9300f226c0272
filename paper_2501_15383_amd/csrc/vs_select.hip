// Selection of the vertical and slash lines (section 5.2, MInference paragraph: critical
// tokens are chosen by the vertical-slash pattern with a per-head count of vertical and
// diagonal lines).  Exact top-k of up to 2^31 fp32 scores per (head, kind) row without sorting;
// all of it is integer work on an order-preserving image of the floats (keys), so the result is
// exact and run-to-run identical:
//   * the forced entries (the lowest `keep` indices) are taken first;
//   * a most-significant-digit radix select (11 + 11 + 10 bits, histograms in LDS) finds the
//     threshold key T and how many entries equal to T are needed;
//   * one ordered compaction emits indices in ascending order: every key > T, and the
//     lowest-index keys == T (ties go to the lower index).  Ranks come from wave ballots.
// One workgroup finishes a row (k_sel_row), from one of three sources:
//   registers   rows of up to kSelRegKeys scores are read once and stay in registers; a call is then
//               this one launch, bound by its vector instructions (of 32 scores per lane: loads and range 3.0 us, first
//               digit 3, the pass that lists the threshold's bin 1.5, emission 2.5) and, of short rows, by its barriers
//   candidates  longer rows are thinned out first.  A sample of 4,096 (8,192, 16,384) scores per row gives a floor that
//               about k + 4.5 sigma entries exceed, and only those entries are kept, in registers (without a workspace: in LDS) if there
//               are at most kSelCand of them.  With a workspace the whole chip makes the lists, in one pass over the scores
//               (k_sel_sample, k_sel_filter; bound by that read at 1M keys); without a workspace k_sel_row makes its
//               row's own.  A threshold that falls on a crowd of equal
//               scores is the floor itself: all candidates are wanted, and of the crowd its first entries, for which the row
//               is read until it has them (28 heads, 1M keys of which 2,097 are not zero, 6,096 wanted: 485 us with the row
//               read to its end, 125 so).
//   the row     where the sample missed, or the list does not fit, every digit and the compaction read the
//               row again: exact in every case.
// Long rows with large budgets (lists longer than sel_most_candidates) are cut into slices, one workgroup each, that read the
// scores once per digit of 8 bits, once for the counts and once for the compaction (k_slice_*): the list would be one
// workgroup's work.
// Measured on one MI355X, 28 heads, budgets 1000 / 6096, against four digits, a count and a write pass over all
// scores in seven launches: 8,192 scores per row 8 us (67), 32,768 15 us (70), 300,001 44 us (152), 1M 88 us
// (345: filter 57 us = 4.1 TB/s, sample 17, rows 16, under a profiler); 4 heads, budgets 128 / 256, 300,000: 24 us.
#include "vs_common.h"

namespace vs {

constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / 64;
constexpr int kSelRegKeys = 48 * kSelThreads;  // longest row that stays in registers (44,000 scores, 28 heads: 20 us, 35 with the
                                               // row's candidates in LDS; three launches 36 at 49,153.  Scores of 2 to 25 values and
                                               // budgets of hundreds take 28 to 39 so, 24 to 33 with candidates)
constexpr int kSelCand = 16384;                // longest list of candidates (128 KB of LDS)
constexpr int kSelSlice = 2048;                // scores per wave of the filter (one slice each)
constexpr int kSelFilterThreads = 256;
constexpr int kSelStep = 8;                    // scores per lane and step where the row is read again and again
constexpr int kSelBins = 2048;
// Counters per bin of rows in registers.  Lanes that share a bin queue for it, the longer the row the longer: 28 heads, of two values
// 44,000 scores 74 us with one, 38 with four; 36,000 of an estimate 17.9 and 17.6; of up to 16 per lane four cost 0.15 us per row more to
// clear and add up.  (Eight lie in too few banks: 20.8.)  A row that lists its own candidates (without a workspace) has its
// LDS full of them.
constexpr int sel_copies(int kpt) { return kpt > 16 ? 4 : 1; }
// control block of a row whose slices go through the digits together, in 32-bit words
constexpr int kSliceMax = 64;                  // slices of a row at most
constexpr int kWHist = 0;                      // [4][256] histogram of every digit
constexpr int kWDone = 1024;                   // [4] workgroups done with the digit
constexpr int kWState = 1028;                  // [5][2] (prefix, entries still to find) before digit 0..3 and after
constexpr int kWCount = 1056;                  // [slices][2] keys > T, keys == T
constexpr int kSliceRowWords = kWCount + 2 * kSliceMax;
// workspace of a row: header, table of slices, candidates
struct SelHeader {
  uint32_t floor_key;  // entries above it are candidates
  uint32_t count;      // candidates so far (beyond the list's room: it is incomplete)
  uint32_t equal;      // entries equal to the floor
  uint32_t pad;
};

__device__ __forceinline__ uint32_t order_key(float x) {
  const uint32_t b = __float_as_uint(x);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

struct SelArgs {
  const float* vscore;
  const float* sscore;
  int64_t n;  // n_k
  int32_t n_q_heads;
  int32_t v_budget, s_budget, keep_v, keep_s;  // budgets: row lengths of the outputs (maxima)
  const int32_t* v_budget_h;  // optional per-head budgets (clamped to 1 .. maximum), else null
  const int32_t* s_budget_h;
  int32_t* v_idx;
  int32_t* v_cnt;
  int32_t* s_idx;
  int32_t* s_cnt;
  // null: every row lists its own candidates
  SelHeader* hdr;      // [2 Hq]
  uint2* slices;       // [2 Hq][n_slices] (first candidate, candidates) of every slice
  uint2* cand;         // [2 Hq][cap] (key, index)
  uint32_t cap;
  int32_t n_slices;
  int32_t samples_v, samples_s;  // samples per thread for the rows of each kind
  // rows in slices
  uint32_t* ctl;       // [2 Hq][kSliceRowWords]
  int64_t slice_len;   // a multiple of kSelStep * kSelThreads
};

// row = kind * Hq + h
struct SelRow {
  const float* sc;
  int32_t* out;
  int kind, h, row_len;
  int k;        // entries of the result
  int f;        // forced entries 0 .. f - 1
  uint32_t kp;  // still to choose among indices f .. n - 1
};
__device__ __forceinline__ SelRow sel_row(const SelArgs& a, int row) {
  SelRow r;
  r.kind = row >= a.n_q_heads;
  r.h = row - r.kind * a.n_q_heads;
  r.sc = (r.kind ? a.sscore : a.vscore) + (int64_t)r.h * a.n;
  r.row_len = r.kind ? a.s_budget : a.v_budget;
  r.out = (r.kind ? a.s_idx : a.v_idx) + (int64_t)r.h * r.row_len;
  const int32_t* per_head = r.kind ? a.s_budget_h : a.v_budget_h;
  int budget = r.row_len;
  if (per_head) {
    budget = per_head[r.h];
    budget = budget < 1 ? 1 : (budget > r.row_len ? r.row_len : budget);
  }
  const int keep = r.kind ? a.keep_s : a.keep_v;
  r.k = budget < a.n ? budget : (int)a.n;
  r.f = keep < r.k ? keep : r.k;
  r.kp = (uint32_t)(r.k - r.f);
  return r;
}

// sample rank whose score about k + 4.5 sigma entries of a row of n reach (sigma: of the number of the
// row's best k that a sample of `samples` meets)
__host__ __device__ inline float sel_sample_rank(float k, float n, float samples) {
  const float mu = k * (samples / n);
  return mu + 4.5f * sqrtf(mu) + 4.f;
}

// R: counters per bin (lane x adds to the (x % R)-th; a power of two)
template <int R>
struct SelShared {
  alignas(16) uint32_t hist[R * kSelBins];
  alignas(16) uint32_t wsum[kSelWaves];          // (read four words at a time: 0.35 us of a row's 7 to 10)
  alignas(16) uint32_t wtot[2][kSelWaves][2];
  alignas(16) uint32_t wmin[kSelWaves], wmax[kSelWaves];
  uint32_t digit, rest, in_bin;
  int32_t first[kSelWaves + 1];
  uint32_t few, few_T, few_need;   // keys of the last bin listed so far (in hist), and what they decide
  uint32_t extra[kSelWaves];       // of a wave's keys in that bin, those taken
};

// smallest and largest of the threads' keys
template <int R>
__device__ __forceinline__ void sel_range(SelShared<R>& sh, uint32_t lo, uint32_t hi, uint32_t& all_lo, uint32_t& all_hi) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t l = __shfl_xor(lo, d), h = __shfl_xor(hi, d);
    lo = l < lo ? l : lo;
    hi = h > hi ? h : hi;
  }
  if (lane == 0) { sh.wmin[wv] = lo; sh.wmax[wv] = hi; }
  __syncthreads();
  all_lo = sh.wmin[0]; all_hi = sh.wmax[0];
#pragma unroll
  for (int x = 1; x < kSelWaves; ++x) {
    all_lo = sh.wmin[x] < all_lo ? sh.wmin[x] : all_lo;
    all_hi = sh.wmax[x] > all_hi ? sh.wmax[x] : all_hi;
  }
}

// The kp-th largest of the keys that for_each(f) hands to f(key, valid) (valid keys lie in lo .. hi and number at least
// kp >= 1): keys above T, and need_eq of those equal to it, are the kp largest; need_eq is 0 wherever every key equal to the
// kp-th is wanted (T is the key below it then).  Digits of 11 bits from the top of the range
// hi - lo, so that keys that share their exponent still spread over the bins (scores do: with digits of the
// whole key a wave's 64 additions met in four bins, 65 to 250 clocks each); done as soon as a bin is taken whole.
// Keys equal to lo are not counted, their bin has whatever the others leave of kp: a crowd of the smallest score (zeros) would
// queue for it (32,768 scores, 2 in 1,000 of them not zero: 102 us counted, 25 so).
// Called by the whole workgroup; every thread gets the result.
constexpr uint32_t kSelAtLo = ~0u;
struct SelDigits {
  uint32_t prefix, krem, in_bin;   // digits so far (of key - lo), wanted keys of that bin, keys in it (kSelAtLo: krem keys equal to lo)
  int shift;                       // bits below the prefix
  bool first;
};
__device__ __forceinline__ SelDigits sel_digits(uint32_t kp, uint32_t lo, uint32_t hi) {
  SelDigits d;
  d.prefix = 0; d.krem = kp; d.in_bin = 0; d.first = true;
  d.shift = 32 - __clz((int)(hi - lo) | 1);
  return d;
}
template <int R, typename ForEach>
__device__ __forceinline__ void sel_digit(SelShared<R>& sh, ForEach&& for_each, uint32_t lo, SelDigits& s) {
  static_assert(kSelBins == 2 * kSelThreads, "two bins per thread");
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int width = s.shift < 11 ? s.shift : 11, sh0 = s.shift - width;
  const uint32_t dmask = (1u << width) - 1u, copy = (uint32_t)lane & (R - 1);
  asm volatile("" : "+v"(lo));   // (key - lo is made again for every digit, not kept beside the keys)
#pragma unroll
  for (int x = 0; x < 2 * R; ++x) sh.hist[x * kSelThreads + tid] = 0;
  __syncthreads();
  for_each([&](uint32_t key, bool valid) {
    const uint32_t d = key - lo;
    if (valid && d != 0u && (s.first || (d >> s.shift) == s.prefix)) atomicAdd(&sh.hist[R * ((d >> sh0) & dmask) + copy], 1u);
  });
  __syncthreads();
  // bins from the top: thread t takes the bins 2047 - 2 t and 2046 - 2 t
  uint32_t c0 = 0, c1 = 0;
#pragma unroll
  for (int x = 0; x < R; ++x) {
    c0 += sh.hist[R * (kSelBins - 1 - 2 * tid) + x];
    c1 += sh.hist[R * (kSelBins - 2 - 2 * tid) + x];
  }
  const bool has_lo = tid == kSelThreads - 1 && s.prefix == 0;   // the bin of lo: what the others leave
  const uint32_t but_lo = c1;
  if (has_lo) c1 = 0x7FFFFFFFu;
  uint32_t inc = c0 + c1;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t y = __shfl_up(inc, d);
    if (lane >= d) inc += y;
  }
  if (lane == 63) sh.wsum[wv] = inc;
  __syncthreads();
  uint32_t above = inc - c0 - c1;
#pragma unroll
  for (int x = 0; x < kSelWaves; ++x) above += x < wv ? sh.wsum[x] : 0u;
  if (above < s.krem && s.krem <= above + c0 + c1) {
    const bool second = above + c0 < s.krem;
    sh.digit = (uint32_t)(kSelBins - 1 - 2 * tid - (second ? 1 : 0));
    uint32_t rest = s.krem - above - (second ? c0 : 0u), in_bin = second ? c1 : c0;
    if (has_lo && second && rest > but_lo) {   // the kp-th is lo itself
      rest -= but_lo;
      in_bin = kSelAtLo;
    }
    sh.rest = rest;
    sh.in_bin = in_bin;
  }
  __syncthreads();
  s.prefix = s.first ? sh.digit : (s.prefix << width) | sh.digit;
  s.krem = sh.rest;
  s.in_bin = sh.in_bin;
  s.shift = sh0;
  s.first = false;
}
// The krem-th largest of the c <= kSelFew keys in sh.hist, for every thread.  (They are compared with one another: the bin that
// the first digit leaves of 6,000 to 48,000 scores has a few dozen, and a second and third digit took 1.2 us each.)
constexpr uint32_t kSelFew = 64;
template <int R>
__device__ __forceinline__ void sel_few(SelShared<R>& sh, uint32_t c, uint32_t krem, uint32_t& T, uint32_t& need_eq) {
  if (threadIdx.x < c) {
    const uint32_t mine = sh.hist[threadIdx.x];
    uint32_t above = 0, equal = 0;
    for (uint32_t x = 0; x < c; x += 8) {   // eight at a time: one trip to the LDS
      uint32_t y[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) y[e] = sh.hist[x + e];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if (x + e >= c) y[e] = 0u;   // (no key of a list is 0)
        above += y[e] > mine ? 1u : 0u;
        equal += y[e] == mine ? 1u : 0u;
      }
    }
    if (above < krem && krem <= above + equal) {   // (threads of equal keys write the same)
      const bool all = krem == above + equal;
      sh.few_T = mine - (all ? 1u : 0u);
      sh.few_need = all ? 0u : krem - above;
    }
  }
  __syncthreads();
  T = sh.few_T;
  need_eq = sh.few_need;
}
template <int R, typename ForEach>
__device__ __forceinline__ void radix_kth(SelShared<R>& sh, ForEach&& for_each, uint32_t kp, uint32_t lo, uint32_t hi, uint32_t& T,
                                          uint32_t& need_eq) {
  SelDigits s = sel_digits(kp, lo, hi);
  while (s.shift > 0) {                       // uniform: at most three times
    sel_digit(sh, for_each, lo, s);
    if (s.in_bin == kSelAtLo) break;
    if (s.krem == s.in_bin) {   // the whole bin is wanted: everything above the key below it
      T = lo + (s.prefix << s.shift) - 1u;
      need_eq = 0;
      return;
    }
  }
  T = lo + s.prefix;
  need_eq = s.krem;
}

// Emits one wave-wide group of 64 entries in order; gt / eq: entries above / equal to the threshold before it
__device__ __forceinline__ void sel_emit(const SelRow& r, uint32_t need_eq, bool is_g, bool is_e, int32_t index, uint32_t& gt,
                                         uint32_t& eq) {
  const uint64_t bg = __ballot(is_g), be = __ballot(is_e);
  if ((bg | be) == 0) return;
  const uint32_t gr = gt + __builtin_amdgcn_mbcnt_hi((uint32_t)(bg >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bg, 0u));
  const uint32_t er = eq + __builtin_amdgcn_mbcnt_hi((uint32_t)(be >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)be, 0u));
  if (is_g) r.out[r.f + gr + (er < need_eq ? er : need_eq)] = index;
  else if (is_e && er < need_eq) r.out[r.f + gr + er] = index;
  gt += __popcll(bg);
  eq += __popcll(be);
}
// The same where all keys equal to the threshold are wanted (they count as above it): one ballot instead of two
__device__ __forceinline__ void sel_emit(const SelRow& r, bool is_g, int32_t index, uint32_t& gt) {
  const uint64_t b = __ballot(is_g);
  if (is_g) r.out[r.f + gt + __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u))] = index;
  gt += __popcll(b);
}
// totals of the waves before this one (par: a parity, where a loop does this step after step)
template <int R>
__device__ __forceinline__ void sel_wave_base(SelShared<R>& sh, int par, uint32_t g, uint32_t e, uint32_t& gt, uint32_t& eq,
                                              uint32_t& all_g, uint32_t& all_e) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane == 0) { sh.wtot[par][wv][0] = g; sh.wtot[par][wv][1] = e; }
  __syncthreads();
  all_g = all_e = 0;
  for (int x = 0; x < kSelWaves; ++x) {
    const uint32_t g_ = sh.wtot[par][x][0], e_ = sh.wtot[par][x][1];
    if (x < wv) { gt += g_; eq += e_; }
    all_g += g_; all_e += e_;
  }
}

// A row in registers: KPT scores per thread, a wave's scores contiguous (KPT groups of 64).  After the first digit a pass over the
// scores lists the threshold's bin and counts every wave's scores above it; what a wave takes of the bin, and how many scores equal
// to the threshold, follows from the list, so that nearly every wave emits against one threshold.  (With two more digits, a count
// of both kinds and two ballots per group of 64, one counter per bin and 8, 16 or 32 scores per lane, 28 heads, 20,000 scores took 21.0
// us against 12.6, 32,768 20.9 against 15.4, 12,288 12.1 against 9.8, 4,096 8.4 against 6.9.)
// index(e): that of the lane's score e; settle: see RowIndex
template <int KPT, int R, typename Index>
__device__ __forceinline__ void sel_keys(SelShared<R>& sh, const SelRow& r, uint32_t (&key)[KPT], Index&& index) {
  const int wv = threadIdx.x >> 6;
  if (threadIdx.x == 0) sh.few = 0;
  if (threadIdx.x < kSelWaves) sh.extra[threadIdx.x] = 0;
  uint32_t lo = ~0u, hi = 0u, T, need_eq;
#pragma unroll
  for (int e = 0; e < KPT; ++e) {
    lo = key[e] - 1u < lo ? key[e] - 1u : lo;   // (a missing entry is no minimum)
    hi = key[e] > hi ? key[e] : hi;
  }
  sel_range(sh, lo, hi, lo, hi);
  ++lo;
  auto for_each = [&](auto&& f) {
    uint32_t none = 0u;
    if constexpr (KPT > 16) asm volatile("" : "+v"(none));   // (KPT lane masks held from pass to pass do not fit the scalar registers)
#pragma unroll
    for (int e = 0; e < KPT; ++e) f(key[e], key[e] != none);
  };
  SelDigits s = sel_digits(r.kp, lo, hi);
  bool few = false, whole = false;
  uint32_t g = 0, q = 0, gt = 0, eq = 0, ag, ae;
  while (s.shift > 0 && !few && !whole && s.in_bin != kSelAtLo) {
    sel_digit(sh, for_each, lo, s);
    whole = s.krem == s.in_bin;
    few = !whole && s.shift > 0 && s.in_bin <= kSelFew;
  }
  if (few) {
    // one pass lists the keys of the threshold's bin and counts the wave's keys above it; the wave's share of the bin follows
    uint32_t b0 = lo + (s.prefix << s.shift);
    asm volatile("" : "+v"(b0));
    const uint64_t b1 = (uint64_t)b0 + (1ull << s.shift) - 1u;
    const uint32_t top = b1 < 0xFFFFFFFFull ? (uint32_t)b1 : 0xFFFFFFFFu;
#pragma unroll
    for (int e = 0; e < KPT; ++e) {
      g += __popcll(__ballot(key[e] > top));
      if (key[e] - b0 <= top - b0) {
        const uint32_t at = atomicAdd(&sh.few, 1u);
        sh.hist[at] = key[e];
        sh.hist[kSelFew + at] = (uint32_t)wv;
      }
    }
    __syncthreads();
    sel_few(sh, s.in_bin, s.krem, T, need_eq);
    if (need_eq == 0) {
      if (threadIdx.x < s.in_bin && sh.hist[threadIdx.x] > T) atomicAdd(&sh.extra[sh.hist[kSelFew + threadIdx.x]], 1u);
      __syncthreads();
      g += sh.extra[wv];
    }
  } else {
    T = whole ? lo + (s.prefix << s.shift) - 1u : lo + s.prefix;
    need_eq = whole ? 0u : s.krem;
  }
  if (need_eq == 0) {
    if (!few)
#pragma unroll
      for (int e = 0; e < KPT; ++e) g += __popcll(__ballot(key[e] > T));
  } else {
    g = 0;
#pragma unroll
    for (int e = 0; e < KPT; ++e) {
      g += __popcll(__ballot(key[e] > T));
      q += __popcll(__ballot(key[e] == T));
    }
  }
  sel_wave_base(sh, 0, g, q, gt, eq, ag, ae);
  index.settle();
  asm volatile("" : "+v"(T));   // the lane masks are made again: KPT of them do not fit the scalar registers
  const uint32_t eq_s = __builtin_amdgcn_readfirstlane(eq), q_s = __builtin_amdgcn_readfirstlane(q), need_s = __builtin_amdgcn_readfirstlane(need_eq);
  if (eq_s >= need_s || eq_s + q_s <= need_s) {
    // of this wave's keys equal to T none is wanted, or all: they count as below or above the threshold
    if (eq_s < need_s) --T;
    gt += eq_s < need_s ? eq_s : need_s;
#pragma unroll
    for (int e = 0; e < KPT; ++e) sel_emit(r, key[e] > T, index(e), gt);
  } else {
#pragma unroll
    for (int e = 0; e < KPT; ++e) sel_emit(r, need_eq, key[e] > T, key[e] == T, index(e), gt, eq);
  }
}

template <int KPT>
struct RowIndex {
  int i0;
  __device__ __forceinline__ void settle() {
    if constexpr (KPT > 32) asm volatile("" : "+v"(i0));   // (the indices are made again: held from the loads on they were what spilled)
  }
  __device__ __forceinline__ int operator()(int e) const { return i0 + 64 * e; }
};
template <int KPT, int R>
__device__ __forceinline__ void sel_from_registers(SelShared<R>& sh, const SelRow& r, int64_t n) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  RowIndex<KPT> index = {r.f + wv * (64 * KPT) + lane};
  uint32_t key[KPT];
#pragma unroll
  for (int e = 0; e < KPT; ++e) {
    const int i = index(e);
    const uint32_t x = order_key(r.sc[i < n ? i : (int)n - 1]);   // unconditional, so that the loads overlap
    key[e] = i < n ? x : 0u;   // no finite score has key 0: neither counted nor emitted below
  }
  sel_keys<KPT>(sh, r, key, index);
}
// The m <= 1,024 KPT candidates of a row whose at most kSelBins slices lie anywhere in its list (the filter's), into registers in the
// order of their indices: the slices' places from a sum over their lengths, a candidate's slice by bisection in LDS, all of a lane's
// at once.  (Copied to LDS as they lay there and brought in order 64 at a time by bisection over lanes, for the count and again
// for the compaction, three digits: 28 heads, 50,000 scores 35.5 us, 24.4 so, 300,001
// 54.8 and 46.5, 1M 103 and 90.)
template <int KPT>
struct ListIndex {
  int at[KPT];
  __device__ __forceinline__ void settle() {}
  __device__ __forceinline__ int operator()(int e) const { return at[e]; }
};
template <int KPT, int R>
__device__ __forceinline__ void sel_from_list(SelShared<R>& sh, uint32_t (&place)[kSelBins], const uint2* cand, const uint2* slices,
                                              const SelRow& r, int n_slices, int m) {
  static_assert(kSelBins == 2 * kSelThreads, "two slices per thread");
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const uint2 none = make_uint2(0u, 0u), s0 = 2 * tid < n_slices ? slices[2 * tid] : none, s1 = 2 * tid + 1 < n_slices ? slices[2 * tid + 1] : none;
  uint32_t inc = s0.y + s1.y;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t y = __shfl_up(inc, d);
    if (lane >= d) inc += y;
  }
  if (lane == 63) sh.wsum[wv] = inc;
  __syncthreads();
  uint32_t at = inc - s0.y - s1.y;
#pragma unroll
  for (int x = 0; x < kSelWaves; ++x) at += x < wv ? sh.wsum[x] : 0u;
  sh.hist[2 * tid] = at;
  sh.hist[2 * tid + 1] = at + s0.y;
  place[2 * tid] = s0.x - at;
  place[2 * tid + 1] = s1.x - at - s0.y;
  __syncthreads();
  const int first = wv * (64 * KPT) + lane;
  int j[KPT];
#pragma unroll
  for (int e = 0; e < KPT; ++e) j[e] = 0;
  for (int d = n_slices > 1 ? 1 << (31 - __clz(n_slices - 1)) : 0; d >= 1; d >>= 1)
#pragma unroll
    for (int e = 0; e < KPT; ++e)
      if (sh.hist[j[e] + d] <= (uint32_t)(first + 64 * e)) j[e] += d;   // (places behind the last slice are m)
  ListIndex<KPT> index;
  uint32_t key[KPT];
#pragma unroll
  for (int e = 0; e < KPT; ++e) {
    const int i = first + 64 * e;
    const uint2 c = cand[i < m ? (uint32_t)i + place[j[e]] : 0u];
    key[e] = i < m ? c.x : 0u;
    index.at[e] = (int)c.y;
  }
  sel_keys<KPT>(sh, r, key, index);
}

// The m candidates of a row (keys above floor_key, with their indices), in n_slices slices: slice_of(s) = (first candidate,
// candidates).  Slices lie there in any order; the entries of a slice ascend, and so do the slices' indices.  The ordered
// compaction gives every wave consecutive slices that hold about an equal share of the candidates (the best offsets crowd near the
// diagonal: with equal numbers of slices one wave had half of the 10,000 candidates of a 1M-key row, 45 us against 29).
template <int R, typename SliceOf>
__device__ __forceinline__ void sel_from_candidates(SelShared<R>& sh, const uint2* cl, const SelRow& r, int n_slices, int m,
                                                    uint32_t floor_key, SliceOf&& slice_of) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint32_t T, need_eq, hi = 0u, lo;
  for (int i = tid; i < m; i += kSelThreads) hi = cl[i].x > hi ? cl[i].x : hi;
  sel_range(sh, 0u, hi, lo, hi);
  radix_kth(sh, [&](auto&& f) {
    for (int i = tid; i < m; i += kSelThreads) f(cl[i].x, true);
  }, r.kp, floor_key + 1u, hi, T, need_eq);
  // sh.first[w]: the first slice that starts at or past candidate w m / kSelWaves of the ordered list
  if (tid <= kSelWaves) sh.first[tid] = n_slices;
  uint32_t before = 0;   // candidates of the slices before this round's
  for (int sb = 0; sb < n_slices; sb += kSelThreads) {
    const int s = sb + tid;
    const uint32_t c = s < n_slices ? slice_of(s).y : 0u, c_prev = s > 0 && s < n_slices ? slice_of(s - 1).y : 0u;
    uint32_t inc = c;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t y = __shfl_up(inc, d);
      if (lane >= d) inc += y;
    }
    __syncthreads();   // (wsum's last readers; sh.first)
    if (lane == 63) sh.wsum[wv] = inc;
    __syncthreads();
    uint32_t at = before + inc - c;
    for (int x = 0; x < kSelWaves; ++x) {
      at += x < wv ? sh.wsum[x] : 0u;
      before += sh.wsum[x];
    }
    if (s < n_slices) {
      const int w1 = (int)((uint64_t)at * kSelWaves / (uint32_t)m);
      const int w0 = s > 0 ? (int)((uint64_t)(at - c_prev) * kSelWaves / (uint32_t)m) + 1 : 0;
      for (int w = w0; w <= w1; ++w) sh.first[w] = s;
    }
  }
  __syncthreads();
  const int s0 = __builtin_amdgcn_readfirstlane(sh.first[wv]), s1 = __builtin_amdgcn_readfirstlane(sh.first[wv + 1]);
  // 64 slices at a time: a lane of a group of 64 consecutive candidates finds its slice by bisection over the lanes
  auto walk = [&](auto&& f) {
    for (int sb = s0; sb < s1; sb += 64) {
      const uint2 mine = sb + lane < s1 ? slice_of(sb + lane) : make_uint2(0u, 0u);
      int end = (int)mine.y;   // candidates up to and with this lane's slice
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const int y = __shfl_up(end, d);
        if (lane >= d) end += y;
      }
      const int shift = (int)mine.x - (end - (int)mine.y);   // place in the list, less the place in the order
      const int total = __builtin_amdgcn_readlane(end, 63);
      constexpr int U = 4;
      for (int i = 0; i < total; i += 64 * U) {
        int p[U], j[U];
        uint2 c[U];
#pragma unroll
        for (int e = 0; e < U; ++e) {
          p[e] = i + 64 * e + lane < total ? i + 64 * e + lane : total - 1;
          j[e] = 0;
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1)
#pragma unroll
          for (int e = 0; e < U; ++e)
            if (__shfl(end, j[e] + d - 1) <= p[e]) j[e] += d;
#pragma unroll
        for (int e = 0; e < U; ++e) c[e] = cl[p[e] + __shfl(shift, j[e])];
#pragma unroll
        for (int e = 0; e < U; ++e) {
          const bool in = i + 64 * e + lane < total;
          f(in && c[e].x > T, in && c[e].x == T, (int32_t)c[e].y);
        }
      }
    }
  };
  uint32_t g = 0, q = 0, gt = 0, eq = 0, ag, ae;
  if (need_eq == 0) {   // no two kinds to tell apart
    walk([&](bool is_g, bool, int32_t) { g += __popcll(__ballot(is_g)); });
    sel_wave_base(sh, 0, g, q, gt, eq, ag, ae);
    walk([&](bool is_g, bool, int32_t index) { sel_emit(r, is_g, index, gt); });
    return;
  }
  walk([&](bool is_g, bool is_e, int32_t) {
    g += __popcll(__ballot(is_g));
    q += __popcll(__ballot(is_e));
  });
  sel_wave_base(sh, 0, g, q, gt, eq, ag, ae);
  walk([&](bool is_g, bool is_e, int32_t index) { sel_emit(r, need_eq, is_g, is_e, index, gt, eq); });
}

// Steps over a row in order: step(key, i0, par) gets kSelStep groups of 64 entries per wave (key[e] is the image of entry
// i0 + 64 e, 0 behind the row's end), a wave's entries contiguous and the waves one after the other; par alternates.  It
// returns whether to go on (uniform).  The scores of the next step are on their way meanwhile.
template <typename Step>
__device__ __forceinline__ void sel_walk_row(const SelRow& r, int64_t n, Step&& step) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  int par = 0;
  float next[kSelStep];
  constexpr int kLen = kSelThreads * kSelStep;
  const int at = wv * (64 * kSelStep) + lane;   // of this lane's first entry inside a step
  auto fetch = [&](int64_t base) {
    if (base + kLen <= n) {   // a whole step: one address
      const float* const p = r.sc + base;
#pragma unroll
      for (int e = 0; e < kSelStep; ++e) next[e] = p[at + 64 * e];
    } else {
#pragma unroll
      for (int e = 0; e < kSelStep; ++e) {
        const int64_t i = base + at + 64 * e;
        next[e] = r.sc[i < n ? i : n - 1];
      }
    }
  };
  fetch(r.f);
  for (int64_t base = r.f; base < n; base += kLen, par ^= 1) {
    uint32_t key[kSelStep];
    const int left = n - base < kLen ? (int)(n - base) : kLen;
#pragma unroll
    for (int e = 0; e < kSelStep; ++e) key[e] = at + 64 * e < left ? order_key(next[e]) : 0u;
    fetch(base + kLen);
    if (!step(key, (int32_t)base + at, par)) break;
  }
}

// The ordered compaction of a row whose threshold is known, as far as the row has to be read: until it is complete or, where a
// list holds the keys > T (`listed`), until the equal ones are (the smallest scores, if most of a row's are the same: a few
// thousand entries).  Returns how many of the keys > T it has met.
template <bool listed, int R>
__device__ __forceinline__ uint32_t sel_compact_row(SelShared<R>& sh, const SelRow& r, int64_t n, uint32_t T, uint32_t need_eq) {
  uint32_t run_g = 0, run_e = 0;
  sel_walk_row(r, n, [&](const uint32_t (&key)[kSelStep], int32_t i0, int par) {
    uint32_t g = 0, q = 0;
#pragma unroll
    for (int e = 0; e < kSelStep; ++e) {
      g += __popcll(__ballot(key[e] > T));
      q += __popcll(__ballot(key[e] == T));
    }
    uint32_t gt = run_g, eq = run_e, all_g, all_e;
    sel_wave_base(sh, par, g, q, gt, eq, all_g, all_e);
#pragma unroll
    for (int e = 0; e < kSelStep; ++e) sel_emit(r, need_eq, key[e] > T, key[e] == T, i0 + 64 * e, gt, eq);
    run_g += all_g;
    run_e += all_e;
    if (listed) return run_e < need_eq;
    return run_g + (run_e < need_eq ? run_e : need_eq) < r.kp;   // else the row is complete
  });
  return run_g;
}

// The candidates of a row from number `from` of the order on, for a row all of whose candidates are wanted, behind `equal` other
// entries.  1,024 slices at a time: their places in the order, then 16 lanes per slice.
template <int R, typename SliceOf>
__device__ __forceinline__ void sel_copy_candidates(SelShared<R>& sh, const uint2* cl, const SelRow& r, int n_slices, uint32_t from,
                                                    uint32_t equal, SliceOf&& slice_of) {
  static_assert(kSelBins == 2 * kSelThreads, "two words per thread");
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  uint32_t before = 0;   // candidates of the slices before this round's
  for (int sb = 0; sb < n_slices; sb += kSelThreads) {
    const uint2 mine = sb + tid < n_slices ? slice_of(sb + tid) : make_uint2(0u, 0u);
    uint32_t inc = mine.y;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t y = __shfl_up(inc, d);
      if (lane >= d) inc += y;
    }
    __syncthreads();   // (the last readers of wsum and hist)
    if (lane == 63) sh.wsum[wv] = inc;
    __syncthreads();
    uint32_t at = before + inc - mine.y;
    for (int x = 0; x < kSelWaves; ++x) {
      at += x < wv ? sh.wsum[x] : 0u;
      before += sh.wsum[x];
    }
    sh.hist[tid] = at;
    sh.hist[kSelThreads + tid] = mine.x;
    __syncthreads();
    for (int t = tid >> 4; t < kSelThreads; t += kSelThreads / 16) {
      const uint32_t a = sh.hist[t], end = t + 1 < kSelThreads ? sh.hist[t + 1] : before, first = sh.hist[kSelThreads + t];
      uint32_t i = (a < from ? from : a) + (tid & 15);
      for (; i < end; i += 16) r.out[r.f + equal + i] = (int32_t)cl[first + (i - a)].y;
    }
  }
}

// A row read from memory for its range, once per digit and once more for the compaction.
template <int R>
__device__ __forceinline__ void sel_from_row(SelShared<R>& sh, const SelRow& r, int64_t n) {
  uint32_t lo = ~0u, hi = 0u, T, need_eq;
  sel_walk_row(r, n, [&](const uint32_t (&key)[kSelStep], int32_t, int) {
#pragma unroll
    for (int e = 0; e < kSelStep; ++e) {
      lo = key[e] - 1u < lo ? key[e] - 1u : lo;
      hi = key[e] > hi ? key[e] : hi;
    }
    return true;
  });
  sel_range(sh, lo, hi, lo, hi);
  radix_kth(sh, [&](auto&& f) {
    sel_walk_row(r, n, [&](const uint32_t (&key)[kSelStep], int32_t, int) {
#pragma unroll
      for (int e = 0; e < kSelStep; ++e) f(key[e], key[e] != 0u);
      return true;
    });
  }, r.kp, lo + 1u, hi, T, need_eq);
  sel_compact_row<false>(sh, r, n, T, need_eq);
}

// The floor of a row's candidates: one score from each of SPT x kSelThreads stretches of the row (at a place inside its
// stretch that a hash of its number gives), and among these the one at sel_sample_rank.
template <int SPT, int R>
__device__ __forceinline__ uint32_t sel_floor(SelShared<R>& sh, const SelRow& r, int64_t n) {
  constexpr int S = SPT * kSelThreads;
  const int64_t m = n - r.f;   // more than 2 S entries
  const float rank = sel_sample_rank((float)r.kp, (float)m, (float)S);
  if (!(rank < (float)S)) return 0u;   // (nearly) everything is wanted
  const uint32_t len = (uint32_t)(m / S);
  uint32_t key[SPT], lo = ~0u, hi = 0u, T, need_eq;
#pragma unroll
  for (int e = 0; e < SPT; ++e) {
    const uint32_t x = (uint32_t)(e * kSelThreads) + threadIdx.x;
    const uint32_t hash = (x * 0x9E3779B1u) >> 16;
    key[e] = order_key(r.sc[r.f + (int64_t)((uint64_t)m * x / S) + ((uint64_t)hash * len >> 16)]);
  }
#pragma unroll
  for (int e = 0; e < SPT; ++e) {
    lo = key[e] < lo ? key[e] : lo;
    hi = key[e] > hi ? key[e] : hi;
  }
  sel_range(sh, lo, hi, lo, hi);
  radix_kth(sh, [&](auto&& f) {
#pragma unroll
    for (int e = 0; e < SPT; ++e) f(key[e], true);
  }, (uint32_t)rank, lo, hi, T, need_eq);
  return T;   // (the floor may lie just below the sample of that rank: everything above it is a candidate)
}

template <int R>
__device__ __forceinline__ uint32_t sel_floor(SelShared<R>& sh, const SelRow& r, int64_t n, int samples) {
  return samples == 4 ? sel_floor<4>(sh, r, n) : samples == 8 ? sel_floor<8>(sh, r, n) : sel_floor<16>(sh, r, n);
}

// KPT: scores per thread of a row in registers; 0: a long row.
template <int KPT>
__global__ __launch_bounds__(kSelThreads) void k_sel_row(const SelArgs a) {
  __shared__ SelShared<sel_copies(KPT)> sh;
  extern __shared__ __attribute__((aligned(16))) unsigned char sel_dyn[];
  const int tid = threadIdx.x;
  SelRow r = sel_row(a, blockIdx.x);
  if (r.k == a.n) { r.f = r.k; r.kp = 0; }   // the row is wanted whole
  for (int t = tid; t < r.row_len; t += kSelThreads) {
    if (t < r.f) r.out[t] = t;
    else if (t >= r.k) r.out[t] = -1;
  }
  if (tid == 0) (r.kind ? a.s_cnt : a.v_cnt)[r.h] = r.k;
  if (r.kp == 0) return;
  if constexpr (KPT > 0) {
    sel_from_registers<KPT>(sh, r, a.n);
  } else {
    uint2* const cl = (uint2*)sel_dyn;
    __shared__ uint32_t place[kSelBins];
    const int samples = r.kind ? a.samples_s : a.samples_v;
    const bool listed = a.hdr != nullptr;   // the filter made the list
    uint32_t room = listed ? a.cap : (uint32_t)kSelCand;
    SelHeader hd;
    if (listed) {
      hd = a.hdr[blockIdx.x];
    } else {
      hd.floor_key = sel_floor(sh, r, a.n, samples);
      hd.count = hd.equal = 0;
      sel_walk_row(r, a.n, [&](const uint32_t (&key)[kSelStep], int32_t i0, int par) {
        uint32_t g = 0, q = 0;
#pragma unroll
        for (int e = 0; e < kSelStep; ++e) {
          g += __popcll(__ballot(key[e] > hd.floor_key));
          q += __popcll(__ballot(key[e] == hd.floor_key));
        }
        uint32_t at = hd.count, eq = 0, all_g, all_e;
        sel_wave_base(sh, par, g, q, at, eq, all_g, all_e);
        hd.count += all_g;
        hd.equal += all_e;
        if (hd.count > room) return false;
#pragma unroll
        for (int e = 0; e < kSelStep; ++e) {
          const uint64_t b = __ballot(key[e] > hd.floor_key);
          if (!b) continue;
          if (key[e] > hd.floor_key)
            cl[at + __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u))] =
                make_uint2(key[e], (uint32_t)(i0 + 64 * e));
          at += __popcll(b);
        }
        return true;
      });
      __syncthreads();
    }
    const int m = (int)hd.count;
    const uint2* const cand = a.cand + (int64_t)blockIdx.x * a.cap;
    const uint2* const slices = a.slices + (int64_t)blockIdx.x * a.n_slices;
    auto slice_of = [&](int s) { return slices[s]; };
    if (hd.count > room || hd.count + hd.equal < r.kp) {   // the sample missed
      sel_from_row(sh, r, a.n);
    } else if (hd.count < r.kp) {   // the threshold is the floor
      const uint32_t equal = r.kp - hd.count, met = sel_compact_row<true>(sh, r, a.n, hd.floor_key, equal);
      if (listed) sel_copy_candidates(sh, cand, r, a.n_slices, met, equal, slice_of);
      else
        for (int i = (int)met + tid; i < m; i += kSelThreads) r.out[r.f + equal + i] = (int32_t)cl[i].y;
    } else if (listed) {
      if (m <= kSelCand && a.n_slices <= kSelBins) {
        static_assert(kSelCand == 16 * kSelThreads, "the longest list in registers");
        if (m <= 8 * kSelThreads) sel_from_list<8>(sh, place, cand, slices, r, a.n_slices, m);
        else if (m <= 12 * kSelThreads) sel_from_list<12>(sh, place, cand, slices, r, a.n_slices, m);
        else sel_from_list<16>(sh, place, cand, slices, r, a.n_slices, m);
      } else {
        sel_from_candidates(sh, cand, r, a.n_slices, m, hd.floor_key, slice_of);
      }
    } else {
      // (in order already: one slice per wave)
      const int per = (m + kSelWaves - 1) / kSelWaves;
      sel_from_candidates(sh, cl, r, kSelWaves, m, hd.floor_key, [&](int s) {
        const int at = s * per < m ? s * per : m;
        return make_uint2((uint32_t)at, (uint32_t)(m - at < per ? m - at : per));
      });
    }
  }
}

// Headers of the rows with their floors: one workgroup per row.
__global__ __launch_bounds__(kSelThreads) void k_sel_sample(const SelArgs a) {
  __shared__ SelShared<1> sh;
  const SelRow r = sel_row(a, blockIdx.x);
  SelHeader hd;
  hd.floor_key = ~0u;   // (all entries of the row are forced: no candidates)
  if (r.kp > 0) hd.floor_key = sel_floor(sh, r, a.n, r.kind ? a.samples_s : a.samples_v);
  hd.count = hd.equal = 0;
  hd.pad = 0;
  if (threadIdx.x == 0) a.hdr[blockIdx.x] = hd;
}

// The candidates of a row's slices: the scores are read once, counted, given room in the row's list by one atomic
// addition per workgroup (so the slices lie there in the order of arrival; k_sel_row goes by the table) and written in order,
// a slice per wave.  Four consecutive scores per lane and load, counted in the lane: with one per lane and load and two population
// counts per 64 scores, 28 heads, 300,001 scores 17.4 us, 15.7 so, 1M 61 and 57 (4.1 TB/s).
__global__ __launch_bounds__(kSelFilterThreads) void k_sel_filter(const SelArgs a) {
  const SelRow r = sel_row(a, blockIdx.y);
  SelHeader* const hd = a.hdr + blockIdx.y;
  constexpr int NW = kSelFilterThreads / 64, PER = kSelSlice / 64;
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  // entries and floor as signed integers in the order of the scores.  Against a floor >= 0 (scores are) the bits of a float
  // are that integer already: a negative float is a negative integer, whatever its place among those.
  const uint32_t floor_key = hd->floor_key;
  int32_t floor_x = (int32_t)(floor_key ^ 0x80000000u);
  const int slice = blockIdx.x * NW + wv;
  const int64_t s0 = r.f + (int64_t)slice * kSelSlice;
  __shared__ uint32_t wcnt[NW][2], base_s;
  // entry 4 e + f: 256 e + 4 lane + f of the slice (rows start at any word)
  int32_t x[PER];
  typedef int32_t i32x4 __attribute__((ext_vector_type(4), aligned(4)));
  if (s0 + kSelSlice <= a.n) {   // a whole slice: one address
    const int32_t* const p = (const int32_t*)r.sc + s0;
#pragma unroll
    for (int e = 0; e < PER / 4; ++e) {
      const i32x4 v = *(const i32x4*)(p + 256 * e + 4 * lane);
#pragma unroll
      for (int f = 0; f < 4; ++f) x[4 * e + f] = v[f];
    }
  } else {
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int64_t i = s0 + 256 * (e / 4) + 4 * lane + e % 4;
      const int32_t b = ((const int32_t*)r.sc)[i < a.n ? i : a.n - 1];
      x[e] = i < a.n ? b : (int32_t)0xFFFFFFFF;   // behind the row: the image is the least one
    }
  }
  if (floor_x < 0) {
#pragma unroll
    for (int e = 0; e < PER; ++e) x[e] ^= (x[e] >> 31) & 0x7FFFFFFF;
  }
  uint32_t c = 0, q = 0;   // of the lane first: entries above the floor, and at or above it
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    c += x[e] > floor_x ? 1u : 0u;
    q += x[e] >= floor_x ? 1u : 0u;
  }
  uint32_t both = c | q << 16;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) both += __shfl_xor(both, d);
  c = __builtin_amdgcn_readfirstlane(both & 0xFFFFu);
  q = __builtin_amdgcn_readfirstlane(both >> 16) - c;
  if (lane == 0) { wcnt[wv][0] = c; wcnt[wv][1] = q; }
  __syncthreads();
  uint32_t before = 0, total = 0, equal = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    before += w < wv ? wcnt[w][0] : 0u;
    total += wcnt[w][0];
    equal += wcnt[w][1];
  }
  if (tid == 0) {
    base_s = total ? __hip_atomic_fetch_add(&hd->count, total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
    if (equal) __hip_atomic_fetch_add(&hd->equal, equal, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  const uint32_t base = base_s;
  if (lane == 0 && slice < a.n_slices) a.slices[(int64_t)blockIdx.y * a.n_slices + slice] = make_uint2(base + before, c);
  if (base + total > a.cap || c == 0) return;   // (the list overflows: k_sel_row reads the row instead)
  uint2* const out = a.cand + (int64_t)blockIdx.y * a.cap + base + before;
  uint32_t pos = 0;
  asm volatile("" : "+s"(floor_x));   // the lane masks are made again rather than kept
#pragma unroll
  for (int e = 0; e < PER / 4; ++e) {
    uint64_t b[4];
    uint32_t at = pos;
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      b[f] = __ballot(x[4 * e + f] > floor_x);
      at = __builtin_amdgcn_mbcnt_hi((uint32_t)(b[f] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b[f], at));
    }
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      if (x[4 * e + f] > floor_x) {
        out[at] = make_uint2((uint32_t)x[4 * e + f] ^ 0x80000000u, (uint32_t)(s0 + 256 * e + 4 * lane + f));
        ++at;
      }
      pos += __popcll(b[f]);
    }
  }
}

// ---- rows in slices ---------------------------------------------------------------------------
constexpr int64_t kSliceStep = (int64_t)kSelStep * kSelThreads;

// Forced entries, padding, the count, and a cleared control block.
__global__ __launch_bounds__(256) void k_slice_init(const SelArgs a) {
  const SelRow r = sel_row(a, blockIdx.x);
  uint32_t* const ctl = a.ctl + (int64_t)blockIdx.x * kSliceRowWords;
  const int tid = threadIdx.x;
  for (int x = tid; x < kSliceRowWords; x += 256) ctl[x] = x == kWState + 1 ? r.kp : 0u;
  for (int t = tid; t < r.row_len; t += 256) {
    if (t < r.f) r.out[t] = t;
    else if (t >= r.k) r.out[t] = -1;
  }
  if (tid == 0) (r.kind ? a.s_cnt : a.v_cnt)[r.h] = r.k;
}

// One digit of the radix select: threshold key T = kp-th largest key among the candidates.
__global__ __launch_bounds__(kSelThreads) void k_slice_digit(const SelArgs a, const int pass) {
  const SelRow r = sel_row(a, blockIdx.y);
  uint32_t* const ctl = a.ctl + (int64_t)blockIdx.y * kSliceRowWords;
  if (r.kp == 0) return;
  const int64_t lo = (int64_t)r.f + (int64_t)blockIdx.x * a.slice_len;
  const int64_t hi = lo + a.slice_len < a.n ? lo + a.slice_len : a.n;
  const uint32_t prefix = ctl[kWState + 2 * pass], krem = ctl[kWState + 2 * pass + 1];
  const int tid = threadIdx.x, lane = tid & 63;
  // 16 copies of the 256-bin histogram, copy = lane % 16 in consecutive banks: the top digits of
  // real scores crowd into a few bins, and 64 lanes adding to one address would serialise
  __shared__ uint32_t hist16[256 * 16];
  __shared__ uint32_t hist[256];
  __shared__ bool last;
  const int shift = 24 - 8 * pass;
  const uint32_t himask = pass == 0 ? 0u : (0xFFFFFFFFu << (shift + 8));
  for (int x = tid; x < 256 * 16; x += kSelThreads) hist16[x] = 0;
  __syncthreads();
  // kSelStep independent loads per thread in flight (the pass is latency-bound otherwise)
  for (int64_t base = lo; base < hi; base += kSliceStep) {
    uint32_t key[kSelStep];
    bool ok[kSelStep];
#pragma unroll
    for (int e = 0; e < kSelStep; ++e) {
      const int64_t i = base + (int64_t)e * kSelThreads + tid;
      ok[e] = i < hi;
      key[e] = order_key(r.sc[ok[e] ? i : hi - 1]);  // unconditional, so that the loads overlap
    }
#pragma unroll
    for (int e = 0; e < kSelStep; ++e)
      if (ok[e] && (key[e] & himask) == prefix)
        atomicAdd(&hist16[(((key[e] >> shift) & 255u) << 4) | (lane & 15)], 1u);
  }
  __syncthreads();
  uint32_t* const gh = ctl + kWHist + 256 * pass;
  // The additions and the ticket are device-wide atomics, performed where all workgroups see
  // them.  The additions return a value, and the wait for it is the wait for their completion;
  // only then does the workgroup draw its ticket, so the one that draws the last ticket finds
  // every addition done.  (No cache is involved: a fence would write back the whole L2.)
  if (tid < 256) {
    uint32_t c = 0;
#pragma unroll
    for (int x = 0; x < 16; ++x) c += hist16[(tid << 4) | x];
    uint32_t old = 0;
    if (c) old = __hip_atomic_fetch_add(&gh[tid], c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" : "+v"(old) : : "memory");
  }
  __syncthreads();
  if (tid == 0)
    last = __hip_atomic_fetch_add(&ctl[kWDone + pass], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
  __syncthreads();
  if (!last) return;
  if (tid < 256) hist[tid] = __hip_atomic_load(&gh[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (tid == 0) {
    uint32_t cum = 0;
    int b = 255;
    for (; b > 0; --b) {
      const uint32_t c = hist[b];
      if (cum + c >= krem) break;
      cum += c;
    }
    ctl[kWState + 2 * (pass + 1)] = prefix | ((uint32_t)b << shift);
    ctl[kWState + 2 * (pass + 1) + 1] = krem - cum;
  }
}

// Keys above and equal to the threshold in every slice.
__global__ __launch_bounds__(kSelThreads) void k_slice_count(const SelArgs a) {
  const SelRow r = sel_row(a, blockIdx.y);
  uint32_t* const ctl = a.ctl + (int64_t)blockIdx.y * kSliceRowWords;
  if (r.kp == 0) return;
  const int64_t lo = (int64_t)r.f + (int64_t)blockIdx.x * a.slice_len;
  const int64_t hi = lo + a.slice_len < a.n ? lo + a.slice_len : a.n;
  const uint32_t T = ctl[kWState + 8];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  __shared__ uint32_t wtot[kSelWaves][2];
  uint32_t tg = 0, te = 0;
  for (int64_t base = lo; base < hi; base += kSliceStep) {
    uint32_t key[kSelStep];
#pragma unroll
    for (int e = 0; e < kSelStep; ++e) {
      const int64_t i = base + (int64_t)e * kSelThreads + tid;
      key[e] = order_key(r.sc[i < hi ? i : hi - 1]);
    }
#pragma unroll
    for (int e = 0; e < kSelStep; ++e) {
      const bool in = base + (int64_t)e * kSelThreads + tid < hi;
      tg += __popcll(__ballot(in && key[e] > T));
      te += __popcll(__ballot(in && key[e] == T));
    }
  }
  if (lane == 0) { wtot[wv][0] = tg; wtot[wv][1] = te; }
  __syncthreads();
  if (tid == 0) {
    uint32_t g = 0, e = 0;
    for (int w = 0; w < kSelWaves; ++w) { g += wtot[w][0]; e += wtot[w][1]; }
    ctl[kWCount + 2 * blockIdx.x] = g;
    ctl[kWCount + 2 * blockIdx.x + 1] = e;
  }
}

// Ordered compaction of one slice.
__global__ __launch_bounds__(kSelThreads) void k_slice_write(const SelArgs a) {
  const SelRow r = sel_row(a, blockIdx.y);
  const uint32_t* const ctl = a.ctl + (int64_t)blockIdx.y * kSliceRowWords;
  const uint32_t kp = r.kp;
  if (kp == 0) return;
  const int f = r.f;
  const int64_t lo = (int64_t)f + (int64_t)blockIdx.x * a.slice_len;
  const int64_t hi = lo + a.slice_len < a.n ? lo + a.slice_len : a.n;
  const uint32_t T = ctl[kWState + 8];
  const uint32_t need_eq = ctl[kWState + 9];  // >= 1
  int32_t* const out = r.out;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  __shared__ uint32_t wtot[2][kSelWaves][2];
  uint32_t run_gt = 0, run_eq = 0;  // totals over everything before this slice, then before the step
  for (int sl = 0; sl < (int)blockIdx.x; ++sl) {
    run_gt += ctl[kWCount + 2 * sl];
    run_eq += ctl[kWCount + 2 * sl + 1];
  }
  if (run_gt + (run_eq < need_eq ? run_eq : need_eq) >= kp) return;  // the row is complete already
  const uint64_t lt_mask = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  int par = 0;
  for (int64_t base = lo; base < hi; base += kSliceStep, par ^= 1) {
    uint64_t bg[kSelStep], be[kSelStep];
    uint32_t tg = 0, te = 0, keys[kSelStep];
#pragma unroll
    for (int e = 0; e < kSelStep; ++e) {
      const int64_t i = base + (int64_t)wv * (64 * kSelStep) + e * 64 + lane;
      keys[e] = order_key(r.sc[i < hi ? i : hi - 1]);
    }
#pragma unroll
    for (int e = 0; e < kSelStep; ++e) {
      const int64_t i = base + (int64_t)wv * (64 * kSelStep) + e * 64 + lane;
      const uint32_t key = keys[e];
      bg[e] = __ballot(i < hi && key > T);
      be[e] = __ballot(i < hi && key == T);
      tg += __popcll(bg[e]);
      te += __popcll(be[e]);
    }
    if (lane == 0) { wtot[par][wv][0] = tg; wtot[par][wv][1] = te; }
    __syncthreads();
    uint32_t gt_before = run_gt, eq_before = run_eq, cg = 0, ce = 0;
    for (int w = 0; w < kSelWaves; ++w) {
      const uint32_t g_ = wtot[par][w][0], e_ = wtot[par][w][1];
      if (w < wv) { gt_before += g_; eq_before += e_; }
      cg += g_; ce += e_;
    }
#pragma unroll
    for (int e = 0; e < kSelStep; ++e) {
      const int64_t i = base + (int64_t)wv * (64 * kSelStep) + e * 64 + lane;
      const uint32_t gr = gt_before + __popcll(bg[e] & lt_mask);
      const uint32_t er = eq_before + __popcll(be[e] & lt_mask);
      const bool is_g = (bg[e] >> lane) & 1ull, is_e = (be[e] >> lane) & 1ull;
      if (is_g) out[f + gr + (er < need_eq ? er : need_eq)] = (int32_t)i;
      else if (is_e && er < need_eq) out[f + gr + er] = (int32_t)i;
      gt_before += __popcll(bg[e]);
      eq_before += __popcll(be[e]);
    }
    run_gt += cg;
    run_eq += ce;
    if (run_gt + (run_eq < need_eq ? run_eq : need_eq) >= kp) break;
  }
}

// Entries that a row's list may get: what is to be expected from the sample and 4.5 sigma of it to spare.
static int64_t sel_list_len(int64_t n, int32_t budget, int spt) {
  const float s = (float)(spt * kSelThreads), rank = sel_sample_rank((float)budget, (float)n, s);
  if (!(rank < s)) return n;
  const int64_t len = (int64_t)((rank + 4.5f * sqrtf(rank)) * ((float)n / s)) + 64;
  return len < n ? len : n;
}
// Samples per thread: the smallest number whose list fits the registers, else the largest; 0: the rows stay in registers.  The samples
// of a row lie in a cache line each, which one compute unit fetches (8,192 of them a megabyte): half as many and a list a sixth longer,
// 28 heads, 300,001 scores 44.2 us -> 40.8, four heads 23.6 -> 21.8, 1M 36.0 -> 31.1; a quarter as many 44.3, 21.1, 30.9.
// least: no fewer than eight, with which the list is shorter.
static int sel_samples(int64_t n, int32_t budget, bool least) {
  if (n <= kSelRegKeys) return 0;
  if (!least && sel_list_len(n, budget, 4) <= kSelCand) return 4;
  return sel_list_len(n, budget, 8) <= kSelCand ? 8 : 16;
}
// The longest list that is worth making.  The row's one workgroup takes about 1.45 us per 1,000 candidates, and the slices
// read the scores seven times.  Measured over 1 to 64 heads, 50,000 to 4M keys and 8,000 to 106,000 candidates, with lists
// against in slices (us): break-even at 26,000 candidates for two rows of 50,000 keys (70), 33,000 for 56 (90), 39,000 for two
// of 1M (88), 52,000 for eight of 1M (118), 74,000 for 56 of 300,001 (170); the line below stays under these.  (56 rows of 1M
// keys, budgets 50,000 / 300,000: 835 with lists, 419 in slices.)
static int64_t sel_most_candidates(int64_t n, int rows) {
  const int64_t most = 24000 + (int64_t)((double)n * rows * 2.5e-3);
  return most < 65536 ? most : 65536;
}
struct SelLayout {
  size_t slices, cand, total;
  int32_t n_slices;
  uint32_t cap;
  int samples_v, samples_s;
  bool sliced;
};
static size_t sel_ctl_bytes(const vs_params& p) {
  return align_up((size_t)2 * p.n_q_heads * kSliceRowWords * sizeof(uint32_t), 256);
}
static SelLayout sel_layout(const vs_params& p, bool least) {
  SelLayout l;
  const int64_t n = p.q_start + p.q_len;
  const size_t rows = 2 * (size_t)p.n_q_heads;
  l.samples_v = sel_samples(n, p.vertical_budget, least);
  l.samples_s = sel_samples(n, p.slash_budget, least);
  l.n_slices = (int32_t)ceil_div(n, kSelSlice);
  const int64_t cv = sel_list_len(n, p.vertical_budget, l.samples_v), cs = sel_list_len(n, p.slash_budget, l.samples_s);
  l.cap = (uint32_t)(cv > cs ? cv : cs);
  l.slices = align_up(rows * sizeof(SelHeader), 256);
  l.cand = l.slices + align_up(rows * (size_t)l.n_slices * sizeof(uint2), 256);
  l.sliced = n > kSelRegKeys && (int64_t)l.cap > sel_most_candidates(n, (int)rows);
  l.total = n <= kSelRegKeys ? 256 : (l.sliced ? sel_ctl_bytes(p) : l.cand + align_up(rows * l.cap * sizeof(uint2), 256));
  return l;
}
size_t select_ws_bytes(const vs_params& p, bool least) { return sel_layout(p, least).total; }

static hipError_t launch_slices(SelArgs a, void* ws, hipStream_t st) {
  a.ctl = (uint32_t*)ws;
  // whole steps of the workgroup, enough slices for about 2048 workgroups in all
  const int rows = 2 * a.n_q_heads;
  int64_t want = 2048 / rows;
  want = want < 1 ? 1 : (want > kSliceMax ? kSliceMax : want);
  a.slice_len = ceil_div(ceil_div(a.n, kSliceStep), want) * kSliceStep;
  const dim3 grid((unsigned)ceil_div(a.n, a.slice_len), (unsigned)rows), block(kSelThreads);
  hipLaunchKernelGGL(k_slice_init, dim3((unsigned)rows), dim3(256), 0, st, a);
  for (int pass = 0; pass < 4; ++pass) hipLaunchKernelGGL(k_slice_digit, grid, block, 0, st, a, pass);
  hipLaunchKernelGGL(k_slice_count, grid, block, 0, st, a);
  hipLaunchKernelGGL(k_slice_write, grid, block, 0, st, a);
  return hipGetLastError();
}

// ws: ws_bytes bytes.  With fewer than select_ws_bytes(p, true), which only the static entry point has, every row lists its own
// candidates where the list fits the LDS; longer lists' rows go in slices (56 rows of 1M keys, 20,000 of them to choose: 371 us,
// row by row 989).
hipError_t launch_select(const vs_params& p, const float* vscore, const float* sscore,
                         const int32_t* v_budget_h, const int32_t* s_budget_h,
                         int32_t* v_idx, int32_t* v_cnt, int32_t* s_idx, int32_t* s_cnt, void* ws,
                         size_t ws_bytes, hipStream_t st) {
  SelArgs a = {};
  a.vscore = vscore; a.sscore = sscore; a.n = p.q_start + p.q_len;
  a.n_q_heads = p.n_q_heads;
  a.v_budget = p.vertical_budget; a.s_budget = p.slash_budget;
  a.keep_v = p.keep_first_cols; a.keep_s = p.keep_local_band;
  a.v_budget_h = v_budget_h; a.s_budget_h = s_budget_h;
  a.v_idx = v_idx; a.v_cnt = v_cnt; a.s_idx = s_idx; a.s_cnt = s_cnt;
  SelLayout l = sel_layout(p, false);
  if (ws_bytes < l.total) l = sel_layout(p, true);
  a.n_slices = l.n_slices; a.samples_v = l.samples_v; a.samples_s = l.samples_s;
  const dim3 rows(2u * (unsigned)p.n_q_heads), block(kSelThreads);
  const auto in_registers = [&](auto&& kernel, int kpt) {
    if (a.n > (int64_t)kpt * kSelThreads) return false;
    hipLaunchKernelGGL(kernel, rows, block, 0, st, a);
    return true;
  };
  if (in_registers(k_sel_row<4>, 4) || in_registers(k_sel_row<8>, 8) || in_registers(k_sel_row<12>, 12) || in_registers(k_sel_row<16>, 16) ||
      in_registers(k_sel_row<24>, 24) || in_registers(k_sel_row<32>, 32) || in_registers(k_sel_row<40>, 40) || in_registers(k_sel_row<48>, 48))
    return hipGetLastError();
  static_assert(kSelRegKeys == 48 * kSelThreads, "the rows from here on are long ones");
  if (l.sliced || (ws_bytes < l.total && l.cap > kSelCand)) {
    if (!ws || ws_bytes < sel_ctl_bytes(p)) return hipErrorInvalidValue;
    return launch_slices(a, ws, st);
  }
  static DeviceOnce once;   // the opt-in to more than 64 KiB of LDS
  const hipError_t e = once.run([]() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(&k_sel_row<0>), hipFuncAttributeMaxDynamicSharedMemorySize,
                               kSelCand * (int)sizeof(uint2));
  });
  if (e != hipSuccess) return e;
  if (ws && ws_bytes >= l.total) {
    a.hdr = (SelHeader*)ws;
    a.slices = (uint2*)((char*)ws + l.slices);
    a.cand = (uint2*)((char*)ws + l.cand);
    a.cap = l.cap;
    hipLaunchKernelGGL(k_sel_sample, rows, block, 0, st, a);
    hipLaunchKernelGGL(k_sel_filter, dim3((unsigned)ceil_div(l.n_slices, kSelFilterThreads / 64), rows.x),
                       dim3(kSelFilterThreads), 0, st, a);
  }
  hipLaunchKernelGGL(k_sel_row<0>, rows, block, a.hdr ? 0 : kSelCand * sizeof(uint2), st, a);
  return hipGetLastError();
}

// ---- the selection for callers that cannot allocate ------------------------------------------
// vs_select_static: the headers, tables and candidate lists of the rows live in a file-scope device array instead of a
// caller workspace, where they fit (28 heads at 1M keys take 7 MB); beyond that every row lists its own candidates, or goes
// in slices (launch_select).
// Every device the library runs on holds its own copy of the array at its own address until the process ends; in host
// code the array's name is only a handle, the address comes from hipGetSymbolAddress, once per device, with that
// device current.  A call writes what it reads, so it never sees the contents the call before it left behind; calls
// that overlap in time on one device share the array and race.
static __device__ __align__(256) unsigned char scratch[12 << 20];

hipError_t select_static_scratch(void** ptr_out, size_t* bytes_out) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* ptr_of[kMaxDevices] = {nullptr};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!ptr_of[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!ptr) return hipErrorInvalidSymbol;
    ptr_of[dev] = ptr;
  }
  *ptr_out = ptr_of[dev];
  *bytes_out = sizeof(scratch);
  return hipSuccess;
}

// ---- sparsity refinement ("Sparsity refinement" paragraph and Algorithm 1) --------------------
// recall[h] = mean over the chunk's rows of exp(lse_sparse - lse_full); a row without any
// selected key counts 0.  One workgroup per head, fixed reduction tree.
__global__ __launch_bounds__(256) void k_recall(const float* lse_sparse, const float* lse_full, int64_t rows,
                                                float* recall) {
  const int h = blockIdx.x, tid = threadIdx.x;
  const float* ls = lse_sparse + (int64_t)h * rows;
  const float* lf = lse_full + (int64_t)h * rows;
  float acc = 0.f;
  for (int64_t i = tid; i < rows; i += 256) {
    const float r = __expf(ls[i] - lf[i]);
    acc += (r == r && r <= 3.0e38f) ? r : 0.f;
  }
  __shared__ float part[256];
  part[tid] = acc;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (tid < w) part[tid] += part[tid + w];
    __syncthreads();
  }
  if (tid == 0) recall[h] = rows > 0 ? part[0] / (float)rows : 0.f;
}

// One pass of Algorithm 1 over the heads: a head below the threshold gets dv / ds more lines.
__global__ __launch_bounds__(256) void k_refine(const float* recall, float threshold, int32_t dv, int32_t ds,
                                                int32_t v_max, int32_t s_max, int n_heads,
                                                int32_t* v_budget, int32_t* s_budget, int32_t* changed) {
  __shared__ int cnt;
  if (threadIdx.x == 0) cnt = 0;
  __syncthreads();
  for (int h = threadIdx.x; h < n_heads; h += 256) {
    if (recall[h] < threshold) {
      int nv = v_budget[h] + dv, ns = s_budget[h] + ds;
      nv = nv > v_max ? v_max : nv;
      ns = ns > s_max ? s_max : ns;
      if (nv != v_budget[h] || ns != s_budget[h]) atomicAdd(&cnt, 1);
      v_budget[h] = nv;
      s_budget[h] = ns;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0 && changed) *changed = cnt;
}

hipError_t launch_recall(const vs_params& p, const float* lse_sparse, const float* lse_full, float* recall,
                         hipStream_t st) {
  hipLaunchKernelGGL(k_recall, dim3(p.n_q_heads), dim3(256), 0, st, lse_sparse, lse_full, (int64_t)p.q_len, recall);
  return hipGetLastError();
}

hipError_t launch_refine(const vs_params& p, const float* recall, float threshold, int32_t dv, int32_t ds,
                         int32_t* v_budget, int32_t* s_budget, int32_t* changed, hipStream_t st) {
  hipLaunchKernelGGL(k_refine, dim3(1), dim3(256), 0, st, recall, threshold, dv, ds, p.vertical_budget,
                     p.slash_budget, p.n_q_heads, v_budget, s_budget, changed);
  return hipGetLastError();
}

}  // namespace vs
