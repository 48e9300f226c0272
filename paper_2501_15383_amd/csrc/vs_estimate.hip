// Estimation for the vertical-slash pattern (section 5.2, MInference paragraph: attention
// between the last query tokens and all key tokens; chunked-prefill paragraph: the last 64
// tokens of each chunk).  For the W' <= 64 window rows of every head: causal softmax rows
// over all n_k keys, summed along columns (vscore) and along diagonals pos - j (sscore).
//
// Two sweeps over the K cache (read once for every workgroup's share of the heads of a KV group, up to seven):
//   sweep A  per-row (reference, sum) over a range of keys -> partials -> k_estimate_combine -> lse
//   sweep B  P = exp2(S * scale*log2e - lse2), summed along columns and diagonals; run-to-run identical
// bf16 MFMA (32x32x16) with fp32 accumulation; sweep A uses the K Q^T orientation (a lane owns one query), sweep B the Q K^T
// orientation (a lane owns one key).  With Dual Chunk Attention (template parameter DCA) the rotations of the window rows
// that a workgroup's keys meet lie in LDS side by side, and every lane reads its row in the rotation that the row meets the nearest
// key of the tile in: rows on both sides of a chunk boundary still take one product.  Where the window ends inside the tile, a
// second product has the rows in the rotation of the farthest key, and every pair keeps that of its own side.  (Before, a tile took
// one product per rotation that any of 32 rows needed: 28 heads, 300,001 keys 640 us -> 424, with the window of rows across a
// chunk boundary 1,224 -> 433; 2,558 keys 38 -> 29.)
#include <math.h>

#include "vs_common.h"

namespace vs {

struct EstArgs {
  const __bf16* q;
  // Dual Chunk Attention (template parameter DCA; section 5.1 and "Integrating with DCA" in
  // section 5.2): the window rows rotated for the successive-chunk and the inter-chunk pattern
  // (q is the intra-chunk one; same strides), chunk length and local window in tokens
  const __bf16* q_succ;
  const __bf16* q_inter;
  int64_t dca_chunk, dca_window;
  const __bf16* k;
  int64_t q_stride_tok, q_stride_head, k_stride_tok, k_stride_head;
  float* vscore;
  float* sscore;
  float* lse_lastq;  // optional, natural log
  float* part;       // [Hq][n_ranges][64][2]  (max, sum) in the base-2 scaled domain
  float* lse2;       // [Hq][64] base-2 scaled lse (+inf for rows >= W')
  float* far;        // [Hq][n_ranges][waves][64]  references of sweep A past kEstNear (written and read only where there are any)
  int32_t n_q_heads, n_kv_heads, group;
  int32_t wp;        // W'
  int32_t n_ranges;  // partials per head
  int32_t fold;      // sweep B folds them itself (k_estimate_combine is not launched)
  int64_t q_len, n_k, p0;  // p0: position of window row 0
  float scale_log2;
};

// A wave holds the K rows of 64 keys in registers, as MFMA operands straight from memory, and takes the query heads of the KV
// group one after the other; the window rows of all of them wait in LDS.  Nothing is staged and there is no barrier on the way.
// Bound: issue cycles and, at long contexts, power: both sweeps run at 1.7 to 2.0 GHz.  Per 64 scores there are 16 cycles of MFMA and,
// as measured one by one (cycles of a SIMD, from any number of waves): exp 8.3, a lane swap or a half of it 4.2, an add with a lane
// shift 4.3, fma and add 2 each, MFMA issue 4.  Sweep A has exp, fma and add (vector instructions 71 % of the clocked cycles,
// MFMA 51 %, they overlap), sweep B half a lane swap and one shifted add more (two thirds and 37 %).  1M keys, 28 query / 4 KV heads of
// 128, in kernel traces: sweep A 560 -> 475 us (a running maximum took half an instruction per score, and its state two shares of heads:
// K went by twice, 2.24 GB), sweep B 734 -> 619 (three vector instructions fewer per row, see there), 1.27 -> 1.09 ms with everything.  Without
// the stores of sweep B, its lse loads, new K rows per tile or the lane shifts, one at a time, it would be 2 to 9 % faster.
// The next block's product interleaved with this one's exponentials by hand, two or three waves per SIMD and more
// registers, were 5 to 20 % slower.
constexpr int kEstWaves = 16;    // waves per workgroup at most, and per compute unit: four per SIMD, 128 registers
constexpr int est_waves(bool dca) { return dca ? 12 : kEstWaves; }   // (a block of several rotations needs the registers)
constexpr int kEstLds = 160 << 10;
constexpr int kEstFold = 16;     // ranges per wave that sweep B folds itself
constexpr float kEstNear = 131072.f;   // references of sweep A (base 2) that an eighth in a half-word stands for

struct EstShape {
  int32_t heads;     // query heads per workgroup
  int32_t n_hb;      // workgroups per (key range, KV head)
  int32_t waves;     // per workgroup
  int32_t tiles;     // 64-key tiles per wave
  int32_t n_blocks;  // workgroups along the keys
};

// what a workgroup of either sweep is: its KV head, heads, and the tiles of its waves.  The n_hb workgroups of one (key range,
// KV head) are placed on one XCD (blockIdx b and b + 8).  At long contexts the second does not find the K rows in that XCD's L2 all
// the same (see above: its 32 workgroups have 4 MB of them on their way).
struct EstPlace {
  int g, h0, n_h, blk;
  bool ok;
};
__device__ __forceinline__ EstPlace est_place(const EstArgs& a, const EstShape& z) {
  EstPlace p;
  const int b = blockIdx.x, unit = (b / (8 * z.n_hb)) * 8 + (b & 7), hb = (b >> 3) % z.n_hb;
  p.ok = unit < z.n_blocks * a.n_kv_heads;
  p.blk = unit % z.n_blocks;
  p.g = unit / z.n_blocks;
  p.h0 = p.g * a.group + hb * z.heads;
  p.n_h = a.group - hb * z.heads < z.heads ? a.group - hb * z.heads : z.heads;
  return p;
}
// Dual Chunk Attention: rotation that window row r meets key j0 + x with (0 intra-chunk, 1 successive-chunk inside the window, 2
// inter-chunk), for a tile whose keys (all in one chunk: chunks are multiples of 64) lie in chunk ck.
struct EstDca {
  int32_t row_bound;  // rows at or past it lie in the next chunk (64: none of them)
  int32_t ck_rel;     // chunk of the keys less that of row 0, no less than -2
  int32_t dist0;      // position of row 0 less j0
  int32_t window;
  __device__ __forceinline__ int of(int r, int x) const {
    const int cq = r >= row_bound ? 1 : 0;
    if (ck_rel == cq) return 0;
    return ck_rel == cq - 1 && dist0 + r - x < window ? 1 : 2;
  }
  // the rotations that rows r0 .. r0 + 31 need, as bits (of is monotone in r on either side of row_bound, and in x)
  __device__ __forceinline__ uint32_t need(int r0) const {
    uint32_t m = 0;
    const int rb = row_bound;
    const int lo[2] = {r0, rb > r0 ? rb : r0}, hi[2] = {rb < r0 + 32 ? rb - 1 : r0 + 31, r0 + 31};
#pragma unroll
    for (int k = 0; k < 2; ++k)
      if (lo[k] <= hi[k]) m |= (1u << of(lo[k], 63)) | (1u << of(hi[k], 0));
    return m;
  }
};
__device__ __forceinline__ EstDca est_dca(const EstArgs& a, int64_t j0) {
  EstDca d;
  const int64_t cq = a.p0 / a.dca_chunk, rel = j0 / a.dca_chunk - cq, bound = (cq + 1) * a.dca_chunk - a.p0, d0 = a.p0 - j0;
  d.row_bound = bound < 64 ? (int)bound : 64;
  d.ck_rel = rel < -2 ? -2 : (int)rel;
  d.dist0 = (int)d0;   // (fewer than 2^31 keys)
  d.window = (int)(a.dca_window < (1 << 30) ? a.dca_window : (1 << 30));
  return d;
}
// window rows of n_h heads into LDS: row r of head x at (64 x + r) D, its 16-byte piece c in slot c ^ ((r / R) % DCH)
template <int D>
__device__ __forceinline__ void est_load_q(const EstArgs& a, const __bf16* q, const EstPlace& p, __bf16* qs) {
  constexpr int DCH = D / 8, R = 128 / D;
  for (int x = threadIdx.x; x < p.n_h * 64 * DCH; x += blockDim.x) {
    const int c = x % DCH, r = (x / DCH) & 63, hd = x / (64 * DCH);
    const int rw = r < a.wp ? r : a.wp - 1;
    const __bf16* qp = q + (a.q_len - a.wp + rw) * a.q_stride_tok + (int64_t)(p.h0 + hd) * a.q_stride_head + 8 * c;
    *(u32x4*)&qs[(64 * hd + r) * D + ((c ^ ((r / R) % DCH)) * 8)] = *(const u32x4*)qp;
  }
}
// K rows j0 .. j0 + 63 as MFMA operands: lane (row 32 jb + lane % 32, 8 elements from 16 st + 8 hh)
template <int D>
__device__ __forceinline__ void est_load_k(const EstArgs& a, int g, int64_t j0, int lane, bf16x8 (&kf)[2][D / 16]) {
#pragma unroll
  for (int jb = 0; jb < 2; ++jb) {
    int64_t j = j0 + 32 * jb + (lane & 31);
    if (j > a.n_k - 1) j = a.n_k - 1;
    const __bf16* kp = a.k + (int64_t)g * a.k_stride_head + j * a.k_stride_tok + 8 * (lane >> 5);
#pragma unroll
    for (int st = 0; st < D / 16; ++st) kf[jb][st] = *(const bf16x8*)(kp + 16 * st);
  }
}

// the rotations that the workgroup's tiles meet into LDS, [rotation][head]; returns the elements of one rotation
template <int D, bool DCA>
__device__ __forceinline__ int est_load_all_q(const EstArgs& a, const EstShape& z, const EstPlace& p, int n_tiles, __bf16* qs) {
  const int one = z.heads * 64 * D;
  if constexpr (DCA) {
    __shared__ uint32_t need_s;
    if (threadIdx.x == 0) need_s = 0u;
    __syncthreads();
    for (int x = threadIdx.x; x < z.waves * z.tiles; x += blockDim.x) {
      const int t = p.blk * z.waves * z.tiles + x;
      if (t < n_tiles) {
        const EstDca d = est_dca(a, 64 * (int64_t)t);
        atomicOr(&need_s, d.need(0) | d.need(32));
      }
    }
    __syncthreads();
    const uint32_t need = need_s;
    if (need & 1u) est_load_q<D>(a, a.q, p, qs);
    if (need & 2u) est_load_q<D>(a, a.q_succ, p, qs + one);
    if (need & 4u) est_load_q<D>(a, a.q_inter, p, qs + 2 * one);
  } else {
    est_load_q<D>(a, a.q, p, qs);
  }
  return one;
}

// mul(st, operand) for the MFMA steps of window rows 32 x .. 32 x + 31 of the workgroup's heads
template <int D, typename Mul>
__device__ __forceinline__ void est_product(const __bf16* qs, int x, int lane, Mul&& mul) {
  constexpr int DCH = D / 8, R = 128 / D;
  const __bf16* const qr = qs + (32 * x + (lane & 31)) * D;
  const int sw = (lane >> 5) ^ (((lane & 31) / R) % DCH);
#pragma unroll
  for (int st = 0; st < D / 16; ++st) {
    mul(st, *(const bf16x8*)(qr + ((2 * st) ^ sw) * 8));
    if (st & 1) __builtin_amdgcn_sched_barrier(0);   // two operands at a time: the registers are full of K
  }
}

// Sweep A: (reference, sum) of every window row over the workgroup's keys.  K Q^T: a lane owns a query row (32 half + lane % 32
// of the head) and half of the keys.  A row's reference is the largest score of the wave's first tile (base 2), an eighth of it
// kept as a half-word, and stays until a tile's sum of 32 probabilities goes past 2^8 (first tiles and such tiles take the exact way:
// the largest score first).  So there is no maximum in the steady step, and the state of a head is 64 sums and 64 half-words, small
// enough for seven heads beside their rows in LDS: K goes by once.  An eighth, because a reference rounded to 11 bits is then within
// 2^5 of scores up to 2^17, so that no probability overflows and none that counts is lost.  (The upper half of a float was off by up
// to 2^7 from 2^14 on: sums of infinity or nothing; and past 2^18 so is the eighth.)  A reference past 2^17 is kept whole, in
// memory, and its half-word is a NaN: the sum against it is one too, and so the row takes the exact way in every tile, as a running
// maximum: any score is as good as fp32 makes it.
template <int D, bool DCA>
__global__ __launch_bounds__(64 * est_waves(DCA)) void k_est_sums(const EstArgs a, const EstShape z, const int tiles_b) {
  constexpr int DSTEPS = D / 16;
  extern __shared__ __attribute__((aligned(16))) unsigned char est_lds[];
  __bf16* const qs = (__bf16*)est_lds;
  float* const sums = (float*)(qs + (DCA ? 3 : 1) * z.heads * 64 * D);         // [wave][head][64]
  _Float16* const refs = (_Float16*)(sums + z.waves * z.heads * 64);           // the same, an eighth of each
  const EstPlace p = est_place(a, z);
  if (!p.ok) return;
  const int tid = threadIdx.x, lane = tid & 63, hh = lane >> 5;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_tiles = (int)((a.n_k + 63) >> 6);
  const int one_q = est_load_all_q<D, DCA>(a, z, p, n_tiles, qs);
  float* const my_sum = sums + wv * z.heads * 64;
  _Float16* const my_ref = refs + wv * z.heads * 64;
  auto ref_of = [](_Float16 w) { return 8.f * (float)w; };
  auto far_of = [&](int x, int w) -> float* {   // of wave w: the rows of head x
    return a.far + (((int64_t)(p.h0 + x) * z.n_blocks + p.blk) * z.waves + w) * 64;
  };
  __shared__ uint32_t far_s;   // a reference in memory
  if (tid == 0) far_s = 0u;
  for (int x = 0; x < p.n_h; ++x) {
    my_sum[64 * x + lane] = 0.f;
    my_ref[64 * x + lane] = (_Float16)-INFINITY;
  }
  __syncthreads();
  const int t0 = (p.blk * z.waves + wv) * z.tiles, t1 = t0 + z.tiles < n_tiles ? t0 + z.tiles : n_tiles;
  for (int t = t0; t < t1; ++t) {
    const int64_t j0 = 64 * (int64_t)t;
    bf16x8 kf[2][DSTEPS];
    est_load_k<D>(a, p.g, j0, lane, kf);
    EstDca dca = {};
    if constexpr (DCA) dca = est_dca(a, j0);
    // sweep B adds two parts to the offsets of a wave's first tile, and to those behind the last one: cleared here
    auto clear = [&](int tile) {
      const int64_t o = a.p0 + 63 - 64 * (int64_t)tile - lane;
      if (o >= 0 && o < a.n_k)
        for (int x = 0; x < p.n_h; ++x) a.sscore[(int64_t)(p.h0 + x) * a.n_k + o] = 0.f;
    };
    if (t % tiles_b == 0) clear(t);
    if (t == n_tiles - 1) clear(n_tiles);
    const bool causal = j0 + 63 > a.p0;   // some (row, key) of this tile is acausal
    for (int x = 0; x < p.n_h; ++x) {
      float part[2] = {0.f, 0.f};
#pragma clang loop unroll(disable)
      for (int half = 0; half < 2; ++half) {
        part[0] = part[1];
        f32x16 s[2];
        auto product = [&](int rot, f32x16 (&d)[2]) {
#pragma unroll
          for (int jb = 0; jb < 2; ++jb)
#pragma unroll
            for (int e = 0; e < 16; ++e) d[jb][e] = 0.f;
          est_product<D>(qs + rot * one_q, 2 * x + half, lane, [&](int k, bf16x8 qf) {
            d[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[0][k], qf, d[0], 0, 0, 0);
            d[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[1][k], qf, d[1], 0, 0, 0);
          });
        };
        _Float16* const ref = my_ref + 64 * x + 32 * half + (lane & 31);
        float m = ref_of(*ref);
        if constexpr (DCA) {
          const int row = 32 * half + (lane & 31), near = dca.of(row, 63), far = dca.of(row, 0);
          product(near, s);
          if (__builtin_amdgcn_ballot_w64(near != far)) {
            // keys behind the window: those up to `past` (counted from the lane's first)
            int past = (near != far ? row + dca.dist0 - dca.window : -64) - 4 * hh;
            asm volatile("" : "+v"(past));
#pragma unroll
            for (int jb = 0; jb < 2; ++jb) {
              f32x16 d;
#pragma unroll
              for (int e = 0; e < 16; ++e) d[e] = 0.f;
              est_product<D>(qs + far * one_q, 2 * x + half, lane, [&](int k, bf16x8 qf) {
                d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[jb][k], qf, d, 0, 0, 0);
              });
#pragma unroll
              for (int e = 0; e < 16; ++e)
                if (32 * jb + 8 * (e >> 2) + (e & 3) <= past) s[jb][e] = d[e];
            }
          }
        } else {
          product(0, s);
        }
        if (causal) {
          // element e of jb is key 32 jb + 8 (e/4) + 4 hh + (e%4); it is masked for row r iff j - p0 > r
          int dr = 32 * half + (lane & 31) - (int)(j0 - a.p0) - 4 * hh;
          asm volatile("" : "+v"(dr));   // (32 comparisons here, not 32 masks held through the loop)
#pragma unroll
          for (int jb = 0; jb < 2; ++jb)
#pragma unroll
            for (int e = 0; e < 16; ++e)
              if (32 * jb + 8 * (e >> 2) + (e & 3) > dr) s[jb][e] = -INFINITY;
        }
        auto sum = [&](float m_use) -> float {
          float acc0 = 0.f, acc1 = 0.f;
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            acc0 += __builtin_amdgcn_exp2f(__builtin_fmaf(s[0][e], a.scale_log2, -m_use));
            acc1 += __builtin_amdgcn_exp2f(__builtin_fmaf(s[1][e], a.scale_log2, -m_use));
          }
          return acc0 + acc1;
        };
        bool exact = t == t0;
        if (!exact) {
          part[1] = sum(m);
          exact = __builtin_amdgcn_ballot_w64(!(part[1] <= 256.f)) != 0;   // (a reference of -inf makes inf or NaN)
        }
        if (exact) {
          float mx = fmaxf(s[0][0], s[1][0]);
#pragma unroll
          for (int e = 1; e < 16; ++e) mx = fmaxf(fmaxf(mx, s[0][e]), s[1][e]);
          mx = fmaxf(mx, __shfl_xor(mx, 32));
          // (-inf stays -inf; rows without a key so far take 0 in its place)
          float top = fmaxf(m, mx * a.scale_log2);
          _Float16 w = (_Float16)(0.125f * top);
          float m_new = ref_of(w);
          if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(fabsf(top) <= kEstNear) || m != m) != 0, 0)) {
            int hd = x, row = 32 * half + (lane & 31);
            asm volatile("" : "+s"(hd), "+v"(row));   // (the address is made here, not held through the loop)
            float* const at = far_of(hd, wv) + row;
            if (m != m) m = *at;   // (as the lane itself stored it: both of a row store the same)
            top = fmaxf(m, top);
            if (fabsf(top) > kEstNear && top != -INFINITY) {
              *at = m_new = top;
              w = (_Float16)NAN;
              far_s = 1u;
            }
          }
          const float m_use = m_new == -INFINITY ? 0.f : m_new;
          if (lane < 32) {
            float* const l = my_sum + 64 * x + 32 * half + lane;
            *l *= __builtin_amdgcn_exp2f(m - m_use);
            *ref = w;
          }
          part[1] = sum(m_use);
        }
      }
      // the key halves of a row added: lanes 0..31 get the rows of the first half, lanes 32..63 those of the second
      const auto w = __builtin_amdgcn_permlane32_swap(__float_as_uint(part[0]), __float_as_uint(part[1]), false, false);
      const uint32_t w0 = w[0], w1 = w[1];
      my_sum[64 * x + lane] += __uint_as_float(w0) + __uint_as_float(w1);
    }
  }
  __syncthreads();
  // the waves folded in a fixed order: one partial per (head, workgroup, row)
  for (int x = tid; x < 64 * p.n_h; x += blockDim.x) {
    float M = -INFINITY, L = 0.f;
    if (__builtin_expect(far_s != 0u, 0)) {
      auto ref_at = [&](int w) {
        const float m = ref_of(refs[w * z.heads * 64 + x]);
        return m != m ? far_of(x >> 6, w)[x & 63] : m;
      };
#pragma clang loop unroll(disable)
      for (int w = 0; w < z.waves; ++w) M = fmaxf(M, ref_at(w));
      const float Mu = (M == -INFINITY) ? 0.f : M;
#pragma clang loop unroll(disable)
      for (int w = 0; w < z.waves; ++w) L += sums[w * z.heads * 64 + x] * __builtin_amdgcn_exp2f(ref_at(w) - Mu);
    } else {
      for (int w = 0; w < z.waves; ++w) M = fmaxf(M, ref_of(refs[w * z.heads * 64 + x]));
      const float Mu = (M == -INFINITY) ? 0.f : M;
      for (int w = 0; w < z.waves; ++w) L += sums[w * z.heads * 64 + x] * __builtin_amdgcn_exp2f(ref_of(refs[w * z.heads * 64 + x]) - Mu);
    }
    float* const pp = a.part + (((int64_t)(p.h0 + (x >> 6)) * a.n_ranges + p.blk) * 64 + (x & 63)) * 2;
    pp[0] = M;
    pp[1] = L;
  }
}

// (M, L) <- the partial (m, l) added
__device__ __forceinline__ void est_fold(float& M, float& L, float m, float l) {
  const float Mn = fmaxf(M, m);
  const float Mu = (Mn == -INFINITY) ? 0.f : Mn;
  L = L * __builtin_amdgcn_exp2f(M - Mu) + l * __builtin_amdgcn_exp2f(m - Mu);
  M = Mn;
}
// lse2 of row r of head h from its folded partials (rows >= W' get +inf: their P is 0), and the caller's lse
__device__ __forceinline__ void est_store_lse(const EstArgs& a, int h, int r, float M, float L, bool caller) {
  const float l2 = M + __builtin_amdgcn_logf(L);
  a.lse2[(int64_t)h * 64 + r] = r < a.wp ? l2 : INFINITY;
  if (caller && a.lse_lastq && r < a.wp) a.lse_lastq[(int64_t)h * a.wp + r] = l2 * kLn2;
}
// The partials of a workgroup's heads folded by itself: waves / heads waves per head (two or more, see launch_est), every one a share
// of the ranges, and the shares in order: the same numbers in every workgroup of the head, which all store them (scratch: 512 bytes
// per wave; ends with the stores done and all waves past them).  A launch less, 4 to 5 us with its gap, for a trip to memory beside
// that of the window rows.
__device__ __forceinline__ void est_fold_ranges(const EstArgs& a, const EstPlace& p, int waves, float2* scratch) {
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int shares = waves / p.n_h, per = (a.n_ranges + shares - 1) / shares;
  if (wv < p.n_h * shares) {
    const int hd = wv / shares, sh = wv - hd * shares, r0 = sh * per, r1 = r0 + per < a.n_ranges ? r0 + per : a.n_ranges;
    const float2* const pp = (const float2*)a.part + (int64_t)(p.h0 + hd) * a.n_ranges * 64 + lane;
    float M = -INFINITY, L = 0.f;
    constexpr int U = 8;
#pragma clang loop unroll(disable)
    for (int r = r0; r < r1; r += U) {
      float2 v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = pp[64 * (r + u < r1 ? r + u : r1 - 1)];
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (r + u < r1) est_fold(M, L, v[u].x, v[u].y);
    }
    scratch[64 * wv + lane] = make_float2(M, L);
  }
  __syncthreads();
  if (wv < p.n_h) {
    float M = -INFINITY, L = 0.f;
    for (int sh = 0; sh < shares; ++sh) {
      const float2 v = scratch[64 * (wv * shares + sh) + lane];
      est_fold(M, L, v.x, v.y);
    }
    est_store_lse(a, p.h0 + wv, lane, M, L, p.blk == 0);
  }
  __threadfence_block();
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
}
typedef __attribute__((address_space(3))) float lds_float;
// lane 63's four floats to LDS byte address `at` + 16 * slot (all lanes are active before and after)
__device__ __forceinline__ void est_store_last(uint32_t at, f32x4 v, const int slot) {
  asm volatile("s_mov_b64 exec, %2\n\tds_write_b128 %0, %1 offset:%3\n\ts_mov_b64 exec, -1"
               :: "v"(at), "v"(v), "s"(1ull << 63), "n"(16 * slot));
}
// Sweep B: P = exp2(S scale_log2 - lse2), summed along columns and diagonals.  Q K^T, and the two blocks of 32 keys swapped
// by half-waves: a register then is one window row, its 64 lanes the tile's 64 keys.  A column sum is a plain sum over the
// registers.  A diagonal moves on by one lane from row to row, so its sum is an add with a lane rotation per row:
//   acc <- shift(acc, 1) + P[q],   q = 0 .. 63
// after which lane f holds the offset p0 + 63 - (j0 + f), all in one register.  What leaves lane 63 on the way is complete as far as
// this tile goes and belongs to the next tile's offsets: lane 63 stores it, row by row, into LDS, where it waits for the next
// tile of the wave.  (A lane rotation with two sums, of the lanes up to q and of those past it, took three more vector
// instructions per row; the stores are the LDS's work.)
// Offsets at the seam of two waves get their two parts by atomic adds (cleared by sweep A; x + y is commutative, so scores are
// run-to-run identical).
template <int D, bool DCA>
__global__ __launch_bounds__(64 * est_waves(DCA)) void k_est_scores(const EstArgs a, const EstShape z) {
  constexpr int DSTEPS = D / 16;
  extern __shared__ __attribute__((aligned(16))) unsigned char est_lds[];
  __bf16* const qs = (__bf16*)est_lds;
  const EstPlace p = est_place(a, z);
  if (!p.ok) return;
  const int tid = threadIdx.x, lane = tid & 63, hh = lane >> 5;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  float* const carry = (float*)(qs + (DCA ? 3 : 1) * z.heads * 64 * D) + wv * z.heads * 64;   // [wave][head][64]
  const int n_tiles = (int)((a.n_k + 63) >> 6);
  const int one_q = est_load_all_q<D, DCA>(a, z, p, n_tiles, qs);
  const float* lse2 = a.lse2;
  if (a.fold) {
    est_fold_ranges(a, p, z.waves, (float2*)(qs + (DCA ? 3 : 1) * z.heads * 64 * D));   // (where the carries go later)
    asm volatile("" : "+s"(lse2));   // (read through the scalar cache from here on, and not before)
  }
  __syncthreads();
  const int t0 = (p.blk * z.waves + wv) * z.tiles, t1 = t0 + z.tiles < n_tiles ? t0 + z.tiles : n_tiles;
  float c = a.scale_log2;
  asm("" : "+v"(c));   // (one scalar operand per instruction, and that is the row's lse2)
  auto shift = [](float v) -> float {   // lane f takes lane f - 1's value, lane 0 a zero
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x138, 0xF, 0xF, true));
  };
  for (int t = t0; t < t1; ++t) {
    const int64_t j0 = 64 * (int64_t)t;
    bf16x8 kf[2][DSTEPS];
    est_load_k<D>(a, p.g, j0, lane, kf);
    EstDca dca = {};
    if constexpr (DCA) dca = est_dca(a, j0);
    const int64_t o = a.p0 + 63 - j0 - lane;
    const bool causal = j0 + 63 > a.p0;
    for (int x = 0; x < p.n_h; ++x) {
      const int h = __builtin_amdgcn_readfirstlane(p.h0 + x);
      float col[2] = {0.f, 0.f}, diag = 0.f;
      // (volatile: the stores of lane 63 below are not the compiler's)
      const float before = t == t0 ? 0.f : *(volatile float*)(carry + 64 * x + lane);
#pragma clang loop unroll(disable)
      for (int half = 0; half < 2; ++half) {
        // lse2 of the rows (the scalar cache: they are the same in every lane), on their way during the product; with Dual Chunk
        // Attention the scalar registers are full and they are read behind it
        f32x16 lse_lo, lse_hi;
        auto load_lse = [&]() {
          typedef const __attribute__((address_space(4))) f32x16* const_ptr;
          const const_ptr lse = (const_ptr)(lse2 + (int64_t)h * 64 + 32 * half);
          lse_lo = lse[0];
          lse_hi = lse[1];
        };
        if constexpr (!DCA) load_lse();
        f32x16 s[2];
        auto product = [&](int rot, f32x16 (&d)[2]) {
#pragma unroll
          for (int jb = 0; jb < 2; ++jb)
#pragma unroll
            for (int e = 0; e < 16; ++e) d[jb][e] = 0.f;
          est_product<D>(qs + rot * one_q, 2 * x + half, lane, [&](int k, bf16x8 qf) {
            d[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf, kf[0][k], d[0], 0, 0, 0);
            d[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf, kf[1][k], d[1], 0, 0, 0);
          });
        };
        if constexpr (DCA) {
          const int row = 32 * half + (lane & 31), near = dca.of(row, 63), far = dca.of(row, 0);
          product(near, s);
          if (__builtin_amdgcn_ballot_w64(near != far)) {
            // rows for which a key lies behind the window: from `first` on (counted from the lane's first row; of the second 32 keys
            // 32 later) and below `end`.  (Rows that meet the whole tile behind it are `far` in both products.)
            const int rb = dca.row_bound, lo = dca.ck_rel == 0 ? rb : 0, own = 32 * half + 4 * hh;
            int first = (lane & 31) + dca.window - dca.dist0 - own, end = (dca.ck_rel == 0 ? 64 : rb) - own;
            asm volatile("" : "+v"(first), "+v"(end));
#pragma unroll
            for (int jb = 0; jb < 2; ++jb) {
              const int from = first + 32 * jb > lo - own ? first + 32 * jb : lo - own;
              f32x16 d;
#pragma unroll
              for (int e = 0; e < 16; ++e) d[e] = 0.f;
              est_product<D>(qs + far * one_q, 2 * x + half, lane, [&](int k, bf16x8 qf) {
                d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf, kf[jb][k], d, 0, 0, 0);
              });
#pragma unroll
              for (int e = 0; e < 16; ++e)
                if (8 * (e >> 2) + (e & 3) >= from && 8 * (e >> 2) + (e & 3) < end) s[jb][e] = d[e];
            }
          }
        } else {
          product(0, s);
        }
        if (causal) {
          // element e is row 32 half + 8 (e/4) + 4 hh + (e%4), the lane key 32 jb + lane % 32; masked iff j - p0 > row
          const int dj = (int)(j0 - a.p0) + (lane & 31) - 4 * hh - 32 * half;
#pragma unroll
          for (int jb = 0; jb < 2; ++jb)
#pragma unroll
            for (int e = 0; e < 16; ++e)
              if (dj + 32 * jb > 8 * (e >> 2) + (e & 3)) s[jb][e] = -INFINITY;
        }
        if constexpr (DCA) load_lse();
        const uint32_t carry_at = (uint32_t)(uintptr_t)(lds_float*)(carry + 64 * x + 32 * (1 - half));
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {
          // rows 8 e4 + 0..3 of the half in s[0], rows 8 e4 + 4..7 in s[1] after the swap
#pragma unroll
          for (int e = 4 * e4; e < 4 * e4 + 4; ++e) {
            const float x0 = s[0][e], x1 = s[1][e];
            const auto w = __builtin_amdgcn_permlane32_swap(__float_as_uint(x0), __float_as_uint(x1), false, false);
            const uint32_t w0 = w[0], w1 = w[1];
            s[0][e] = __uint_as_float(w0);
            s[1][e] = __uint_as_float(w1);
          }
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            f32x4 out;   // lane 63 before rows q .. q + 3: offsets p0 + q - 1 - (j0 + 63) and on, the next tile's lanes 63 - q and down
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int q = 8 * e4 + 4 * k + e;
              const float pr = __builtin_amdgcn_exp2f(__builtin_fmaf(s[k][4 * e4 + e], c, -(q < 16 ? lse_lo : lse_hi)[q & 15]));
              col[q & 1] += pr;
              out[3 - e] = diag;
              diag = shift(diag) + pr;
            }
            est_store_last(carry_at, out, 7 - 2 * e4 - k);
          }
        }
      }
      float* const so = a.sscore + (int64_t)h * a.n_k + o;
      const bool in = o >= 0 && o < a.n_k;
      if (t == t0) {
        if (in) atomicAdd(so, diag);
      } else {
        if (in) *so = diag + before;
      }
      if (j0 + lane < a.n_k) a.vscore[(int64_t)h * a.n_k + j0 + lane] = col[0] + col[1];
    }
  }
  if (t0 < t1) {
    const int64_t o = a.p0 + 63 - 64 * (int64_t)t1 - lane;
    if (o >= 0 && o < a.n_k)
      for (int x = 0; x < p.n_h; ++x) atomicAdd(&a.sscore[(int64_t)(p.h0 + x) * a.n_k + o], *(volatile float*)(carry + 64 * x + lane));
  }
}

// lse2[h][r] = M + log2(L) over all range partials; rows >= W' get +inf (their P is 0).
// 16 groups of 64 threads each fold every 16th range, then group 0 folds the 16 results: a
// fixed order, so the result is run-to-run identical.
__global__ __launch_bounds__(1024) void k_estimate_combine(const EstArgs a) {
  const int h = blockIdx.x, r = threadIdx.x & 63, grp = threadIdx.x >> 6;
  float M = -INFINITY, L = 0.f;
  for (int rg = grp; rg < a.n_ranges; rg += 16) {
    const float* pp = a.part + (((int64_t)h * a.n_ranges + rg) * 64 + r) * 2;
    est_fold(M, L, pp[0], pp[1]);
  }
  __shared__ float sm[16][64], sl[16][64];
  sm[grp][r] = M;
  sl[grp][r] = L;
  __syncthreads();
  if (grp != 0) return;
  for (int g2 = 1; g2 < 16; ++g2) est_fold(M, L, sm[g2][r], sl[g2][r]);
  est_store_lse(a, h, r, M, L, true);
}

// The cut of a sweep, by the time it should take, in units of one row block of a wave with 16 waves on the compute unit
// (about 2.5 us): a tile costs 2 per head and something for its K rows, a row block is faster with fewer waves around; a
// workgroup costs its start and the window rows that it puts into LDS, a wave per head what it adds to its neighbours' offsets
// (atomic additions), and every share of the heads its K rows once more.  With Dual Chunk Attention the start (up to three
// rotations, patterns) weighs more.  Workgroups of one key range stay on one XCD (est_place), so rounds are those of the XCD that gets
// most (20 heads on one KV head, 45,000 keys: 25 ranges of 10 shares had 40 workgroups on an XCD of 32 compute units, 105 us; 61 now).
// The weights are fitted to all cuts of 189 calls (1 to 64 heads, 2,558 to 300,001 keys): the chosen cuts are within 0.9 % of the
// best ones on average, 0.8 % with Dual Chunk Attention, the worst 10 and 12 % off.  Small calls are made of few rounds of workgroups,
// so the waves per workgroup are whatever fills them.  head_bytes: LDS per head and wave, beside the rows.
// Shares are those that leave fewest heads for the last one (of 32 heads 4 each, not 7, 7, 7, 7 and 4); with Dual Chunk Attention three
// heads only where that leaves no more places empty than two (five heads 131,072 keys 346 us with two, 300 with three; of seven the
// third share would have one).
static EstShape est_shape(const vs_params& p, int most, int head_bytes, bool dca) {
  const int group = p.n_q_heads / p.n_kv_heads, n_cu = 256;
  const int64_t n_tiles = ceil_div(p.q_start + p.q_len, 64), units = n_tiles * p.n_kv_heads;
  const double busy = dca ? 0.2 : 0.1, k_rows = dca ? 1.5 : 4.0, start = dca ? 4.0 : 1.5, fill = 0.2, seam = dca ? 1.5 : 2.0, again = 0.5e-3;
  EstShape best = {};
  double best_cost = -1.0;
  static constexpr int kWaves[] = {16, 14, 12, 10, 9, 8, 7, 6, 5, 4};
  for (int heads = most < group ? most : group; heads >= 1; --heads) {
    const int n_hb = (group + heads - 1) / heads;
    if (heads > 1 && (group + heads - 2) / (heads - 1) == n_hb) continue;
    if (dca && heads == 3 && n_hb * 3 > (group + 1) / 2 * 2) continue;
    for (const int waves : kWaves) {
      const int lds = heads * ((dca ? 3 : 1) * 64 * p.head_dim * 2 + waves * head_bytes);
      if (lds > kEstLds - 64 || waves > est_waves(dca)) continue;
      const int by_lds = kEstLds / lds, by_waves = est_waves(dca) / waves, per_cu = by_lds < by_waves ? by_lds : by_waves;
      for (int want = 1; want <= 3; ++want) {   // rounds
        const int64_t tiles = ceil_div(units * n_hb, (int64_t)waves * per_cu * n_cu * want);
        const int64_t blocks = ceil_div(n_tiles, tiles * waves), wgs = 8 * ceil_div(blocks * p.n_kv_heads, 8) * n_hb;
        const int64_t rounds = ceil_div(wgs, n_cu * per_cu), resident = rounds > 1 ? per_cu : ceil_div(wgs, n_cu);
        const double rate = busy + (1.0 - busy) * (double)(resident * waves) / kEstWaves;
        const double cost = (double)rounds * ((double)tiles * (2.0 * heads + k_rows) * rate + start + fill * heads * kEstWaves / waves +
                                              seam * heads) + again * (double)(n_hb * units);
        if (best_cost < 0 || cost < best_cost) {
          best_cost = cost;
          best.heads = heads; best.n_hb = n_hb; best.waves = waves;
          best.tiles = (int32_t)tiles; best.n_blocks = (int32_t)blocks;
        }
        if (tiles == 1) break;   // (no finer)
      }
    }
  }
  return best;
}
static EstShape est_shape_a(const vs_params& p, bool dca) { return est_shape(p, dca ? 3 : 7, 64 * (sizeof(float) + sizeof(_Float16)), dca); }
static EstShape est_shape_b(const vs_params& p, bool dca) { return est_shape(p, dca ? 3 : 7, 64 * sizeof(float), dca); }

size_t estimate_ws_bytes(const vs_params& p) {
  auto bytes = [&](const EstShape& z) {   // (partial, lse, far references)
    const size_t rows = (size_t)p.n_q_heads * 64;
    return rows * z.n_blocks * 2 * sizeof(float) + rows * sizeof(float) + rows * z.n_blocks * z.waves * sizeof(float);
  };
  const size_t n = bytes(est_shape_a(p, false)), n_dca = bytes(est_shape_a(p, true));   // (the size serves either call)
  return n > n_dca ? n : n_dca;
}

template <int D, bool DCA>
static hipError_t launch_est(const vs_params& p, EstArgs a, void* ws, hipStream_t st) {
  static DeviceOnce once;
  const hipError_t e = once.run([] {   // more than 64 KiB of LDS per workgroup
    const hipError_t r = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_est_sums<D, DCA>), hipFuncAttributeMaxDynamicSharedMemorySize, kEstLds - 64);
    return r != hipSuccess ? r : hipFuncSetAttribute(reinterpret_cast<const void*>(&k_est_scores<D, DCA>), hipFuncAttributeMaxDynamicSharedMemorySize, kEstLds - 64);
  });
  if (e != hipSuccess) return e;
  const EstShape za = est_shape_a(p, DCA), zb = est_shape_b(p, DCA);
  a.n_ranges = za.n_blocks;
  // Sweep B folds up to 16 ranges per wave itself, in two trips to memory: 28 heads, 2,558 keys 23.0 us -> 20.6, 20,000 48.3 -> 46.7; 4 heads of
  // 64, 8,192 keys 20.7 -> 15.6.  With seven heads per workgroup a wave has 30 and more, four trips: as long as the launch.
  // Not where a head has no two waves of its own (never so few ranges, over 20,000 sizes and head shapes).
  const int shares = zb.waves / zb.heads;
  a.fold = shares > 1 && a.n_ranges <= kEstFold * shares;
  a.part = (float*)ws;
  a.lse2 = a.part + (size_t)p.n_q_heads * a.n_ranges * 64 * 2;   // (every part a multiple of 256 bytes)
  a.far = a.lse2 + (size_t)p.n_q_heads * 64;
  auto grid = [&](const EstShape& z) { return dim3((unsigned)(ceil_div((int64_t)z.n_blocks * a.n_kv_heads, 8) * 8 * z.n_hb)); };
  const size_t q_bytes = (DCA ? 3 : 1) * 64 * D * sizeof(__bf16);
  hipLaunchKernelGGL((k_est_sums<D, DCA>), grid(za), dim3(64 * za.waves), za.heads * (q_bytes + (size_t)za.waves * 64 * (sizeof(float) + sizeof(_Float16))), st, a, za, zb.tiles);
  if (!a.fold) hipLaunchKernelGGL(k_estimate_combine, dim3(a.n_q_heads), dim3(1024), 0, st, a);
  const size_t carry = (size_t)zb.heads * 64 * sizeof(float), fold = 64 * sizeof(float2);   // per wave
  hipLaunchKernelGGL((k_est_scores<D, DCA>), grid(zb), dim3(64 * zb.waves), zb.heads * q_bytes + zb.waves * (carry > fold ? carry : fold), st, a, zb);
  return hipGetLastError();
}

hipError_t launch_estimate(const vs_params& p, const void* q, const DcaArgs* dca, const void* k, float* vscore,
                           float* sscore, float* lse_lastq, void* ws, hipStream_t st) {
  EstArgs a;
  a.q = (const __bf16*)q; a.k = (const __bf16*)k;
  a.q_succ = dca ? (const __bf16*)dca->q_succ : nullptr;
  a.q_inter = dca ? (const __bf16*)dca->q_inter : nullptr;
  a.dca_chunk = dca ? dca->chunk : 0;
  a.dca_window = dca ? dca->window : 0;
  a.q_stride_tok = p.q_stride_tok; a.q_stride_head = p.q_stride_head;
  a.k_stride_tok = p.k_stride_tok; a.k_stride_head = p.k_stride_head;
  a.vscore = vscore; a.sscore = sscore; a.lse_lastq = lse_lastq;
  a.n_q_heads = p.n_q_heads; a.n_kv_heads = p.n_kv_heads; a.group = p.n_q_heads / p.n_kv_heads;
  a.wp = (int32_t)(p.last_q < p.q_len ? p.last_q : p.q_len);
  a.q_len = p.q_len; a.n_k = p.q_start + p.q_len; a.p0 = a.n_k - a.wp;
  a.scale_log2 = p.softmax_scale * kLog2e;
  if (p.head_dim == 128) return dca ? launch_est<128, true>(p, a, ws, st) : launch_est<128, false>(p, a, ws, st);
  return dca ? launch_est<64, true>(p, a, ws, st) : launch_est<64, false>(p, a, ws, st);
}

}  // namespace vs
