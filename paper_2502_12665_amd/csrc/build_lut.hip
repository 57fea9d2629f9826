// Steps 1-2 of a decode step: WRoPE query rotation (section 4.1: q~ = q R_b) and the
// per-subspace query x centroid tables (section 4.2 last equation, tabulated per subspace).
//
// One workgroup per (sequence, KV head, group of 4 query heads).  The contraction is
// 2*B*Hq*256*D flop in total (8.4 Mflop at the 131072-token configuration), far below
// anything a matrix core would help with, so it runs on the vector ALU in float64: products
// of two float32 values are exact in float64, which makes every table entry the correctly
// rounded inner product.  Three things are written per head (see "Lookup-table format" in
// a2ats.h): the exact 32-bit fixed-point table [c][m], a 16-bit coarse copy of it interleaved
// over the four heads of the group [c][m][4] for the streaming kernel, and the numbers that
// relate them (sum of the per-subspace minima, shift, sum of the per-subspace maxima).
#include <algorithm>

#include "common.hpp"
#include "internal.hpp"
#include "encode_few.hpp"
#include "coarse_score.hpp"
#include "exact_select.hpp"
#include "group_select.hpp"
#include "list_select.hpp"

namespace a2ats {

constexpr int kLutThreads = 1024;
constexpr uint32_t kWriteCommon = 1u << kHeadsPerGroup, kWriteAll = 2 * kWriteCommon - 1;

// LDS of build_lut_body.  Kernels that go on to score against the coarse table have it at LDS address 0 (score_coarse), so they
// have no static LDS and place this behind the table.
template <int DS, bool SHARED>
struct LutLds {
  static constexpr int M = 128 / DS;
  alignas(16) float q[kHeadsPerGroup][128];
  alignas(16) int32_t min[M][kHeadsPerGroup], max[M][kHeadsPerGroup];   // (aligned: the four heads are one read)
  alignas(16) uint32_t maxbits[kHeadsPerGroup];                         // largest |entry| per head, as float bits
  alignas(16) int32_t shift[kHeadsPerGroup];
  float qall[SHARED ? 8 : 1][SHARED ? 128 : 1];
};
template <int DS, bool SHARED>
constexpr size_t lut_lds_bytes() { return (sizeof(LutLds<DS, SHARED>) + 15) / 16 * 16; }

// SHARED: one table per KV head, built from the sum of the rotated queries of its G heads (the
// group's summed score sum_g q~_g . c equals (sum_g q~_g) . c); the rotated queries themselves
// are still written per head.  The table array is then laid out as for n_q_heads == n_kv_heads.
template <int DS, bool QBF16, bool SHARED = false>
__device__ __forceinline__ void build_lut_body(
    int prob, const void* __restrict__ q_in, const float* __restrict__ cos_b,
    const float* __restrict__ sin_b, const float* __restrict__ codebook, float* __restrict__ q_rot,
    int32_t* __restrict__ lut, float* __restrict__ lut_scale, int B, int Hq, int Hkv, int NG, LutLds<DS, SHARED>& S,
    uint32_t write = kWriteAll, unsigned char* coarse_lds = nullptr) {
  // write: what goes to global memory, where other workgroups write the rest: bit r the exact table of head r of the
  // group, its constants and its scale, kWriteCommon the coarse table and the rotated queries; coarse_lds: the group's coarse table is also put there, in the layout the
  // scoring kernels read (one 256-byte row per centroid id).
  constexpr int D = 128, HALF = 64, M = D / DS;
  constexpr int ENTRIES = kCentroids * M;
  constexpr int EPT = ENTRIES / kLutThreads;
  constexpr int MAXQ = 65535 / M;       // a sum of M coarse entries fits 16 bits
  constexpr int LOG2M = M == 16 ? 4 : 5;
  static_assert(M == 16 || M == 32, "M is 16 or 32");

  const int Gq = Hq / Hkv;                 // query heads per KV head
  const int G = SHARED ? 1 : Gq;           // table heads per KV head
  const int Hq_q = Hq;
  if (SHARED) Hq = Hkv;                    // table indexing below is per table head
  const int g4 = prob % NG, kv = (prob / NG) % Hkv, b = prob / (NG * Hkv);
  const int tid = threadIdx.x;
  const LutLayout lay = lut_layout(B, Hq, Hkv, M);

  // The codebook rows of this thread's entries (e = c * M + m, so its entries share m = tid % M)
  // are requested first: their latency overlaps the query rotation.
  const int m = tid % M;
  float cv[EPT][DS];
#pragma unroll
  for (int k = 0; k < EPT; ++k) {
    const int c = (tid + k * kLutThreads) / M;
    const float* cw = codebook + (((size_t)kv * M + m) * kCentroids + c) * DS;
#pragma unroll
    for (int t = 0; t < DS; t += 4) {
      const float4 f = *(const float4*)(cw + t);
      cv[k][t] = f.x; cv[k][t + 1] = f.y; cv[k][t + 2] = f.z; cv[k][t + 3] = f.w;
    }
  }

  // --- q~ = q R_b for the (up to) four heads of this group (SHARED: all G <= 8 heads of the KV head)
  if (tid < (SHARED ? 8 : kHeadsPerGroup) * HALF) {
    const int r = tid / HALF, t = tid % HALF;
    const int hg = SHARED ? r : g4 * kHeadsPerGroup + r;
    float o1 = 0.f, o2 = 0.f;
    if (hg < Gq) {
      const int h = kv * Gq + hg;
      const size_t base = ((size_t)b * Hq_q + h) * D;
      double x1, x2;
      if (QBF16) {
        const uint16_t* qp = (const uint16_t*)q_in;
        x1 = (double)bf16_to_f32(qp[base + t]);
        x2 = (double)bf16_to_f32(qp[base + t + HALF]);
      } else {
        const float* qp = (const float*)q_in;
        x1 = (double)qp[base + t];
        x2 = (double)qp[base + t + HALF];
      }
      const double c = (double)cos_b[t], s = (double)sin_b[t];
      o1 = (float)(x1 * c - x2 * s);
      o2 = (float)(x2 * c + x1 * s);
      if (write & kWriteCommon) {
        q_rot[base + t] = o1;
        q_rot[base + t + HALF] = o2;
      }
    }
    if (SHARED) {
      S.qall[r][t] = o1;
      S.qall[r][t + HALF] = o2;
    } else {
      S.q[r][t] = o1;
      S.q[r][t + HALF] = o2;
    }
  }
  if (SHARED) {
    __syncthreads();
    if (tid < kHeadsPerGroup * D) {
      const int r = tid / D, t = tid % D;
      double sum = 0.0;
      if (r == 0)
        for (int g = 0; g < 8; ++g) sum += (double)S.qall[g][t];   // heads past G hold zeros
      S.q[r][t] = (float)sum;
    }
  }
  if (tid < kHeadsPerGroup) S.maxbits[tid] = 0u;
  if (tid < M * kHeadsPerGroup) {
    S.min[tid / kHeadsPerGroup][tid % kHeadsPerGroup] = INT32_MAX;
    S.max[tid / kHeadsPerGroup][tid % kHeadsPerGroup] = INT32_MIN;
  }
  __syncthreads();

  // --- table entries in float64
  double val[EPT][kHeadsPerGroup];
  double mxd[kHeadsPerGroup] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int k = 0; k < EPT; ++k) {
#pragma unroll
    for (int r = 0; r < kHeadsPerGroup; ++r) {
      double acc = 0.0;
#pragma unroll
      for (int t = 0; t < DS; ++t) acc += (double)S.q[r][m * DS + t] * (double)cv[k][t];
      val[k][r] = acc;
      mxd[r] = fmax(mxd[r], fabs(acc));
    }
  }
  // The thread's maximum as a float rounded up, so that it is never below the true one (rounding is
  // monotone: the same number as the maximum of the rounded entries, with one change of the rounding
  // mode per head instead of one per entry).
  float mx[kHeadsPerGroup];
#pragma unroll
  for (int r = 0; r < kHeadsPerGroup; ++r) mx[r] = __double2float_ru(mxd[r]);

  // --- per-head power-of-two scale: M * max|entry| * 2^e < 2^30.  Non-negative floats order like
  // their bit patterns, so the block maximum is an integer atomic max in LDS (one per wave and head
  // after a reduction over the wave).
#pragma unroll
  for (int r = 0; r < kHeadsPerGroup; ++r) {
    const uint32_t v = wave_max_to_last_lane(__float_as_uint(mx[r]));
    if ((tid & 63) == 63) atomicMax(&S.maxbits[r], v);
  }
  __syncthreads();
  // Every thread derives the four exponents itself (M is a power of two and v a float, so the
  // exponent of v * M is the float's exponent field plus a constant; a subnormal maximum takes the
  // general route): no second barrier, no double-precision library call on the critical path.
  int s_exp[kHeadsPerGroup];
#pragma unroll
  for (int r = 0; r < kHeadsPerGroup; ++r) {
    const uint32_t bits = S.maxbits[r];
    int e = 0;
    if (bits != 0u) {
      int x;   // v * M < 2^x
      if ((bits >> 23) != 0u) {
        x = (int)(bits >> 23) - 126 + LOG2M;
      } else {
        frexp((double)__uint_as_float(bits) * (double)M, &x);
      }
      e = 30 - x;
      e = e > 100 ? 100 : (e < -100 ? -100 : e);
    }
    s_exp[r] = e;
  }
  if (tid < kHeadsPerGroup) {
    const int hg = g4 * kHeadsPerGroup + tid;
    if (hg < G && ((write >> tid) & 1u)) lut_scale[(size_t)b * Hq + kv * G + hg] = (float)ldexp(1.0, -s_exp[tid]);
  }

  // --- exact fixed-point entries; per-(subspace, head) minimum and maximum over the centroids
  // (LDS atomics: the four lanes of a wave that share a subspace collide, nothing else does)
  int32_t iv[EPT][kHeadsPerGroup];
  {
    int32_t mn[4] = {INT32_MAX, INT32_MAX, INT32_MAX, INT32_MAX};
    int32_t mxv[4] = {INT32_MIN, INT32_MIN, INT32_MIN, INT32_MIN};
#pragma unroll
    for (int k = 0; k < EPT; ++k)
#pragma unroll
      for (int r = 0; r < kHeadsPerGroup; ++r) {
        const int32_t v = (int32_t)rint(ldexp(val[k][r], s_exp[r]));
        iv[k][r] = v;
        mn[r] = min(mn[r], v);
        mxv[r] = max(mxv[r], v);
      }
#pragma unroll
    for (int r = 0; r < kHeadsPerGroup; ++r) {
      atomicMin(&S.min[m][r], mn[r]);
      atomicMax(&S.max[m][r], mxv[r]);
    }
  }
  __syncthreads();
  if (tid < kHeadsPerGroup) {
    const int r = tid;
    uint32_t range = 0;
    int32_t base = 0, top = 0;
    for (int mm = 0; mm < M; ++mm) {
      range = max(range, (uint32_t)(S.max[mm][r] - S.min[mm][r]));
      base += S.min[mm][r];
      top += S.max[mm][r];
    }
    int sh = 0;
    while ((range >> sh) > (uint32_t)MAXQ) ++sh;
    S.shift[r] = sh;
    const int hg = g4 * kHeadsPerGroup + r;
    if (hg < G && ((write >> r) & 1u)) {
      int32_t* meta = lut + lay.off_meta + ((size_t)b * Hq + kv * G + hg) * 4;
      meta[0] = base;   // sum over subspaces of the smallest entry
      meta[1] = sh;     // coarse entry = (exact entry - subspace minimum) >> sh
      meta[2] = top;    // sum over subspaces of the largest entry: no score exceeds it
      meta[3] = 0;
    }
  }
  // --- exact tables, one per head as [c][m]: entry e of a thread is word e of the head's table
#pragma unroll
  for (int r = 0; r < kHeadsPerGroup; ++r) {
    const int hg = g4 * kHeadsPerGroup + r;
    if (hg < G && ((write >> r) & 1u)) {
      int32_t* ex = lut + lay.off_exact + ((size_t)b * Hq + kv * G + hg) * ENTRIES;
#pragma unroll
      for (int k = 0; k < EPT; ++k) ex[tid + k * kLutThreads] = iv[k][r];
    }
  }
  __syncthreads();

  // --- coarse table, [half][c][m & 15][4 heads] 16-bit: one 8-byte entry per (c, m)
  {
    uint2* coarse = (uint2*)(lut + lay.off_coarse) + (size_t)prob * ENTRIES;
    const int sh0 = S.shift[0], sh1 = S.shift[1], sh2 = S.shift[2], sh3 = S.shift[3];
    const int mn0 = S.min[m][0], mn1 = S.min[m][1], mn2 = S.min[m][2], mn3 = S.min[m][3];
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
      const int c = (tid + k * kLutThreads) / M;
      const uint32_t q0 = (uint32_t)(iv[k][0] - mn0) >> sh0, q1 = (uint32_t)(iv[k][1] - mn1) >> sh1;
      const uint32_t q2 = (uint32_t)(iv[k][2] - mn2) >> sh2, q3 = (uint32_t)(iv[k][3] - mn3) >> sh3;
      const uint2 entry = make_uint2(q0 | (q1 << 16), q2 | (q3 << 16));
      if (write & kWriteCommon) coarse[(m >> 4) * (kCentroids * 16) + c * 16 + (m & 15)] = entry;
      if (coarse_lds) store_coarse_lds<M>(coarse_lds, c, m, entry);
    }
  }
}

template <int DS, bool QBF16>
__global__ __launch_bounds__(kLutThreads) void build_lut_kernel(
    const void* __restrict__ q_in, const float* __restrict__ cos_b, const float* __restrict__ sin_b,
    const float* __restrict__ codebook, float* __restrict__ q_rot, int32_t* __restrict__ lut,
    float* __restrict__ lut_scale, int B, int Hq, int Hkv, int NG) {
  __shared__ LutLds<DS, false> S;
  build_lut_body<DS, QBF16>(blockIdx.x, q_in, cos_b, sin_b, codebook, q_rot, lut, lut_scale, B, Hq, Hkv, NG, S);
}

template <int DS, bool QBF16>
__global__ __launch_bounds__(kLutThreads) void build_lut_shared_kernel(
    const void* __restrict__ q_in, const float* __restrict__ cos_b, const float* __restrict__ sin_b,
    const float* __restrict__ codebook, float* __restrict__ q_rot, int32_t* __restrict__ lut,
    float* __restrict__ lut_scale, int B, int Hq, int Hkv) {
  __shared__ LutLds<DS, true> S;
  build_lut_body<DS, QBF16, true>(blockIdx.x, q_in, cos_b, sin_b, codebook, q_rot, lut, lut_scale, B, Hq, Hkv, 1, S);
}

// An encoding workgroup of the prologues below: wave w takes the pairs (block * sweeps + s) * 16 + w.
template <int DS>
__device__ __forceinline__ void encode_few_block(int block, int sweeps, const float* __restrict__ keys,
                                                 const float* __restrict__ codebook,
                                                 const float* __restrict__ weights, int mode,
                                                 uint8_t* __restrict__ codes, int B, int Hkv, int n_new, int pos0,
                                                 int64_t ctx_stride) {
  constexpr int M = 128 / DS;
  static_assert(kLutThreads / 64 == kFewPairsPerSweep, "one pair per wave and sweep");
  const long n_pairs = (long)B * Hkv * n_new * M;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (int s = 0; s < sweeps; ++s) {
    const long pair = ((long)block * sweeps + s) * kFewPairsPerSweep + wave;
    if (pair < n_pairs)   // (uniform over the wave)
      encode_few_wave<DS>(keys, codebook, weights, mode, codes, Hkv, M, n_new, pos0, ctx_stride, pair, lane);
  }
}

// Decode prologue in one launch: the first n_lut workgroups build the tables of the current query,
// the others encode the few keys appended this step, one (key, subspace) pair per wave and sweep.
// The two halves touch disjoint data.  The kernel holds one workgroup per CU, so when the two kinds
// together would not fit one round of the CUs the launch is "folded": no encoding workgroups, the
// table workgroups share the pairs out among themselves.
template <int DS, bool QBF16>
__global__ __launch_bounds__(kLutThreads) void decode_prologue_kernel(
    const void* __restrict__ q_in, const float* __restrict__ cos_b, const float* __restrict__ sin_b,
    const float* __restrict__ codebook, float* __restrict__ q_rot, int32_t* __restrict__ lut,
    float* __restrict__ lut_scale, int B, int Hq, int Hkv, int NG, int n_lut,
    const float* __restrict__ keys, const float* __restrict__ weights, int mode,
    uint8_t* __restrict__ codes, int n_new, int pos0, int64_t ctx_stride, int sweeps, int folded) {
  __shared__ LutLds<DS, false> S;
  if ((int)blockIdx.x < n_lut) {
    build_lut_body<DS, QBF16>(blockIdx.x, q_in, cos_b, sin_b, codebook, q_rot, lut, lut_scale, B, Hq, Hkv, NG, S);
    // folded: the table workgroups encode as well, after their stores have been issued (their tail
    // waits for those to drain anyway)
    if (folded)
      encode_few_block<DS>((int)blockIdx.x, sweeps, keys, codebook, weights, mode, codes, B, Hkv, n_new, pos0,
                           ctx_stride);
    return;
  }
  encode_few_block<DS>((int)blockIdx.x - n_lut, sweeps, keys, codebook, weights, mode, codes, B, Hkv, n_new, pos0,
                       ctx_stride);
}

// The decode prologue and the first launch of a2ats_score_topk's streaming route in one: every
// sampling workgroup (P0 per problem) builds its problem's tables itself -- the arithmetic is a few
// microseconds and identical in all of them -- keeps the coarse table in LDS and scores its share of
// the sample against it; part 0 of a problem also writes the tables out for the launches that
// follow.  The remaining workgroups encode the appended keys, or (folded, as in decode_prologue_kernel) these do.  Saves one launch and the copy of the
// table from global memory per step; every result is bit for bit that of the separate calls.
// SHARED: one table per KV head from the summed rotated queries of its heads (build_lut_body<.., true>);
// the thresholds are then per KV head (NG is 1 and the sampling sees Hkv table heads).
template <int DS, bool QBF16, bool SHARED>
__global__ __launch_bounds__(kLutThreads) void decode_select_prologue_kernel(
    const void* __restrict__ q_in, const float* __restrict__ cos_b, const float* __restrict__ sin_b,
    const float* __restrict__ codebook, float* __restrict__ q_rot, int32_t* __restrict__ lut,
    float* __restrict__ lut_scale, int B, int Hq, int Hkv, int NG, int n_sample,
    const float* __restrict__ keys, const float* __restrict__ weights, int mode,
    uint8_t* __restrict__ codes, int n_new, int pos0, int64_t ctx_stride,
    const int32_t* __restrict__ seq_lens, int32_t* __restrict__ thr, int P0, int sample_rows, int ctx_len,
    int top_k, int window, int n_sink, int sweeps, int folded) {
  constexpr int M = 128 / DS;
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  LutLds<DS, SHARED>& S = lds_at<LutLds<DS, SHARED>>(kCoarseLdsBytes + kSampleHistBytes);
  if ((int)blockIdx.x < n_sample) {
    int prob, p;
    xcd_map_sets(blockIdx.x, P0, n_sample / P0, NG, prob, p);
    build_lut_body<DS, QBF16, SHARED>(prob, q_in, cos_b, sin_b, codebook, q_rot, lut, lut_scale, B, Hq, Hkv, NG, S,
                                      p == 0 ? kWriteAll : 0u, dyn_lds);
    __syncthreads();
    sample_threshold_body<M, kLutThreads, true>(prob, p, codes, CodePages{nullptr, 0, 0}, lut, seq_lens,
                                                threshold_in(thr, prob, p, P0, NG, SHARED ? Hkv : Hq, Hkv), B,
                                                SHARED ? Hkv : Hq, Hkv, NG, P0, sample_rows, ctx_len, ctx_stride,
                                                top_k, window, n_sink, dyn_lds, lds_at<uint32_t[2][kHistBins]>(kCoarseLdsBytes));
    if (folded)   // (see decode_prologue_kernel)
      encode_few_block<DS>((int)blockIdx.x, sweeps, keys, codebook, weights, mode, codes, B, Hkv, n_new, pos0, ctx_stride);
    return;
  }
  encode_few_block<DS>((int)blockIdx.x - n_sample, sweeps, keys, codebook, weights, mode, codes, B, Hkv, n_new, pos0,
                       ctx_stride);
}

// A whole a2ats_decode_select for short contexts (group_select.hpp) in one launch: a workgroup builds its
// problem's tables, keeps the coarse one in LDS and selects from it at once.  Against the prologue and the
// selection as two launches this saves a launch and the copy of the table.  Of the `split` workgroups of a problem each
// writes the exact tables of the heads that it selects for (it reads them back).  The appended keys are encoded as in
// decode_prologue_kernel.
template <int DS, bool QBF16, bool SHARED, bool MANY>
__global__ __launch_bounds__(kLutThreads) void decode_select_group_kernel(
    const void* __restrict__ q_in, const float* __restrict__ cos_b, const float* __restrict__ sin_b,
    const float* __restrict__ codebook, float* __restrict__ q_rot, int32_t* __restrict__ lut,
    float* __restrict__ lut_scale, int B, int Hq, int Hkv, int NG, int n_lut, GridMap gm, int split,
    const float* __restrict__ keys, const float* __restrict__ weights, int mode,
    uint8_t* __restrict__ codes, int n_new, int pos0, int64_t ctx_stride, int sweeps, int folded,
    const int32_t* __restrict__ seq_lens, int32_t* __restrict__ topk_idx, int32_t* __restrict__ topk_count,
    float* __restrict__ topk_score, int ctx_len, int top_k, int window, int n_sink) {
  constexpr int M = 128 / DS;
  static_assert(kGroupThreads == kLutThreads, "one workgroup does both");
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  if ((int)blockIdx.x < n_lut) {
    int prob, part, b, kv, g4;
    map_block(blockIdx.x, gm, prob, part);
    split_problem(prob, gm, b, kv, g4);
    const int G = SHARED ? 1 : Hq / Hkv;
    const uint32_t mine = group_part(part, split, min(G, kHeadsPerGroup), min(kHeadsPerGroup, G - g4 * kHeadsPerGroup));
    build_lut_body<DS, QBF16, SHARED>(prob, q_in, cos_b, sin_b, codebook, q_rot, lut, lut_scale, B, Hq, Hkv, NG,
                                      lds_at<LutLds<DS, SHARED>>(kGroupLdsBytes),
                                      part == 0 ? mine | kWriteCommon : mine, dyn_lds);
    group_select_body<M, true, MANY>(b, kv, g4, prob, mine, codes, CodePages{nullptr, 0, 0}, lut, lut_scale, seq_lens, topk_idx,
                                     topk_count, topk_score, B, SHARED ? Hkv : Hq, Hkv, ctx_len, ctx_stride, top_k, window,
                                     n_sink, dyn_lds);
    if (folded)
      encode_few_block<DS>((int)blockIdx.x, sweeps, keys, codebook, weights, mode, codes, B, Hkv, n_new, pos0,
                           ctx_stride);
    return;
  }
  encode_few_block<DS>((int)blockIdx.x - n_lut, sweeps, keys, codebook, weights, mode, codes, B, Hkv, n_new, pos0,
                       ctx_stride);
}

// The same for long contexts of many problems (list_select.hpp).
template <int DS, bool QBF16, bool SHARED>
__global__ __launch_bounds__(kLutThreads) void decode_select_list_kernel(
    const void* __restrict__ q_in, const float* __restrict__ cos_b, const float* __restrict__ sin_b,
    const float* __restrict__ codebook, float* __restrict__ q_rot, int32_t* __restrict__ lut,
    float* __restrict__ lut_scale, int B, int Hq, int Hkv, int NG, int n_lut, GridMap gm,
    const float* __restrict__ keys, const float* __restrict__ weights, int mode,
    uint8_t* __restrict__ codes, int n_new, int pos0, int64_t ctx_stride, int sweeps, int folded,
    const int32_t* __restrict__ seq_lens, int32_t* __restrict__ topk_idx, int32_t* __restrict__ topk_count,
    float* __restrict__ topk_score, uint32_t* __restrict__ stats, int sample_rows, int ctx_len, int top_k, int window,
    int n_sink) {
  constexpr int M = 128 / DS;
  static_assert(kListThreads == kLutThreads, "one workgroup does both");
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  if ((int)blockIdx.x < n_lut) {
    int prob, part, b, kv, g4;
    map_block(blockIdx.x, gm, prob, part);
    split_problem(prob, gm, b, kv, g4);
    build_lut_body<DS, QBF16, SHARED>(prob, q_in, cos_b, sin_b, codebook, q_rot, lut, lut_scale, B, Hq, Hkv, NG,
                                      lds_at<LutLds<DS, SHARED>>(kListLdsBytes), kWriteAll, dyn_lds);
    list_select_body<M, true>(b, kv, g4, prob, codes, CodePages{nullptr, 0, 0}, lut, lut_scale, seq_lens, topk_idx, topk_count,
                              topk_score, stats, sample_rows, B, SHARED ? Hkv : Hq, Hkv, NG, ctx_len, ctx_stride, top_k, window,
                              n_sink, dyn_lds);
    if (folded)
      encode_few_block<DS>((int)blockIdx.x, sweeps, keys, codebook, weights, mode, codes, B, Hkv, n_new, pos0,
                           ctx_stride);
    return;
  }
  encode_few_block<DS>((int)blockIdx.x - n_lut, sweeps, keys, codebook, weights, mode, codes, B, Hkv, n_new, pos0,
                       ctx_stride);
}

// A whole a2ats_decode_select for short contexts by one workgroup per head: it builds the head's exact table, keeps it in
// LDS and selects from it at once (exact_select.hpp).  Per head the tables are a quarter of the work that they are for a
// group, and no coarse scores and no band stand between the table and the selection; so this is the faster way as long as
// every head has a CU.  The table, its coarse copy (the head's 16 bits of every entry), constants, scale and rotated query
// also go to global memory, bit for bit as build_lut_body writes them.
template <int DS, bool QBF16, bool SHARED>
__global__ __launch_bounds__(kLutThreads) void decode_select_head_kernel(
    const void* __restrict__ q_in, const float* __restrict__ cos_b, const float* __restrict__ sin_b,
    const float* __restrict__ codebook, float* __restrict__ q_rot, int32_t* __restrict__ lut,
    float* __restrict__ lut_scale, int B, int Hq, int Hkv, int n_heads, GridMap gm, const float* __restrict__ keys,
    const float* __restrict__ weights, int mode, uint8_t* __restrict__ codes, int n_new, int pos0, int64_t ctx_stride,
    int sweeps, int folded, const int32_t* __restrict__ seq_lens, int32_t* __restrict__ topk_idx,
    int32_t* __restrict__ topk_count, float* __restrict__ topk_score, int ctx_len, int top_k, int window, int n_sink) {
  constexpr int D = 128, HALF = 64, M = D / DS, ENTRIES = kCentroids * M, EPT = ENTRIES / kLutThreads;
  constexpr int MAXQ = 65535 / M, LOG2M = M == 16 ? 4 : 5;
  static_assert(kExactThreads == kLutThreads, "one workgroup does both");
  extern __shared__ __align__(16) unsigned char tbl[];   // kExactLdsBytes
  __shared__ ExactLds L;
  __shared__ float s_q[D];
  __shared__ float s_all[SHARED ? 8 : 1][SHARED ? D : 1];
  __shared__ uint32_t s_maxbits;
  __shared__ int32_t s_min[M], s_max[M], s_const[3];   // sum of minima, shift, sum of maxima
  if ((int)blockIdx.x >= n_heads) {
    encode_few_block<DS>((int)blockIdx.x - n_heads, sweeps, keys, codebook, weights, mode, codes, B, Hkv, n_new, pos0,
                         ctx_stride);
    return;
  }
  int prob, r, b, kv, g4;
  map_block(blockIdx.x, gm, prob, r);   // r: the head of the KV head (SHARED: 0)
  split_problem(prob, gm, b, kv, g4);
  const int Gq = Hq / Hkv, G = SHARED ? 1 : Gq, Ht = SHARED ? Hkv : Hq, tid = threadIdx.x;
  const int bh = b * Ht + kv * G + r;
  const LutLayout lay = lut_layout(B, Ht, Hkv, M);
  const int m = tid % M;
  float cv[EPT][DS];
#pragma unroll
  for (int k = 0; k < EPT; ++k) {
    const int c = (tid + k * kLutThreads) / M;
    const float* cw = codebook + (((size_t)kv * M + m) * kCentroids + c) * DS;
#pragma unroll
    for (int t = 0; t < DS; t += 4) {
      const float4 f = *(const float4*)(cw + t);
      cv[k][t] = f.x; cv[k][t + 1] = f.y; cv[k][t + 2] = f.z; cv[k][t + 3] = f.w;
    }
  }
  if (tid < (SHARED ? 8 : 1) * HALF) {
    const int g = tid / HALF, t = tid % HALF;
    float o1 = 0.f, o2 = 0.f;
    if (!SHARED || g < Gq) {
      const size_t base = ((size_t)b * Hq + kv * Gq + (SHARED ? g : r)) * D;
      double x1, x2;
      if (QBF16) {
        const uint16_t* qp = (const uint16_t*)q_in;
        x1 = (double)bf16_to_f32(qp[base + t]);
        x2 = (double)bf16_to_f32(qp[base + t + HALF]);
      } else {
        const float* qp = (const float*)q_in;
        x1 = (double)qp[base + t];
        x2 = (double)qp[base + t + HALF];
      }
      const double c = (double)cos_b[t], s = (double)sin_b[t];
      o1 = (float)(x1 * c - x2 * s);
      o2 = (float)(x2 * c + x1 * s);
      q_rot[base + t] = o1;
      q_rot[base + t + HALF] = o2;
    }
    if (SHARED) {
      s_all[g][t] = o1;
      s_all[g][t + HALF] = o2;
    } else {
      s_q[t] = o1;
      s_q[t + HALF] = o2;
    }
  }
  if (SHARED) {
    __syncthreads();
    if (tid < D) {
      double sum = 0.0;
      for (int g = 0; g < 8; ++g) sum += (double)s_all[g][tid];   // heads past G hold zeros
      s_q[tid] = (float)sum;
    }
  }
  if (tid == 0) s_maxbits = 0u;
  if (tid < M) {
    s_min[tid] = INT32_MAX;
    s_max[tid] = INT32_MIN;
  }
  __syncthreads();
  // (the steps of build_lut_body, for one head)
  double val[EPT], most = 0.0;
#pragma unroll
  for (int k = 0; k < EPT; ++k) {
    double acc = 0.0;
#pragma unroll
    for (int t = 0; t < DS; ++t) acc += (double)s_q[m * DS + t] * (double)cv[k][t];
    val[k] = acc;
    most = fmax(most, fabs(acc));
  }
  const uint32_t wave_most = wave_max_to_last_lane(__float_as_uint(__double2float_ru(most)));
  if ((tid & 63) == 63) atomicMax(&s_maxbits, wave_most);
  __syncthreads();
  int e = 0;
  {
    const uint32_t bits = s_maxbits;
    if (bits != 0u) {
      int x;   // largest entry * M < 2^x
      if ((bits >> 23) != 0u) x = (int)(bits >> 23) - 126 + LOG2M;
      else frexp((double)__uint_as_float(bits) * (double)M, &x);
      e = 30 - x;
      e = e > 100 ? 100 : (e < -100 ? -100 : e);
    }
  }
  const float scale = (float)ldexp(1.0, -e);
  if (tid == 0) lut_scale[bh] = scale;
  int32_t iv[EPT], mn = INT32_MAX, mx = INT32_MIN;
  int32_t* ex = lut + lay.off_exact + (size_t)bh * ENTRIES;
#pragma unroll
  for (int k = 0; k < EPT; ++k) {
    iv[k] = (int32_t)rint(ldexp(val[k], e));
    mn = min(mn, iv[k]);
    mx = max(mx, iv[k]);
    const int c = (tid + k * kLutThreads) / M;
    *(int32_t*)(tbl + (c << 8) + (m << 2)) = iv[k];
    if (M == 16) *(int32_t*)(tbl + (c << 8) + 64 + (m << 2)) = iv[k];
    ex[tid + k * kLutThreads] = iv[k];
  }
  // the lanes of a wave that share a subspace, then the waves
#pragma unroll
  for (int off = M; off < 64; off <<= 1) {
    mn = min(mn, __shfl_xor(mn, off));
    mx = max(mx, __shfl_xor(mx, off));
  }
  if ((tid & 63) < M) {
    atomicMin(&s_min[m], mn);
    atomicMax(&s_max[m], mx);
  }
  __syncthreads();
  if (tid < 64) {
    int32_t base = tid < M ? s_min[tid & (M - 1)] : 0, top = tid < M ? s_max[tid & (M - 1)] : 0;
    uint32_t range = (uint32_t)(top - base);
#pragma unroll
    for (int off = M / 2; off >= 1; off >>= 1) {
      base += __shfl_xor(base, off);
      top += __shfl_xor(top, off);
      range = max(range, (uint32_t)__shfl_xor((int)range, off));
    }
    if (tid == 0) {
      int sh = 0;
      while ((range >> sh) > (uint32_t)MAXQ) ++sh;
      s_const[0] = base;
      s_const[1] = sh;
      s_const[2] = top;
      *(int4*)(lut + lay.off_meta + (size_t)bh * 4) = make_int4(base, sh, top, 0);
    }
  }
  __syncthreads();
  const int32_t base = s_const[0], sh = s_const[1], top = s_const[2];
  {
    // this head's 16 bits of the coarse entries; the last head of a group also fills the places of those that there are none
    // of
    const int slot = r % kHeadsPerGroup, NG = (G + kHeadsPerGroup - 1) / kHeadsPerGroup;
    const int n_real = min(kHeadsPerGroup, G - (r / kHeadsPerGroup) * kHeadsPerGroup), last = slot == n_real - 1 ? kHeadsPerGroup : slot + 1;
    uint16_t* coarse = (uint16_t*)(lut + lay.off_coarse) +
                       (size_t)((b * Hkv + kv) * NG + r / kHeadsPerGroup) * ENTRIES * kHeadsPerGroup;
    const int32_t least = s_min[m];
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
      const int c = (tid + k * kLutThreads) / M;
      uint16_t* at = coarse + ((m >> 4) * (kCentroids * 16) + c * 16 + (m & 15)) * kHeadsPerGroup;
      at[slot] = (uint16_t)((uint32_t)(iv[k] - least) >> sh);
      for (int i = slot + 1; i < last; ++i) at[i] = 0;
    }
  }
  const SeqRange sr = seq_range(ctx_len, seq_lens, b, window, n_sink, top_k);
  int32_t* oi = topk_idx + (size_t)bh * top_k;
  float* os = topk_score ? topk_score + (size_t)bh * top_k : nullptr;
  if (tid == 0) topk_count[bh] = sr.kk;
  for (int t = sr.kk + tid; t < top_k; t += kLutThreads) {
    oi[t] = -1;
    if (os) os[t] = 0.f;
  }
  if (sr.kk > 0)   // (uniform)
    exact_select_sized<M, true>(seq_codes_of<M>(codes, CodePages{nullptr, 0, 0}, b, kv, Hkv, ctx_stride), nullptr, base, top,
                                scale, sr, oi, os, tbl, L);
  if (folded)   // (see decode_prologue_kernel)
    encode_few_block<DS>((int)blockIdx.x, sweeps, keys, codebook, weights, mode, codes, B, Hkv, n_new, pos0, ctx_stride);
}

// How the append-time encoding shares a launch with n_lut table workgroups: workgroups of its own, or
// (folded) the table workgroups, where both kinds would not fit one round of the CUs.
struct AppendPlan {
  int sweeps, folded;
  unsigned n_enc;
};
// may_wait: pairs for each CU that the table workgroups leave free, from which these take them, where there are more.
static AppendPlan append_plan(long n_pairs, int n_lut, int may_wait = 0) {
  AppendPlan p;
  p.sweeps = encode_few_sweeps(n_pairs);
  const long per_wg = (long)kFewPairsPerSweep * p.sweeps, n_enc = (n_pairs + per_wg - 1) / per_wg;
  p.folded = n_lut > 0 && n_lut + n_enc > 256 && n_pairs > (long)may_wait * (256 - n_lut);
  if (p.folded) p.sweeps = (int)((n_pairs + (long)kFewPairsPerSweep * n_lut - 1) / ((long)kFewPairsPerSweep * n_lut));
  p.n_enc = p.folded ? 0u : (unsigned)n_enc;
  return p;
}

// Whether a selection that does not stream is taken by a workgroup per head: where every head has a CU, beside the workgroups
// that encode; where it has one only without those (folded), the group route is the faster one for few rows and M = 16.
// Steps, us, group or exact route -> a workgroup per head, one sequence of 32 query and 8 KV heads, M = 16, 1600, 4096, 8300,
// 16384 tokens 24.8 -> 23.8, 26.6 -> 24.3, 32.2 -> 26.8, 36.6 -> 31.3, M = 32 30.3 -> 24.4, 34.3 -> 26.9, 38.5 -> 31.1, 49.4
// -> 38.8; 8 sequences (folded) M = 16 24.7 -> 26.4, 28.3 -> 29.2, 38.7 -> 36.3, 48.9 -> 45.9, M = 32 34.0 -> 28.6, 41.3 -> 32.4,
// 49.1 -> 40.9, 63.0 -> 52.9; 9 sequences (two rounds) 25.3 -> 37.2 and 70.6 -> 80.6.  With one head to a group nothing is shared
// that a second round could lose: 64 sequences of 8 KV heads, one selection each, 4096, 8192, 16000 tokens 81.0 -> 80.6, 97.3 ->
// 88.0, 107.8 -> 98.9.
// Several keys to append are more than the heads should take besides (three sweeps or more), while the groups leave room for
// workgroups that do: 8 sequences, M = 32, 1500 tokens (without the attention), 4 keys 25.7 -> 23.3, 8 25.6 -> 27.7; 16, which
// neither leaves room for, 42.9 -> 36.7.
bool takes_head_route(const a2ats_dims& d, int n_new, int window, int n_sink, bool shared) {
  const long ncand = (long)d.ctx_len - window - n_sink, heads = (long)d.batch * (shared ? d.n_kv_heads : d.n_q_heads);
  const bool one_a_group = shared || d.n_q_heads == d.n_kv_heads;
  if (single_codebook(d) || ncand > kKeepRows * kExactThreads || heads > (one_a_group ? 512 : 256)) return false;
  const long pairs = (long)d.batch * d.n_kv_heads * n_new * d.n_sub;
  const AppendPlan ap = append_plan(pairs, (int)heads);
  if (!ap.folded || ncand > 8192) return true;
  if (d.n_sub == 16) return false;
  const int per = shared ? 1 : d.n_q_heads / d.n_kv_heads;
  const long groups = (long)d.batch * d.n_kv_heads * ((per + kHeadsPerGroup - 1) / kHeadsPerGroup);
  return ap.sweeps < 3 || !takes_group_route(d, window, n_sink) || append_plan(pairs, (int)groups).folded;
}

// Heads that select by themselves (SHARED: KV heads) and the append in one launch, where takes_head_route.
hipError_t launch_decode_select_head(const a2ats_dims& d, const float* keys, int n_new, int pos0, const float* codebook,
                                     const float* weights, int mode, uint8_t* codes, const void* q, int q_dtype,
                                     const float* cos_b, const float* sin_b, float* q_rot, int32_t* lut, float* lut_scale,
                                     const int32_t* seq_lens, int top_k, int window, int n_sink, int32_t* topk_idx,
                                     int32_t* topk_count, float* topk_score, bool shared, hipStream_t stream) {
  const int per = shared ? 1 : d.n_q_heads / d.n_kv_heads, problems = d.batch * d.n_kv_heads, n_heads = problems * per;
  const AppendPlan ap = append_plan((long)problems * n_new * d.n_sub, n_heads);
  const dim3 grid(n_heads + ap.n_enc), block(kLutThreads);
  if (grid.x == 0) return hipSuccess;
  static LdsSlot s_lds[8][16];
  hipError_t err;
#define A2ATS_LAUNCH_HEAD(DS, BF, SH, SLOT)                                                                       \
  do {                                                                                                            \
    if ((err = allow_dynamic_lds(decode_select_head_kernel<DS, BF, SH>, (size_t)kExactLdsBytes, s_lds[SLOT])) !=  \
        hipSuccess)                                                                                               \
      return err;                                                                                                 \
    hipLaunchKernelGGL((decode_select_head_kernel<DS, BF, SH>), grid, block, kExactLdsBytes, stream, q, cos_b,    \
                       sin_b, codebook, q_rot, lut, lut_scale, d.batch, d.n_q_heads, d.n_kv_heads, n_heads,       \
                       make_grid_map(per, problems, 1, d.n_kv_heads), keys, weights, mode, codes, n_new, pos0,    \
                       d.ctx_stride, ap.sweeps, ap.folded, seq_lens, topk_idx, topk_count, topk_score, d.ctx_len,         \
                       top_k, window, n_sink);                                                                    \
  } while (0)
#define A2ATS_LAUNCH_HEAD2(DS, BF, SLOT)                   \
  do {                                                     \
    if (shared) A2ATS_LAUNCH_HEAD(DS, BF, true, SLOT + 4); \
    else A2ATS_LAUNCH_HEAD(DS, BF, false, SLOT);           \
  } while (0)
  if (d.sub_dim == 8) {
    if (q_dtype == A2ATS_BF16) A2ATS_LAUNCH_HEAD2(8, true, 0); else A2ATS_LAUNCH_HEAD2(8, false, 1);
  } else {
    if (q_dtype == A2ATS_BF16) A2ATS_LAUNCH_HEAD2(4, true, 2); else A2ATS_LAUNCH_HEAD2(4, false, 3);
  }
#undef A2ATS_LAUNCH_HEAD2
#undef A2ATS_LAUNCH_HEAD
  return hipGetLastError();
}

hipError_t launch_decode_select_group(const a2ats_dims& d, const float* keys, int n_new, int pos0,
                                      const float* codebook, const float* weights, int mode, uint8_t* codes,
                                      const void* q, int q_dtype, const float* cos_b, const float* sin_b, float* q_rot,
                                      int32_t* lut, float* lut_scale, const int32_t* seq_lens, int top_k, int window,
                                      int n_sink, int32_t* topk_idx, int32_t* topk_count, float* topk_score,
                                      bool shared, hipStream_t stream) {
  const int G = d.n_q_heads / d.n_kv_heads;
  const int NG = shared ? 1 : (G + kHeadsPerGroup - 1) / kHeadsPerGroup;
  const int groups = d.batch * d.n_kv_heads * NG;
  const AppendPlan ap = append_plan((long)d.batch * d.n_kv_heads * n_new * d.n_sub, groups);
  const int split = ap.folded ? 1 : group_split(groups, shared ? 1 : std::min(G, kHeadsPerGroup), ap.n_enc);
  const int n_lut = groups * split;
  const dim3 grid(n_lut + ap.n_enc), block(kLutThreads);
  if (grid.x == 0) return hipSuccess;
  static LdsSlot s_lds[12][16];
  hipError_t err;
#define A2ATS_LAUNCH_GRP(DS, BF, SH, MANY, SLOT)                                                                      \
  do {                                                                                                          \
    const size_t lds = kGroupLdsBytes + lut_lds_bytes<DS, SH>(); \
    if ((err = allow_dynamic_lds(decode_select_group_kernel<DS, BF, SH, MANY>, lds, s_lds[SLOT], true)) !=       \
        hipSuccess)                                                                                             \
      return err;                                                                                               \
    hipLaunchKernelGGL((decode_select_group_kernel<DS, BF, SH, MANY>), grid, block, lds, stream, q, cos_b, \
                       sin_b, codebook, q_rot, lut, lut_scale, d.batch, d.n_q_heads, d.n_kv_heads, NG, n_lut,   \
                       make_grid_map(split, groups, NG, d.n_kv_heads), split, keys, weights, mode, codes, n_new, pos0, \
                       d.ctx_stride, ap.sweeps, ap.folded, seq_lens, topk_idx, topk_count, topk_score, d.ctx_len, \
                       top_k, window, n_sink);                                                                  \
  } while (0)
#define A2ATS_LAUNCH_GRP2(DS, BF, MANY, SLOT)                   \
  do {                                                          \
    if (shared) A2ATS_LAUNCH_GRP(DS, BF, true, MANY, SLOT + 6); \
    else A2ATS_LAUNCH_GRP(DS, BF, false, MANY, SLOT);           \
  } while (0)
  const int heads = shared ? 1 : std::min(G, kHeadsPerGroup);
  if (d.sub_dim == 8) {
    if (q_dtype == A2ATS_BF16) A2ATS_LAUNCH_GRP2(8, true, false, 0); else A2ATS_LAUNCH_GRP2(8, false, false, 1);
  } else if (!group_many(d.n_sub, (long)d.ctx_len - window - n_sink, top_k, (heads + split - 1) / split)) {
    if (q_dtype == A2ATS_BF16) A2ATS_LAUNCH_GRP2(4, true, false, 2); else A2ATS_LAUNCH_GRP2(4, false, false, 3);
  } else {
    if (q_dtype == A2ATS_BF16) A2ATS_LAUNCH_GRP2(4, true, true, 4); else A2ATS_LAUNCH_GRP2(4, false, true, 5);
  }
#undef A2ATS_LAUNCH_GRP2
#undef A2ATS_LAUNCH_GRP
  return hipGetLastError();
}

hipError_t launch_decode_select_list(const a2ats_dims& d, const TopkPlan& plan, const float* keys, int n_new, int pos0,
                                     const float* codebook, const float* weights, int mode, uint8_t* codes, const void* q,
                                     int q_dtype, const float* cos_b, const float* sin_b, float* q_rot, int32_t* lut,
                                     float* lut_scale, const int32_t* seq_lens, int top_k, int window, int n_sink,
                                     int32_t* topk_idx, int32_t* topk_count, float* topk_score, uint32_t* stats, bool shared,
                                     hipStream_t stream) {
  const int n_lut = d.batch * d.n_kv_heads * plan.NG;
  const AppendPlan ap = append_plan((long)d.batch * d.n_kv_heads * n_new * d.n_sub, n_lut);
  const dim3 grid(n_lut + ap.n_enc), block(kLutThreads);
  if (grid.x == 0) return hipSuccess;
  static LdsSlot s_lds[8][16];
  hipError_t err;
#define A2ATS_LAUNCH_LIST(DS, BF, SH, SLOT)                                                                    \
  do {                                                                                                         \
    const size_t lds = kListLdsBytes + lut_lds_bytes<DS, SH>(); \
    if ((err = allow_dynamic_lds(decode_select_list_kernel<DS, BF, SH>, lds, s_lds[SLOT], true)) !=        \
        hipSuccess)                                                                                            \
      return err;                                                                                              \
    hipLaunchKernelGGL((decode_select_list_kernel<DS, BF, SH>), grid, block, lds, stream, q, cos_b,  \
                       sin_b, codebook, q_rot, lut, lut_scale, d.batch, d.n_q_heads, d.n_kv_heads, plan.NG, n_lut, \
                       make_grid_map(1, n_lut, plan.NG, d.n_kv_heads), keys, weights, mode, codes, n_new, pos0, \
                       d.ctx_stride, ap.sweeps, ap.folded, seq_lens, topk_idx, topk_count, topk_score, stats,  \
                       plan.list_rows, d.ctx_len, top_k, window, n_sink);                                      \
  } while (0)
#define A2ATS_LAUNCH_LIST2(DS, BF, SLOT)                   \
  do {                                                     \
    if (shared) A2ATS_LAUNCH_LIST(DS, BF, true, SLOT + 4); \
    else A2ATS_LAUNCH_LIST(DS, BF, false, SLOT);           \
  } while (0)
  if (d.sub_dim == 8) {
    if (q_dtype == A2ATS_BF16) A2ATS_LAUNCH_LIST2(8, true, 0); else A2ATS_LAUNCH_LIST2(8, false, 1);
  } else {
    if (q_dtype == A2ATS_BF16) A2ATS_LAUNCH_LIST2(4, true, 2); else A2ATS_LAUNCH_LIST2(4, false, 3);
  }
#undef A2ATS_LAUNCH_LIST2
#undef A2ATS_LAUNCH_LIST
  return hipGetLastError();
}

hipError_t launch_decode_select_prologue(const a2ats_dims& d, const float* keys, int n_new, int pos0,
                                         const float* codebook, const float* weights, int mode, uint8_t* codes,
                                         const void* q, int q_dtype, const float* cos_b, const float* sin_b,
                                         float* q_rot, int32_t* lut, float* lut_scale, const int32_t* seq_lens,
                                         int32_t* thr, int P0, int sample_rows, int top_k, int window, int n_sink,
                                         bool shared, hipStream_t stream) {
  const int G = d.n_q_heads / d.n_kv_heads;
  const int NG = shared ? 1 : (G + kHeadsPerGroup - 1) / kHeadsPerGroup;
  const int n_sample = d.batch * d.n_kv_heads * NG * P0;
  // The sampling takes longer than the encoding of a few keys, so workgroups that encode may wait for one another on the CUs that
  // it leaves free, up to 48 pairs for each (M = 32: 108).  Sampling workgroups do it themselves -> others, one wait: 176 problems
  // of 40000 tokens (35 pairs a CU) 92.5 -> 90.3 us, M = 32 (70) 147.1 -> 143.1, two keys (70, 141) 95.7 -> 97.1 and 151.7 ->
  // 152.7; 160, M = 32, two keys (107) 137.5 -> 133.8, three (160) 142.7 -> 147.4; 200 (57, M = 32 114) 103.4 -> 106.8 and 161.7
  // -> 166.3.
  const AppendPlan ap = append_plan((long)d.batch * d.n_kv_heads * n_new * d.n_sub, n_sample, d.n_sub == 32 ? 108 : 48);
  const dim3 grid(n_sample + ap.n_enc), block(kLutThreads);
  if (grid.x == 0) return hipSuccess;
  static LdsSlot s_lds[8][16];
  hipError_t err;
#define A2ATS_LAUNCH_SEL(DS, BF, SH, SLOT)                                                                   \
  do {                                                                                                       \
    const size_t lds = kCoarseLdsBytes + kSampleHistBytes + lut_lds_bytes<DS, SH>(); \
    if ((err = allow_dynamic_lds(decode_select_prologue_kernel<DS, BF, SH>, lds,         \
                                 s_lds[SLOT], true)) != hipSuccess)                                                \
      return err;                                                                                            \
    hipLaunchKernelGGL((decode_select_prologue_kernel<DS, BF, SH>), grid, block, lds, stream, q, \
                       cos_b, sin_b, codebook, q_rot, lut, lut_scale, d.batch, d.n_q_heads, d.n_kv_heads, NG, \
                       n_sample, keys, weights, mode, codes, n_new, pos0, d.ctx_stride, seq_lens, thr, P0,   \
                       sample_rows, d.ctx_len, top_k, window, n_sink, ap.sweeps, ap.folded);                               \
  } while (0)
#define A2ATS_LAUNCH_SEL2(DS, BF, SLOT)                                    \
  do {                                                                     \
    if (shared) A2ATS_LAUNCH_SEL(DS, BF, true, SLOT + 4);                  \
    else A2ATS_LAUNCH_SEL(DS, BF, false, SLOT);                            \
  } while (0)
  if (d.sub_dim == 8) {
    if (q_dtype == A2ATS_BF16) A2ATS_LAUNCH_SEL2(8, true, 0); else A2ATS_LAUNCH_SEL2(8, false, 1);
  } else {
    if (q_dtype == A2ATS_BF16) A2ATS_LAUNCH_SEL2(4, true, 2); else A2ATS_LAUNCH_SEL2(4, false, 3);
  }
#undef A2ATS_LAUNCH_SEL2
#undef A2ATS_LAUNCH_SEL
  return hipGetLastError();
}

hipError_t launch_build_lut(const a2ats_dims& d, const void* q, int q_dtype, const float* cos_b,
                            const float* sin_b, const float* codebook, float* q_rot, int32_t* lut,
                            float* lut_scale, hipStream_t stream) {
  const int G = d.n_q_heads / d.n_kv_heads;
  const int NG = (G + kHeadsPerGroup - 1) / kHeadsPerGroup;
  const dim3 grid(d.batch * d.n_kv_heads * NG), block(kLutThreads);
  if (grid.x == 0) return hipSuccess;
#define A2ATS_LAUNCH_LUT(DS, BF)                                                                    \
  hipLaunchKernelGGL((build_lut_kernel<DS, BF>), grid, block, 0, stream, q, cos_b, sin_b, codebook, \
                     q_rot, lut, lut_scale, d.batch, d.n_q_heads, d.n_kv_heads, NG)
  if (d.sub_dim == 8) {
    if (q_dtype == A2ATS_BF16) A2ATS_LAUNCH_LUT(8, true); else A2ATS_LAUNCH_LUT(8, false);
  } else {
    if (q_dtype == A2ATS_BF16) A2ATS_LAUNCH_LUT(4, true); else A2ATS_LAUNCH_LUT(4, false);
  }
#undef A2ATS_LAUNCH_LUT
  return hipGetLastError();
}

hipError_t launch_build_lut_shared(const a2ats_dims& d, const void* q, int q_dtype, const float* cos_b,
                                   const float* sin_b, const float* codebook, float* q_rot, int32_t* lut,
                                   float* lut_scale, hipStream_t stream) {
  const dim3 grid(d.batch * d.n_kv_heads), block(kLutThreads);
  if (grid.x == 0) return hipSuccess;
#define A2ATS_LAUNCH_LUTS(DS, BF)                                                                          \
  hipLaunchKernelGGL((build_lut_shared_kernel<DS, BF>), grid, block, 0, stream, q, cos_b, sin_b, codebook, \
                     q_rot, lut, lut_scale, d.batch, d.n_q_heads, d.n_kv_heads)
  if (d.sub_dim == 8) {
    if (q_dtype == A2ATS_BF16) A2ATS_LAUNCH_LUTS(8, true); else A2ATS_LAUNCH_LUTS(8, false);
  } else {
    if (q_dtype == A2ATS_BF16) A2ATS_LAUNCH_LUTS(4, true); else A2ATS_LAUNCH_LUTS(4, false);
  }
#undef A2ATS_LAUNCH_LUTS
  return hipGetLastError();
}

hipError_t launch_decode_prologue(const a2ats_dims& d, const float* keys, int n_new, int pos0,
                                  const float* codebook, const float* weights, int mode, uint8_t* codes,
                                  const void* q, int q_dtype, const float* cos_b, const float* sin_b,
                                  float* q_rot, int32_t* lut, float* lut_scale, hipStream_t stream) {
  const int G = d.n_q_heads / d.n_kv_heads;
  const int NG = (G + kHeadsPerGroup - 1) / kHeadsPerGroup;
  const int n_lut = d.batch * d.n_kv_heads * NG;
  const AppendPlan ap = append_plan((long)d.batch * d.n_kv_heads * n_new * d.n_sub, n_lut);
  const dim3 grid(n_lut + ap.n_enc), block(kLutThreads);
  if (grid.x == 0) return hipSuccess;
#define A2ATS_LAUNCH_PRO(DS, BF)                                                                       \
  hipLaunchKernelGGL((decode_prologue_kernel<DS, BF>), grid, block, 0, stream, q, cos_b, sin_b, codebook, \
                     q_rot, lut, lut_scale, d.batch, d.n_q_heads, d.n_kv_heads, NG, n_lut, keys, weights, \
                     mode, codes, n_new, pos0, d.ctx_stride, ap.sweeps, ap.folded)
  if (d.sub_dim == 8) {
    if (q_dtype == A2ATS_BF16) A2ATS_LAUNCH_PRO(8, true); else A2ATS_LAUNCH_PRO(8, false);
  } else {
    if (q_dtype == A2ATS_BF16) A2ATS_LAUNCH_PRO(4, true); else A2ATS_LAUNCH_PRO(4, false);
  }
#undef A2ATS_LAUNCH_PRO
  return hipGetLastError();
}

}  // namespace a2ats
