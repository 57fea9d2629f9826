// Step 3 of a decode step: approximate scores by gather-summing fixed-point table entries
// through the uint8 codes (section 4.2 last equation), and exact per-head top-K (section 4).
//
// Four routes, chosen on the host from the shape:
//
//  group route (at most 16384 candidates, see takes_group_route): one workgroup for the four heads of a group,
//  group_select.hpp.
//
//  list route (up to 65536 candidates of 80 head groups and more, see list_route): one workgroup for the four heads of a
//  group again, list_select.hpp.
//
//  exact route (the other short contexts, more than 2048 winners without a workspace, and the in-kernel fallback):
//  one workgroup per query head runs an MSB-first radix select over the 32-bit score keys by
//  re-streaming its sequence (<= 3 histogram passes), then one ordered pass that emits the
//  winners in ascending position, equal scores going to the lower position.
//
//  fast route (the other long contexts): the code matrix is streamed from HBM once, against a 16-bit
//  coarse copy of the tables, and of the survivors only those near the K-th score are scored exactly.
//    1. sample_threshold_kernel scores a sample of each sequence (about 1/8 of it, taken in
//       128-byte runs spread evenly over the candidates) with the coarse tables and derives, per
//       head, a coarse threshold below the K-th score with a 5-sigma margin (distribution-free
//       for independent rows: it only uses ranks of the sample).
//    2. stream_select_kernel streams all code rows: one 8-byte LDS read per code byte serves the
//       four heads of a group (two heads per 32-bit word, 16 bits each, so one integer add
//       accumulates two heads).  A row whose coarse score reaches the threshold of any of the
//       heads is kept in LDS for a while; then the coarse scores and positions of those that reach a head's
//       threshold go to the head's list of the chunk (4 bytes a row).
//    3. final_select_kernel (one workgroup per head) takes the head's lists (about 1.5 K rows), finds the
//       4-wide bin of the K-th coarse score by a histogram, and with it the winners and a band of
//       2 M + 4 units (coarse and exact scores differ by less than M of them) that alone is scored
//       exactly and ranked; winners are written from a bitmap over the positions.  If the band begins
//       below the threshold, a list is too short or overflowed, or the band holds more than 8192 rows -- the
//       sample misled (about 1e-6 per head for independent rows, more when similar rows come in
//       runs) or the input is degenerate -- the workgroup runs the exact route for its head, so
//       the result is always exact with respect to the 32-bit scores.
#include <hip/hip_ext.h>
#include <math.h>

#include <algorithm>
#include <cmath>
#include "common.hpp"
#include "internal.hpp"
#include "coarse_score.hpp"
#include "exact_select.hpp"
#include "group_select.hpp"
#include "list_select.hpp"

namespace a2ats {

constexpr int kStreamThreads = 512;
constexpr int kStreamWaves = kStreamThreads / 64;
constexpr int kSampleThreads = 512;
constexpr int kFinalCrowd = 8192;    // rows of about the K-th score that the final kernel ranks, where its LDS has room (4000 for the longest contexts)
constexpr int kSampleRows = 1024;    // smallest sample of a problem; a sampling workgroup scores up to 8 of these

// Whether a streaming selection is taken by one workgroup for a head group (list_select.hpp), and the sample that it takes.
// The final kernel's workgroups, one a head, fill a round of the CUs with 64 groups, and the streaming pass has several CUs for a
// group until then; beyond that the heads need further rounds, while the groups fill one.  The longer the context, the more groups
// it takes, and of two rounds the second has to be well filled.  Steps, us, streaming -> list route, 32 query and 8 KV heads, K 3
// %, M = 16: 72 groups 17000, 28000 tokens 63.3 -> 64.6, 80.1 -> 82.2; 80 groups 17000, 31000 70.6 -> 66.9, 90.6 -> 88.1; 96 groups
// 20000, 39000 80.8 -> 74.9, 110.4 -> 110.5; 112 groups 30000, 47000 105.0 -> 100.2, 125.4 -> 127.0; 128 groups 32768, 55000
// 109.9 -> 108.3, 156.5 -> 164.8; 144 groups 40000, 63000 140.1 -> 123.2, 181.0 -> 171.3; 192 groups 65000 216.4 -> 195.8; two
// rounds: 264 groups 32768, 65000 231.1 -> 227.1, 317.2 -> 325.0.  M = 32: 96 groups 24000, 39000 105.8 -> 102.0, 133.1 -> 132.6;
// 144 groups 63000 228.4 -> 228.5; 192 groups 65000 278.9 -> 260.2; two rounds: 288 groups 65000 351.8 -> 381.8.  One selection
// per KV head: 128 groups 32768 76.3 -> 74.3, 160 groups 65000 109.6 -> 102.2.
// Sequences of their own lengths (`ragged`): the streaming pass leaves out what is not there, while one workgroup takes as long as the
// longest, so the line lies lower.  Tables and selection, lengths from a quarter up, streaming -> list route: 80 groups 24000, 28000, 36000
// tokens 41.9 -> 41.7, 42.6 -> 47.1, 47.8 -> 54.5; 96 groups 24000, 28000, 36000 43.0 -> 42.1, 47.8 -> 47.5, 50.3 -> 54.8; 112 groups 24000, 32000, 36000
// 47.8 -> 42.4, 50.7 -> 49.4, 52.4 -> 55.3; 120 groups 32000, 36000 52.6 -> 49.4, 54.3 -> 55.3; 128 groups 36000 56.6 -> 55.6.  M = 32: 80 groups 17000,
// 24000 56.0 -> 56.7, 59.5 -> 63.3; 96 groups 17000, 24000 57.1 -> 56.9, 60.9 -> 63.7; 112 groups 24000, 30000 69.3 -> 64.2, 73.5 -> 74.5; 128 groups
// 36000 86.0 -> 81.3.  Beyond 128 groups the list route gains as with full lengths (144 groups 60000 93.7 -> 78.5, two rounds, 264 groups 159.8 ->
// 152.5).
// Three rounds and more, full lengths: 520 groups 32768 223 -> 173, 768 268 -> 186, 1024 364 -> 248; 768 of 60000 393 -> 282; M = 32 1024 of 24000
// 523 -> 347.
// A list holds kListCap rows: what the sample lets through (see below), five standard deviations more, and 8 % for the
// threshold's rounding to a bin.
static void list_route(const a2ats_dims& d, TopkPlan& p, long ncand, int top_k, bool ragged) {
  const long problems = std::max(1L, (long)d.batch * d.n_kv_heads * p.NG);
  p.list_rows = (int)std::min<long>(std::max<long>(ncand / 8 / 512 * 512, kSampleRows), kSampleMost);
  const double r0 = (double)top_k * p.list_rows / (double)ncand;
  const double xr = 0.5 * (kSigma + std::sqrt(kSigma * kSigma + 4.0 * r0));
  const double rows = (xr * xr + 5.0 * xr) / p.list_rows * (double)ncand * 1.08;
  const long rounds = (problems + 255) / 256, a_round = problems / rounds;
  long few = 36000;
  if (ragged && a_round < 128) {
    if (d.n_sub == 16) few = a_round < 88 ? 24000 : (a_round < 112 ? 28000 : 32000);
    else few = a_round < 96 ? 0 : (a_round < 112 ? 18000 : 26000);
  }
  p.list = a_round >= 80 && ncand <= (a_round > (rounds > 1 ? 192 : 128) ? kListMaxCand : few) && rows <= kListCap;
  if (p.list) p.cap = kListCap;
}

TopkPlan make_topk_plan(const a2ats_dims& d, int top_k, int window, int n_sink, bool ragged) {
  TopkPlan p{};
  const int G = d.n_q_heads / d.n_kv_heads;
  p.NG = (G + kHeadsPerGroup - 1) / kHeadsPerGroup;
  long ncand = (long)d.ctx_len - window - n_sink;
  if (ncand < 0) ncand = 0;
  p.cap = kFinalCrowd;
  // The streaming route: the selection is at most a quarter of at least 16384 candidates, and at most the 4096 that a call may
  // ask for.  Above 2048 the route is called wide and reports no survivor statistics.  (2 sequences of 98301 tokens, 32 heads, K
  // 2949: the step takes 59.5 us; 347 on the exact route, which streams and scores a head's rows four times on one CU.)
  const bool streams = !single_codebook(d) && ncand >= 16384 && top_k >= 1 && top_k <= 4096 && 4L * top_k <= ncand;
  p.fast = streams && top_k <= 2048;
  p.wide = streams && top_k > 2048;
  if (streams) {
    // Sample an eighth of the candidates (at most 65536 rows; in units of 512 rows, at least
    // kSampleRows), shared by at most 8 workgroups of at most 8192 rows each.  The survivors the
    // streaming pass writes and the final kernel reads back shrink with the sample (1.95 K per head
    // at a sixteenth, 1.6 K at an eighth), and sampled rows are cheap while few workgroups carry
    // them: every sampling workgroup pays for a table copy (or, in the fused decode prologue, for
    // the table build) whatever it samples.  So the number of parts is what keeps the sampling
    // launch in one round of the 256 CUs beside the workgroups that encode a one-key append
    // (batch * n_kv_heads * M / 16), with about 2048 rows per part where that leaves a choice; a
    // batch whose problems alone exceed one round takes parts of up to 4096 rows where the sampling is a
    // launch of its own, and only one where it shares one with the tables (sample_in_one_part).  Measured steps (one-key append, 1/16 in 1024-row parts before):
    // batch 4 x 131072 tokens 82.4 -> 81.3 us, batch 16 x 32768 tokens 122.2 -> 117.6 us, batch 32 x
    // 65536 tokens with 7 heads per KV head 390.7 -> 382.5 us.
    long s_tot = ncand / 8 / 512 * 512;
    if (s_tot < kSampleRows) s_tot = kSampleRows;
    if (s_tot > 64 * kSampleRows) s_tot = 64 * kSampleRows;
    const long problems = (long)d.batch * d.n_kv_heads * p.NG;
    const long enc = ((long)d.batch * d.n_kv_heads * d.n_sub + 15) / 16;
    const long fit = problems > 0 ? (256 - enc) / problems : 8;   // parts per problem that fit one round
    long parts;
    if (fit >= 1) parts = std::min<long>(std::min<long>(8, fit), (s_tot + 2047) / 2048);
    else parts = std::min<long>(8, (s_tot + 4095) / 4096);
    if (parts < 1) parts = 1;
    long rows = s_tot / parts / 512 * 512;
    if (rows < 512) rows = 512;
    if (rows > 8 * kSampleRows) rows = 8 * kSampleRows;
    p.P0 = (int)parts;
    s_tot = rows * parts;
    p.sample_rows = (int)(s_tot / p.P0);   // at most 8192: the histogram counts are 16 bits wide
    long chunks = (512 + problems - 1) / problems;
    const long max_chunks = (ncand + 2047) / 2048;
    if (chunks > max_chunks) chunks = max_chunks;
    if (chunks < 1) chunks = 1;
    if (chunks > 64) chunks = 64;
    // Survivors.  The sampling rule (rank r with r - 5 sqrt(r) >= K S / N, plus one per part) lets about
    // r N / S rows per head through -- for small K much more than K -- and a row survives if any of
    // the (up to) four heads wants it.  row_cap is twice that share of a wave's rows plus 16
    // standard deviations of a Poisson count; a head's list of a chunk holds that of its eight waves: survivors that come in
    // runs (neighbouring tokens with similar scores) scatter far more between chunks than independent ones.  The final kernel
    // takes at most 64 chunks.  (The workspace is what segments of a wave, with the code bytes of every row, once took.)
    const double r0 = (double)top_k * (double)s_tot / (double)ncand;
    const double xr = 0.5 * (kSigma + std::sqrt(kSigma * kSigma + 4.0 * r0));
    const double survivors = (xr * xr + 2.0 * p.P0) / (double)s_tot * (double)ncand * 1.25;
    const double keep = std::min(1.0, 4.0 * survivors / (double)ncand);
    auto rows_of = [&](long n) { return ((ncand + n - 1) / n + kStreamThreads - 1) / kStreamThreads * kStreamThreads; };
    auto cap_of = [&](long rows) {
      const long rows_per_wave = rows / kStreamWaves;   // a multiple of 64
      const double mu = rows_per_wave * keep;
      const long cap = (long)(mu * 2.0 + 16.0 * std::sqrt(mu)) + 64;
      return std::min((cap + 31) / 32 * 32, rows_per_wave);
    };
    const size_t entry_bytes = 4 + d.n_sub;   // header + code bytes
    long rpc = rows_of(chunks), cap_rows = cap_of(rpc);
    if (chunks < (ncand + 65535) / 65536) {   // (positions in a chunk are 16 bits)
      // More chunks of fewer rows would be more bytes by their deviations and lengths: the lists get what the chunks that the CUs
      // would have been filled with had, so that a workspace sized for those still serves.
      const long bytes = (ncand + rpc - 1) / rpc * (cap_rows * (long)entry_bytes + 32);
      rpc = rows_of((ncand + 65535) / 65536);
      const long most = (bytes / ((ncand + rpc - 1) / rpc) - 32) / (long)entry_bytes / 32 * 32;
      cap_rows = std::min(cap_of(rpc), std::max(most, 64L));
    }
    p.chunks = (int)((ncand + rpc - 1) / rpc);
    p.rows_per_chunk = (int)rpc;
    p.subs = 1;                               // (one segment per wave)
    p.sub_rows = (int)(rpc / kStreamWaves);
    p.row_cap = (int)cap_rows;                // a multiple of 32
    const size_t heads = (size_t)d.batch * d.n_q_heads;
    const size_t segs = (size_t)problems * p.chunks * kStreamWaves;
    list_route(d, p, ncand, top_k, ragged);
    p.off_thr = 0;
    p.off_route = (p.off_thr + heads * p.P0 * sizeof(int32_t) + 255) / 256 * 256;
    p.off_count = (p.off_route + heads * sizeof(uint32_t) + 255) / 256 * 256;
    p.off_cand = (p.off_count + segs * 8 * sizeof(uint32_t) + 255) / 256 * 256;
    p.bytes = (p.off_cand + segs * (size_t)p.row_cap * entry_bytes + 255) / 256 * 256;
  }
  return p;
}

// The exact route spreads the heads of a group over as many CUs; the group route scores a row once for all of
// them.  So it is taken where the heads need more rounds of the 256 CUs than the groups do, and otherwise for
// short contexts, where what it saves is the launch of the tables.  Steps, exact -> group route, 32 query and 8
// KV heads: 16 sequences (two rounds) M = 16, 4096 and 16384 tokens 48.7 -> 36.1 and 78.2 -> 61.9 us, M = 32 60.1
// -> 49.4 and 104.2 -> 91.4; 4 sequences (one round) M = 16, 4096, 8228, 16384 tokens 31.6 -> 30.0, 35.6 -> 35.2,
// 43.9 -> 46.1, M = 32, 1500, 4096, 16384 tokens 35.1 -> 32.5, 38.9 -> 38.4, 56.2 -> 74.6.  A group of one head saves
// nothing but the launch, so the line does not move with the heads of a group (tables and selection of 16 sequences of 16
// heads, one a group, M = 16, 16384 tokens 35.6 -> 42.1, 24 of 8 34.6 -> 37.5, M = 32, 8228 tokens 29.6 -> 30.9).  In more
// than one round it is lower: 64 of 8 heads, M = 16, 4096, 8228, 16384 tokens 49.4 -> 45.1, 55.0 -> 56.8, 66.5 -> 77.8, M =
// 32, 1500, 4096, 8228 tokens 60.9 -> 59.6, 67.3 -> 69.0, 76.9 -> 84.6.  This is the line of the selection by itself; a step
// with up to 256 heads (one round) mostly goes by head, tables included (takes_head_route).
bool takes_group_route(const a2ats_dims& d, int window, int n_sink) {
  const long ncand = (long)d.ctx_len - window - n_sink;
  if (single_codebook(d) || ncand > kGroupMaxCand) return false;
  const int G = d.n_q_heads / d.n_kv_heads;
  const long groups = (long)d.batch * d.n_kv_heads * ((G + kHeadsPerGroup - 1) / kHeadsPerGroup);
  const long head_rounds = ((long)d.batch * d.n_q_heads + 255) / 256, group_rounds = (groups + 255) / 256;
  if (head_rounds > group_rounds) return true;
  const long line = d.n_sub == 16 ? 8192 : 2048;
  return ncand <= (head_rounds > 1 ? line * 3 / 4 : line);
}

// The P0 sampling workgroups of a problem each estimate a head's threshold from their share of the
// sample; the streaming and final kernels use the mean of the estimates (rounded down), which is
// close to what one rank search over the merged sample would give.  INT32_MIN ("take every row")
// from any of them wins.  Exactness never depends on this value: the final kernel proves its
// result complete against whatever threshold was used, or redoes the head exactly.
// Called by all lanes of a wave for NH consecutive heads starting at `head0` (heads at or past
// `n_valid` get 65536, which no coarse score reaches): lane 8 r + p loads part p of head r, so
// the P0 <= 8 values of all heads arrive with one load latency instead of one after another.
// Split in two so that a caller can put its other loads between the request and the use.
template <int NH>
__device__ __forceinline__ int32_t request_thresholds(const int32_t* __restrict__ thr, size_t head0,
                                                      int n_valid, int P0) {
  static_assert(NH * 8 <= 64, "one lane per (head, part)");
  const int lane = threadIdx.x & 63, r = lane >> 3, p = lane & 7;
  int32_t v = 0;
  if (r < NH && r < n_valid && p < P0) v = thr[(head0 + r) * P0 + p];
  return v;
}
template <int NH>
__device__ __forceinline__ void combine_thresholds(int32_t v, int n_valid, int P0, int32_t (&T)[NH]) {
  int32_t all_rows = v == INT32_MIN ? 1 : 0;
  int32_t sum = all_rows ? 0 : v;   // thresholds are >= 0 and below 2^16
  sum = group8_sum(sum);
  all_rows = group8_or(all_rows);
#pragma unroll
  for (int i = 0; i < NH; ++i) {
    const int32_t s_i = __builtin_amdgcn_readlane(sum, 8 * i), a_i = __builtin_amdgcn_readlane(all_rows, 8 * i);
    T[i] = i >= n_valid ? 65536 : (a_i ? INT32_MIN : s_i / P0);
  }
}

template <int M>
__global__ __launch_bounds__(kExactThreads) void select_exact_kernel(
    const uint8_t* __restrict__ codes, const int32_t* __restrict__ lut,
    const float* __restrict__ lut_scale, const int32_t* __restrict__ seq_lens,
    int32_t* __restrict__ topk_idx, int32_t* __restrict__ topk_count,
    float* __restrict__ topk_score, CodePages pg, int B, int Hq, int Hkv, int ctx_len, int64_t ctx_stride,
    int top_k, int window, int n_sink) {
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  __shared__ ExactLds L;
  const int bh = blockIdx.x, b = bh / Hq, h = bh % Hq;
  const int G = Hq / Hkv, kv = h / G;
  const SeqRange sr = seq_range(ctx_len, seq_lens, b, window, n_sink, top_k);
  int32_t* oi = topk_idx + (size_t)bh * top_k;
  float* os = topk_score ? topk_score + (size_t)bh * top_k : nullptr;
  if (threadIdx.x == 0) topk_count[bh] = sr.kk;
  for (int t = sr.kk + threadIdx.x; t < top_k; t += kExactThreads) {
    oi[t] = -1;
    if (os) os[t] = 0.f;
  }
  if (sr.kk == 0) return;
  const LutLayout lay = lut_layout(B, Hq, Hkv, M);
  const int32_t* meta = lut + lay.off_meta + (size_t)bh * 4;
  exact_select_sized<M, false>(seq_codes_of<M>(codes, pg, b, kv, Hkv, ctx_stride),
                               lut + lay.off_exact + (size_t)bh * (kCentroids * M), meta[0], meta[2], lut_scale[bh], sr, oi, os,
                               dyn_lds, L);
}

// ------------------------------------------------------------------------------------------
// Short contexts: one workgroup per problem
// ------------------------------------------------------------------------------------------
template <int M, bool MANY>
__global__ __launch_bounds__(kGroupThreads) void group_select_kernel(
    const uint8_t* __restrict__ codes, const int32_t* __restrict__ lut, const float* __restrict__ lut_scale,
    const int32_t* __restrict__ seq_lens, int32_t* __restrict__ topk_idx, int32_t* __restrict__ topk_count,
    float* __restrict__ topk_score, GridMap gm, CodePages pg, int B, int Hq, int Hkv, int ctx_len, int64_t ctx_stride,
    int top_k, int window, int n_sink, int split) {
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  int prob, part, b, kv, g4;
  map_block(blockIdx.x, gm, prob, part);
  split_problem(prob, gm, b, kv, g4);
  const int G = Hq / Hkv;
  const uint32_t mine = group_part(part, split, min(G, kHeadsPerGroup), min(kHeadsPerGroup, G - g4 * kHeadsPerGroup));
  group_select_body<M, false, MANY>(b, kv, g4, prob, mine, codes, pg, lut, lut_scale, seq_lens, topk_idx, topk_count, topk_score, B,
                              Hq, Hkv, ctx_len, ctx_stride, top_k, window, n_sink, dyn_lds);
}

// ------------------------------------------------------------------------------------------
// Long contexts of many problems: one workgroup per problem
// ------------------------------------------------------------------------------------------
template <int M>
__global__ __launch_bounds__(kListThreads) void list_select_kernel(
    const uint8_t* __restrict__ codes, const int32_t* __restrict__ lut, const float* __restrict__ lut_scale,
    const int32_t* __restrict__ seq_lens, int32_t* __restrict__ topk_idx, int32_t* __restrict__ topk_count,
    float* __restrict__ topk_score, uint32_t* __restrict__ stats, GridMap gm, CodePages pg, int sample_rows, int B, int Hq,
    int Hkv, int NG, int ctx_len, int64_t ctx_stride, int top_k, int window, int n_sink) {
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  int prob, part, b, kv, g4;
  map_block(blockIdx.x, gm, prob, part);
  split_problem(prob, gm, b, kv, g4);
  list_select_body<M, false>(b, kv, g4, prob, codes, pg, lut, lut_scale, seq_lens, topk_idx, topk_count, topk_score, stats,
                             sample_rows, B, Hq, Hkv, NG, ctx_len, ctx_stride, top_k, window, n_sink, dyn_lds);
}

// ------------------------------------------------------------------------------------------
// Debug: dense exact scores for every token (not on the fast path; used by parity tests)
// ------------------------------------------------------------------------------------------
template <int M>
__global__ __launch_bounds__(kStreamThreads) void score_dense_kernel(
    const uint8_t* __restrict__ codes, const int32_t* __restrict__ lut,
    const float* __restrict__ lut_scale, const int32_t* __restrict__ seq_lens,
    float* __restrict__ scores_out, CodePages pg, int B, int Hq, int Hkv, int ctx_len, int64_t ctx_stride) {
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  unsigned char* tbl = dyn_lds;
  const int bh = blockIdx.y, b = bh / Hq, h = bh % Hq;
  const int G = Hq / Hkv, kv = h / G;
  const LutLayout lay = lut_layout(B, Hq, Hkv, M);
  load_exact_table<M, kStreamThreads>(lut + lay.off_exact + (size_t)bh * (kCentroids * M), tbl);
  ExactSwizzle<M> sw;
  sw.init(threadIdx.x & 63);
  __syncthreads();
  int n = seq_lens ? seq_lens[b] : ctx_len;
  n = n < 0 ? 0 : (n > ctx_len ? ctx_len : n);
  const SeqCodes seq_codes = seq_codes_of<M>(codes, pg, b, kv, Hkv, ctx_stride);
  const float sc = lut_scale[bh];
  for (int j = blockIdx.x * kStreamThreads + threadIdx.x; j < n; j += gridDim.x * kStreamThreads)
    scores_out[(size_t)bh * ctx_stride + j] = (float)score_exact_row<M>(row_ptr<M>(seq_codes, j), tbl, sw) * sc;
}

// ------------------------------------------------------------------------------------------
// Fast route, stage 1: sampled coarse thresholds
// ------------------------------------------------------------------------------------------
template <int M>
__global__ __launch_bounds__(kSampleThreads) void sample_threshold_kernel(
    const uint8_t* __restrict__ codes, const int32_t* __restrict__ lut,
    const int32_t* __restrict__ seq_lens, int32_t* __restrict__ thr, CodePages pg, int B, int Hq, int Hkv,
    int NG, int P0, int sample_rows, int problems, int ctx_len, int64_t ctx_stride, int top_k, int window,
    int n_sink) {
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  int p, prob;
  xcd_map_sets(blockIdx.x, P0, problems, NG, prob, p);
  sample_threshold_body<M, kSampleThreads, false>(prob, p, codes, pg, lut, seq_lens, threshold_in(thr, prob, p, P0, NG, Hq, Hkv),
                                                  B, Hq, Hkv, NG, P0, sample_rows, ctx_len, ctx_stride, top_k, window, n_sink,
                                                  dyn_lds, lds_at<uint32_t[2][kHistBins]>(kCoarseLdsBytes));
}

// ------------------------------------------------------------------------------------------
// Fast route, stage 2: one pass over the code matrix
// ------------------------------------------------------------------------------------------
// RESHARED: the rows are read by more than one problem (the head groups of a KV head, placed next
// to each other on one XCD): ordinary loads, so that the line stays in that L2 for the neighbour;
// otherwise non-temporal loads (each row is read once).
// PAGED: the code rows live in a pool of pages; the page numbers of the workgroup's chunk are
// staged in LDS behind the table (up to kPageSlice of them, else they are read from the page table
// row by row), and rows are read with ordinary loads.
constexpr int kPageSlice = 2048;
// Behind the table: two workgroups of 80 KB fit a CU.  The rows of each wave that any head of the group wants; when they are full,
// and at the end, they go to the lists of the heads that want them.  (Appending to four lists row by row took the pass 1.5 to 2 us
// longer; writing these rows to memory and having every head pick its own from there took the final kernel 2.5 to 4.5.)
// 4 sequences of 131072 tokens, K 2048, against entries with the rows' codes: 7.9 -> 1.6 MB written, 19.3 -> 18.3 us.
template <bool PAGED>
struct StreamLds {
  static constexpr int kCap = PAGED ? 100 : 200;
  uint32_t s01[kStreamWaves][kCap], s23[kStreamWaves][kCap];   // coarse scores, two heads a word
  uint16_t pos[kStreamWaves][kCap];                            // in the chunk
  uint32_t n_list[kHeadsPerGroup];
  int32_t page[PAGED ? kPageSlice : 1];
};
static_assert(sizeof(StreamLds<false>) <= 16384 && sizeof(StreamLds<true>) <= 16384, "");

template <int M, bool RESHARED, bool PAGED>
__device__ __forceinline__ void stream_select_body(
    const uint8_t* __restrict__ codes, const int32_t* __restrict__ lut,
    const int32_t* __restrict__ seq_lens, const int32_t* __restrict__ thr,
    uint32_t* __restrict__ counts, uint32_t* __restrict__ lists, GridMap gm, CodePages pg, int B, int Hq, int Hkv, int G,
    int NG, int P0, int n_chunks, int rows_per_chunk, int list_cap, int ctx_len,
    int64_t ctx_stride, int top_k, int window, int n_sink) {
  constexpr int NT = kStreamThreads;
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  unsigned char* tbl = dyn_lds;

  int chunk, prob, b, kv, g4;
  map_block(blockIdx.x, gm, prob, chunk);
  split_problem(prob, gm, b, kv, g4);
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const SeqRange sr = seq_range(ctx_len, seq_lens, b, window, n_sink, top_k);
  const long begin = (long)sr.sink_end + (long)chunk * rows_per_chunk;
  const int end = (int)min((long)sr.win_start, begin + rows_per_chunk);
  const int rows_per_wave = rows_per_chunk / kStreamWaves;
  const long wbegin = begin + (long)wv * rows_per_wave;
  const int wend = (int)min((long)end, wbegin + rows_per_wave);

  // Every (problem, chunk) has four lists of list_cap entries and their lengths in memory; an entry is a coarse score in the
  // upper half and the position in the chunk in the lower.
  uint32_t* my_count = counts + ((size_t)prob * n_chunks + chunk) * kHeadsPerGroup;
  uint32_t* my_list = lists + ((size_t)prob * n_chunks + chunk) * kHeadsPerGroup * (size_t)list_cap;
  StreamLds<PAGED>& L = lds_at<StreamLds<PAGED>>(kCoarseLdsBytes);
  constexpr uint32_t CAP = StreamLds<PAGED>::kCap;
  // thresholds of the group's heads: requested here, combined after the table copy has been issued
  const int32_t thr_lane = request_thresholds<4>(thr, (size_t)b * Hq + kv * G + g4 * kHeadsPerGroup,
                                                G - g4 * kHeadsPerGroup, P0);
  int32_t T[4];   // padded heads never want a row
  // The scoring loop addresses the table by absolute LDS address (it must start at 0, which holds
  // because this kernel has no static LDS).  Should a toolchain ever place it elsewhere, publish
  // overflowing lists instead: the final kernel then takes the exact route.
  const bool misplaced = (uint32_t)(uintptr_t)tbl != 0u;
  if (begin >= sr.win_start || misplaced) {   // nothing to score in this chunk: empty lists
    if (tid < kHeadsPerGroup) my_count[tid] = misplaced ? 0xffffffffu : 0u;
    return;
  }

  LaneSwizzle<M> sw;
  sw.init(lane);
  // Appends the rows of a wave (one a lane, where `in`) to the lists of the heads that want them.
  auto to_lists = [&](uint32_t w01, uint32_t w23, uint32_t pos, bool in) {
    uint64_t h[4];
    h[0] = __builtin_amdgcn_ballot_w64(in && (int32_t)(w01 & 0xffffu) >= T[0]);
    h[1] = __builtin_amdgcn_ballot_w64(in && (int32_t)(w01 >> 16) >= T[1]);
    h[2] = __builtin_amdgcn_ballot_w64(in && (int32_t)(w23 & 0xffffu) >= T[2]);
    h[3] = __builtin_amdgcn_ballot_w64(in && (int32_t)(w23 >> 16) >= T[3]);
    uint32_t at = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) at = write_lane((uint32_t)__popcll(h[r]), r, at);
    if (lane < 4) at = atomicAdd(&L.n_list[lane], at);
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (__builtin_amdgcn_inverse_ballot_w64(h[r])) {
        const uint32_t slot = (uint32_t)__builtin_amdgcn_mbcnt_hi(
            (uint32_t)(h[r] >> 32),
            __builtin_amdgcn_mbcnt_lo((uint32_t)h[r], (uint32_t)__builtin_amdgcn_readlane((int)at, r)));
        const uint32_t a = r < 2 ? w01 : w23;
        if (slot < (uint32_t)list_cap)   // (rows past the capacity are dropped but still counted)
          my_list[(size_t)r * list_cap + slot] = ((r & 1) ? a & 0xffff0000u : a << 16) | pos;
      }
  };

  uint32_t n_kept = 0;   // rows of the wave in LDS (wave-uniform)
  auto flush = [&]() {
    __builtin_amdgcn_wave_barrier();
    for (uint32_t i0 = 0; i0 < n_kept; i0 += 64) {
      const uint32_t i = min(i0 + lane, n_kept - 1);
      to_lists(L.s01[wv][i], L.s23[wv][i], L.pos[wv][i], i0 + lane < n_kept);
    }
    __builtin_amdgcn_wave_barrier();
    n_kept = 0;
  };

  const bool has_rows = wbegin < wend;   // wave-uniform
  {
    const SeqCodes seq_codes = seq_codes_of<M>(codes, pg, b, kv, Hkv, ctx_stride);
    int32_t* pg_lds = L.page;
    const int pg0 = PAGED ? (int)((uint32_t)begin >> seq_codes.shift) : 0;                  // first page slot of the chunk
    const int n_pg = PAGED ? (int)((uint32_t)(end - 1) >> seq_codes.shift) - pg0 + 1 : 0;   // (begin < end here)
    const bool pg_staged = PAGED && n_pg <= kPageSlice;
    // Rows are read U at a time per lane, one full step ahead of their use (two register sets
    // used alternately); loads are unconditional (row index clamped into the wave's range) so
    // that the wait before the gathers only covers the older of the two sets in flight.
    constexpr int U = 4;
    constexpr int STEP = 64 * U;
    uint4 rows_a[U][M / 16], rows_b[U][M / 16];
    auto load_rows = [&](int base, uint4 (&dst)[U][M / 16], bool pages_in_lds) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int j = base + u * 64 + lane;
        const int jl = j < wend ? j : wend - 1;
        const uint8_t* row;
        if (PAGED) {
          const int slot = (int)((uint32_t)jl >> seq_codes.shift);
          row = row_in_page<M>(seq_codes, pages_in_lds ? pg_lds[slot - pg0] : seq_codes.pages[slot], jl);
        } else {
          row = seq_codes.base + (size_t)jl * M;
        }
#pragma unroll
        for (int qd = 0; qd < M / 16; ++qd)
          dst[u][qd] = (RESHARED || PAGED) ? *(const uint4*)(row + ((uint32_t)(qd * 16) ^ sw.row_swz))
                                           : load_stream_u4(row + ((uint32_t)(qd * 16) ^ sw.row_swz));
      }
    };
    auto process = [&](int base, const uint4 (&rows)[U][M / 16]) {
      // Scores and the "reaches the threshold" wave masks are formed together, so the
      // gathered table entries die inside this straight-line block.  The masks live in scalar
      // registers; their popcounts cost no vector instructions.
      uint64_t any[U];
      uint32_t a01[U], a23[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        score_coarse<M>(rows[u], sw, a01[u], a23[u]);
        any[u] = (__builtin_amdgcn_ballot_w64((int32_t)(a01[u] & 0xffffu) >= T[0]) |
                  __builtin_amdgcn_ballot_w64((int32_t)(a01[u] >> 16) >= T[1]) |
                  __builtin_amdgcn_ballot_w64((int32_t)(a23[u] & 0xffffu) >= T[2]) |
                  __builtin_amdgcn_ballot_w64((int32_t)(a23[u] >> 16) >= T[3])) &
                 __builtin_amdgcn_ballot_w64(base + u * 64 + lane < wend);
        if (u & 1) __builtin_amdgcn_sched_barrier(0);   // two rows' gathers at a time: bounds live registers
      }
      uint32_t total = 0;
#pragma unroll
      for (int u = 0; u < U; ++u) total += (uint32_t)__popcll(any[u]);
      if (n_kept + total > CAP) {
        flush();
        if (total > CAP) {   // more in a step than fits
          to_lists(a01[0], a23[0], (uint32_t)(base + lane - (int)begin), __builtin_amdgcn_inverse_ballot_w64(any[0]));
          total -= (uint32_t)__popcll(any[0]);
          any[0] = 0;
          if (total > CAP) {
            to_lists(a01[1], a23[1], (uint32_t)(base + 64 + lane - (int)begin), __builtin_amdgcn_inverse_ballot_w64(any[1]));
            any[1] = 0;
            to_lists(a01[2], a23[2], (uint32_t)(base + 128 + lane - (int)begin), __builtin_amdgcn_inverse_ballot_w64(any[2]));
            any[2] = 0;
          }
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (__builtin_amdgcn_inverse_ballot_w64(any[u])) {
          const uint32_t slot = (uint32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(any[u] >> 32),
                                                                    __builtin_amdgcn_mbcnt_lo((uint32_t)any[u], n_kept));
          L.s01[wv][slot] = a01[u];
          L.s23[wv][slot] = a23[u];
          L.pos[wv][slot] = (uint16_t)(base + u * 64 + lane - (int)begin);
        }
        n_kept += (uint32_t)__popcll(any[u]);
      }
    };
    // The first rows are requested before the table is copied to LDS, so both latencies overlap.
    // (Every wave of the workgroup reaches the barrier, also one whose row range is empty.)
    if (has_rows) load_rows((int)wbegin, rows_a, false);
    load_coarse_table<M, NT>(lut, lut_layout(B, Hq, Hkv, M), prob, tbl);
    if (pg_staged)
      for (int i = tid; i < n_pg; i += NT) pg_lds[i] = seq_codes.pages[pg0 + i];
    combine_thresholds<4>(thr_lane, G - g4 * kHeadsPerGroup, P0, T);
    if (tid < kHeadsPerGroup) L.n_list[tid] = 0;
    __syncthreads();
#pragma unroll 1
    for (int base = (int)wbegin; base < wend; base += 2 * STEP) {
      load_rows(base + STEP, rows_b, pg_staged);
      process(base, rows_a);
      load_rows(base + 2 * STEP, rows_a, pg_staged);
      process(base + STEP, rows_b);
    }
  }
  flush();
  __syncthreads();
  if (tid < kHeadsPerGroup) my_count[tid] = L.n_list[tid];
}

#define A2ATS_STREAM_ARGS                                                                          \
  const uint8_t *__restrict__ codes, const int32_t *__restrict__ lut,                             \
      const int32_t *__restrict__ seq_lens, const int32_t *__restrict__ thr,                      \
      uint32_t *__restrict__ counts, uint32_t *__restrict__ lists, GridMap gm, CodePages pg,      \
      int B, int Hq, int Hkv, int G, int NG, int P0, int n_chunks, int rows_per_chunk,             \
      int list_cap, int ctx_len, int64_t ctx_stride, int top_k, int window, int n_sink
#define A2ATS_STREAM_PASS                                                                          \
  codes, lut, seq_lens, thr, counts, lists, gm, pg, B, Hq, Hkv, G, NG, P0, n_chunks,              \
      rows_per_chunk, list_cap, ctx_len, ctx_stride, top_k, window, n_sink

// 80 KB of LDS per workgroup, the table and what StreamLds has, so two fit a CU.  M = 16: 128 VGPRs -> 4 waves per
// SIMD (two workgroups per CU).
__global__ __launch_bounds__(kStreamThreads) __attribute__((amdgpu_waves_per_eu(4, 4)))
void stream_select_kernel16(A2ATS_STREAM_ARGS) { stream_select_body<16, false, false>(A2ATS_STREAM_PASS); }
__global__ __launch_bounds__(kStreamThreads) __attribute__((amdgpu_waves_per_eu(4, 4)))
void stream_select_kernel16r(A2ATS_STREAM_ARGS) { stream_select_body<16, true, false>(A2ATS_STREAM_PASS); }
__global__ __launch_bounds__(kStreamThreads) __attribute__((amdgpu_waves_per_eu(4, 4)))
void stream_select_kernel16p(A2ATS_STREAM_ARGS) { stream_select_body<16, true, true>(A2ATS_STREAM_PASS); }
// M = 32: twice the row registers.
__global__ __launch_bounds__(kStreamThreads) __attribute__((amdgpu_waves_per_eu(2, 4)))
void stream_select_kernel32(A2ATS_STREAM_ARGS) { stream_select_body<32, false, false>(A2ATS_STREAM_PASS); }
__global__ __launch_bounds__(kStreamThreads) __attribute__((amdgpu_waves_per_eu(2, 4)))
void stream_select_kernel32r(A2ATS_STREAM_ARGS) { stream_select_body<32, true, false>(A2ATS_STREAM_PASS); }
__global__ __launch_bounds__(kStreamThreads) __attribute__((amdgpu_waves_per_eu(4, 4)))
void stream_select_kernel32p(A2ATS_STREAM_ARGS) { stream_select_body<32, true, true>(A2ATS_STREAM_PASS); }

// ------------------------------------------------------------------------------------------
// Fast route, stage 3: exact selection from the lists, ordered output
// ------------------------------------------------------------------------------------------
// One workgroup per head, from the lists of the chunks.  What separates winners from the band, and why that is exact, is told in
// list_select.hpp.
//
// What bounds it: a chain of short dependent phases on one CU (entries, histogram, bin, winners, band rows from the code matrix,
// ranks, output).  Against exact scores of every survivor and a radix select: 14.5 -> 12.1 us (4 sequences of 131072 tokens, K
// 2048, 128 heads), 17.0 -> 12.2 (2 of 98301, K 2949).
//
// A band of more than 1024 rows, and more than 128 equal scores in the bin of the K-th, are ranked by a radix select over (score, position) from
// registers (by the exact route: ten times slower; by counting: 65 us instead of 51 for 800 equal scores).  Tables and selection,
// us, that exact scores of all survivors took -> now, 1100, 3000, 6000 equal scores about the K-th of one head in four: 4 sequences of 131072, M =
// 16, 49.6 -> 50.4, 55.1 -> 55.3, 428 -> 67; 2 of 98301 42.7 -> 42.8, 47.4 -> 46.0, 307 -> 56; 2 of 65536, M = 32, 54.6 -> 55.8, 59.5 -> 60.3,
// 330 -> 75.  M = 32 has such bands without equal scores: one selection per KV head, 16 of 122753, K 4096, 58 -> 59 (the exact route 608).
constexpr int kCounted = 128;         // rows in the bin of the K-th that are ranked by counting
constexpr int kFinalBin = 2;          // a bin of the first histogram is 4 coarse units, from the threshold up; of a second, where
constexpr int kFinalWide = 5;         // the K-th is above those, 32, which is the whole range
constexpr long kFinalTableCand = 1 << 19;   // candidates up to which the exact table is in LDS too
constexpr long kFinalMostCand = 1 << 20;    // the longest context
struct FinalLds {
  uint32_t hist[kHistBins];
  uint64_t band[kBandCap];
  uint32_t n, n_band, n_sure, wave_tot[kExactThreads / 64];
  int32_t bin, overflow;
  uint64_t won[1];   // a bit for each candidate
};
// The table, if it is there, comes first, and the positions of a crowded band last; the exact route takes all of it.
struct FinalRoom {
  int crowd_cap;
  size_t bytes;
};
template <int M>
FinalRoom final_room(long ncand) {
  constexpr size_t kMost = 160 * 1024;
  const size_t table = ncand <= kFinalTableCand ? kCentroids * M * sizeof(int32_t) : 0;
  const size_t fast = table + sizeof(FinalLds) + (size_t)(ncand + 63) / 64 * 8;
  const int crowd_cap = (int)std::min<size_t>(kFinalCrowd, (kMost - fast) / 4);
  return {crowd_cap, std::max(fast + crowd_cap * 4, kExactLdsBytes + sizeof(ExactLds))};
}

template <int M>
__global__ __launch_bounds__(kExactThreads) void final_select_kernel(
    const uint8_t* __restrict__ codes, const int32_t* __restrict__ lut,
    const float* __restrict__ lut_scale, const int32_t* __restrict__ seq_lens,
    const int32_t* __restrict__ thr, const uint32_t* __restrict__ counts,
    const uint32_t* __restrict__ lists, uint32_t* __restrict__ route, int32_t* __restrict__ topk_idx,
    int32_t* __restrict__ topk_count, float* __restrict__ topk_score, GridMap gm, CodePages pg, int B,
    int Hq, int Hkv, int G, int NG, int P0, int n_chunks, int rows_per_chunk, int list_cap, int table_in_lds, int crowd_cap,
    int ctx_len, int64_t ctx_stride, int top_k, int window, int n_sink) {
  constexpr int NT = kExactThreads;
  constexpr int KEEP = 6;   // entries of a thread that stay in registers
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  int32_t* table = (int32_t*)dyn_lds;
  FinalLds& L = *(FinalLds*)(dyn_lds + (table_in_lds ? kCentroids * M * sizeof(int32_t) : 0));

  // one workgroup per (problem, head slot), on the XCD that streamed the problem
  int prob, r, b, kv, g4;
  map_block(blockIdx.x, gm, prob, r);
  split_problem(prob, gm, b, kv, g4);
  const int hg = g4 * kHeadsPerGroup + r;
  if (hg >= G) return;
  const int bh = b * Hq + kv * G + hg, tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  // A group of lanes takes the list of a chunk: its entries are requested before its length is known (list_cap of them are
  // there whatever it is).  n_chunks <= 64.
  int lanes = NT;
  while (lanes * n_chunks > NT) lanes >>= 1;
  const int chunk = min(tid / lanes, n_chunks - 1), l0 = tid & (lanes - 1);
  const size_t list = ((size_t)prob * n_chunks + chunk) * kHeadsPerGroup + r;
  const uint32_t* my_list = lists + list * (size_t)list_cap;
  const uint32_t n_rows = tid / lanes < n_chunks ? counts[list] : 0u;
  uint32_t keep[KEEP];
#pragma unroll
  for (int k = 0; k < KEEP; ++k) keep[k] = my_list[min(l0 + k * lanes, list_cap - 1)];
  const int32_t thr_lane = request_thresholds<1>(thr, (size_t)bh, 1, P0);

  const SeqRange sr = seq_range(ctx_len, seq_lens, b, window, n_sink, top_k);
  int32_t* oi = topk_idx + (size_t)bh * top_k;
  if (tid == 0) topk_count[bh] = sr.kk;
  for (int t = sr.kk + tid; t < top_k; t += NT) {
    oi[t] = -1;
    if (topk_score) topk_score[(size_t)bh * top_k + t] = 0.f;
  }
  if (sr.kk == 0) {
    if (tid == 0) route[bh] = 0u;
    return;
  }
  const LutLayout lay = lut_layout(B, Hq, Hkv, M);
  const int32_t* head_table = lut + lay.off_exact + (size_t)bh * (kCentroids * M);
  const SeqCodes seq_codes = seq_codes_of<M>(codes, pg, b, kv, Hkv, ctx_stride);
  const int32_t* meta = lut + lay.off_meta + (size_t)bh * 4;
  const int32_t m_base = meta[0], m_shift = meta[1], m_top = meta[2];
  const float scale = lut_scale[bh];
  if (table_in_lds) {
#pragma unroll
    for (int i = tid; i < kCentroids * M / 4; i += NT) {
      const int c = i / (M / 4);   // (four entries are turned by their centroid, see band_select.hpp)
      ((uint4*)table)[c * (M / 4) + ((i + c) & (M / 4 - 1))] = ((const uint4*)head_table)[i];
    }
  }
  const int n_words = (sr.ncand + 63) / 64;
  for (int i = tid; i < n_words; i += NT) L.won[i] = 0;
  for (int i = tid; i < kHistBins; i += NT) L.hist[i] = 0;
  if (tid == 0) {
    L.n = 0;
    L.n_band = 0;
    L.n_sure = 0;
    L.overflow = 0;
  }
  int32_t t1[1];
  combine_thresholds<1>(thr_lane, 1, P0, t1);
  const uint32_t T = (uint32_t)max(t1[0], 0);
  __syncthreads();

  // f(coarse score, candidate) for every row of the head
  const uint32_t n_mine = min(n_rows, (uint32_t)list_cap), pos0 = (uint32_t)chunk * (uint32_t)rows_per_chunk;
  auto each = [&](auto f) {
#pragma unroll
    for (int k = 0; k < KEEP; ++k)
      if ((uint32_t)(l0 + k * lanes) < n_mine) f(keep[k] >> 16, pos0 + (keep[k] & 0xffffu));
    for (uint32_t i = l0 + KEEP * lanes; i < n_mine; i += lanes) {
      const uint32_t e = my_list[i];
      f(e >> 16, pos0 + (e & 0xffffu));
    }
  };
  if (l0 == 0) {
    atomicAdd(&L.n, n_mine);
    if (n_rows > (uint32_t)list_cap) L.overflow = 1;
  }
  int shift = kFinalBin;
  for (;;) {
    each([&](uint32_t s, uint32_t) { atomicAdd(&L.hist[min((s - T) >> shift, (uint32_t)kHistBins - 1)], 1u); });
    __syncthreads();
    if (wv == 0) {
      const int bin = wave_find_bin(L.hist, 0, (uint32_t)sr.kk, lane, ~0u);
      if (lane == 0) L.bin = bin;
    }
    __syncthreads();
    if (L.bin != kHistBins - 1 || shift == kFinalWide) break;   // (uniform)
    shift = kFinalWide;
    for (int i = tid; i < kHistBins; i += NT) L.hist[i] = 0;
    __syncthreads();
  }
  const int bin = __builtin_amdgcn_readfirstlane(L.bin);
  uint32_t why = L.overflow ? 3u : (bin < 0 ? 1u : (T != 0u && (bin << shift) < M - 1 ? 4u : 0u));
  const int edge = (int)T + (bin << shift);
  const uint32_t t_lo = (uint32_t)max(0, edge - M + 1), t_hi = (uint32_t)(edge + (1 << shift) + M);
  uint32_t* crowd = (uint32_t*)(L.won + ((ctx_len - window - n_sink + 63) >> 6));   // positions of the band's rows
  if (why == 0u) {
    uint32_t sure = 0;
    each([&](uint32_t s, uint32_t j) {
      if (s >= t_hi) {
        atomicOr((uint32_t*)L.won + (j >> 5), 1u << (j & 31));
        ++sure;
      } else if (s >= t_lo) {
        const uint32_t slot = atomicAdd(&L.n_band, 1u);
        if (slot < (uint32_t)crowd_cap) crowd[slot] = j;
      }
    });
    sure = wave_inclusive_scan(sure);
    if (lane == 63 && sure) atomicAdd(&L.n_sure, sure);
    __syncthreads();
    if (L.n_band > (uint32_t)crowd_cap) why = 2u;
  }
  if (tid == 0) route[bh] = min(L.n, 0x0fffffffu) | why << 28;   // diagnostics only
  if (why != 0u) {
    exact_select_block<M>(seq_codes, head_table, m_base, m_top, scale, sr, oi,
                          topk_score ? topk_score + (size_t)bh * top_k : nullptr, dyn_lds,
                          *(ExactLds*)(dyn_lds + kExactLdsBytes));
    return;
  }

  auto load_row = [&](uint32_t j, uint4 (&w)[M / 16]) {
    const uint8_t* row = row_ptr<M>(seq_codes, sr.sink_end + (int)j);
#pragma unroll
    for (int qd = 0; qd < M / 16; ++qd) w[qd] = *(const uint4*)(row + qd * 16);
  };
  auto exact_by_table = [&](const uint4 (&w)[M / 16]) {
    int32_t s = 0;
#pragma unroll
    for (int qd = 0; qd < M / 16; ++qd) {
      const uint32_t d[4] = {w[qd].x, w[qd].y, w[qd].z, w[qd].w};
#pragma unroll
      for (int t4 = 0; t4 < 16; ++t4) {
        const uint32_t c = (d[t4 >> 2] >> (8 * (t4 & 3))) & 0xffu;
        s += table[c * M + (((qd * 4 + (t4 >> 2) + c) & (M / 4 - 1)) << 2) + (t4 & 3)];
      }
    }
    return s;
  };
  auto exact_at = [&](uint32_t j) {
    if (!table_in_lds) return exact_score_of<M>(head_table, row_ptr<M>(seq_codes, sr.sink_end + (int)j));
    uint4 w[M / 16];
    load_row(j, w);
    return exact_by_table(w);
  };
  const uint32_t n_band = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.n_band), need = (uint32_t)sr.kk - L.n_sure;
  const uint32_t key0 = score_key((int32_t)((uint32_t)m_base + (t_lo << m_shift)));
  const uint32_t range = (t_hi - t_lo + M) << m_shift;   // (a coarse score leaves out less than M units)
  // (score, position) of a row in few bits: its score from the band's lower edge up, and of equal scores the lower position is larger
  constexpr int kPosBits = 20;
  static_assert(kFinalMostCand <= 1 << kPosBits, "");
  const int row_bits = kPosBits + 32 - (int)__clz(range);
  auto relative = [&](uint32_t key, uint32_t j) {
    return (uint64_t)(key > key0 ? min(key - key0, range) : 0u) << kPosBits | ((1u << kPosBits) - 1u - j);
  };
  bool crowded = n_band > (uint32_t)kBandCap;   // (uniform)
  if (!crowded) {
    // --- the band: exact keys, then every row counts those before it in (score, position) order; of many rows only those in the
    // bin of the K-th, of 2048 over the band's range (M = 32, 1000 rows: see band_select.hpp)
    const bool few = n_band <= 256u;
    const int kshift = max(0, 21 - (int)__clz(range));
    auto bin_of = [&](uint32_t key) { return min(key > key0 ? (key - key0) >> kshift : 0u, (uint32_t)kHistBins - 1); };
    if (!few) {
      for (int i = tid; i < kHistBins; i += NT) L.hist[i] = 0;
      __syncthreads();
    }
    if ((uint32_t)tid < n_band) {
      const uint32_t j = crowd[tid], key = score_key(exact_at(j));
      L.band[tid] = ((uint64_t)key << 32) | ~j;   // (of equal scores the lower position is larger)
      if (!few) atomicAdd(&L.hist[bin_of(key)], 1u);
    }
    __syncthreads();
    const int kth_bin = few ? 0 : wave_find_bin(L.hist, 0, need, lane, ~0u);
    crowded = !few && L.hist[kth_bin] > (uint32_t)kCounted;
    if (!crowded) {
      for (uint32_t i = tid >> 3; i < n_band; i += NT / 8) {   // eight lanes a row
        const uint64_t own = L.band[i];
        const int at = few ? 0 : (int)bin_of((uint32_t)(own >> 32));
        if (at < kth_bin) continue;
        int32_t before = 0;
        if (at == kth_bin) {
#pragma unroll 4
          for (uint32_t u = tid & 7; u < n_band; u += 8) before += L.band[u] > own ? 1 : 0;
          before = group8_sum(before);
        }
        if ((tid & 7) == 0 && (uint32_t)before < need) {
          const uint32_t j = ~(uint32_t)own;
          atomicOr((uint32_t*)L.won + (j >> 5), 1u << (j & 31));
        }
      }
    }
  }
  if (__builtin_expect(crowded, 0)) {
    // --- more rows than are ranked so (M = 32, thousands of winners; or equal scores): in registers
    constexpr int kTogether = 4;
    uint64_t row[kFinalCrowd / NT];
#pragma unroll
    for (int k0 = 0; k0 < kFinalCrowd / NT; k0 += kTogether) {
      uint4 w[kTogether][M / 16];
      uint32_t j[kTogether];
      if (k0 * NT >= (int)n_band) continue;   // (uniform)
#pragma unroll
      for (int k = 0; k < kTogether; ++k) j[k] = crowd[min((uint32_t)(tid + (k0 + k) * NT), n_band - 1)];
      if (table_in_lds) {   // (uniform)
#pragma unroll
        for (int k = 0; k < kTogether; ++k) load_row(j[k], w[k]);
#pragma unroll
        for (int k = 0; k < kTogether; ++k) row[k0 + k] = relative(score_key(exact_by_table(w[k])), j[k]);
      } else {
#pragma unroll
        for (int k = 0; k < kTogether; ++k) row[k0 + k] = relative(score_key(exact_at(j[k])), j[k]);
      }
    }
    const uint64_t last = reached_by<NT, true>(
        need, row_bits,
        [&](auto f) {
#pragma unroll
          for (int k = 0; k < kFinalCrowd / NT; ++k)
            if (k * NT < (int)n_band) f((uint32_t)(tid + k * NT) < n_band, row[k]);
        },
        L.hist, L.wave_tot, (uint32_t*)L.band);
#pragma unroll
    for (int k = 0; k < kFinalCrowd / NT; ++k)
      if ((uint32_t)(tid + k * NT) < n_band && row[k] >= last) {
        const uint32_t j = (1u << kPosBits) - 1u - ((uint32_t)row[k] & ((1u << kPosBits) - 1u));
        atomicOr((uint32_t*)L.won + (j >> 5), 1u << (j & 31));
      }
  }
  __syncthreads();
  // --- winners in ascending position
  {
    const int per = (n_words + NT - 1) / NT, w0 = tid * per, w1 = min(n_words, w0 + per);
    uint32_t n = 0;
    for (int w = w0; w < w1; ++w) n += (uint32_t)__popcll(L.won[w]);
    uint32_t total;
    uint32_t at = block_exclusive_scan<NT>(n, L.wave_tot, total);
    for (int w = w0; w < w1; ++w) {
      uint64_t word = L.won[w];
      while (word) {
        const uint32_t j = (uint32_t)w * 64 + __ffsll((unsigned long long)word) - 1;
        if (at < (uint32_t)sr.kk) {
          oi[at] = sr.sink_end + (int)j;
          if (topk_score) topk_score[(size_t)bh * top_k + at] = (float)exact_at(j) * scale;
        }
        ++at;
        word &= word - 1;
      }
    }
  }
}

// ------------------------------------------------------------------------------------------
// Host side
// ------------------------------------------------------------------------------------------
__global__ void fill_words_kernel(uint32_t* __restrict__ out, uint32_t value, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = value;
}

__global__ void copy_words_kernel(const uint32_t* __restrict__ in, uint32_t* __restrict__ out, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = in[i];
}

hipError_t copy_topk_stats(const a2ats_dims& d, int top_k, int window, int n_sink, const void* ws,
                           uint32_t* cand_counts, hipStream_t stream) {
  const TopkPlan plan = make_topk_plan(d, top_k, window, n_sink);
  const int heads = d.batch * d.n_q_heads;
  if (heads == 0) return hipSuccess;
  if (plan.fast) {
    hipLaunchKernelGGL(copy_words_kernel, dim3((heads + 255) / 256), dim3(256), 0, stream,
                       (const uint32_t*)((const unsigned char*)ws + plan.off_route), cand_counts, heads);
    return hipGetLastError();
  }
  // (a fill kernel, not a memset node: the call may be captured into a graph)
  hipLaunchKernelGGL(fill_words_kernel, dim3((heads + 255) / 256), dim3(256), 0, stream, cand_counts, 0xffffffffu, heads);
  return hipGetLastError();
}

template <int M>
static hipError_t launch_score_topk_m(const a2ats_dims& d, const TopkPlan& plan, const uint8_t* codes,
                                      const CodePages& pg, const int32_t* lut, const float* lut_scale, int top_k, int window,
                                      int n_sink, const int32_t* seq_lens, int32_t* topk_idx,
                                      int32_t* topk_count, float* topk_score, float* scores_out,
                                      void* ws, int presampled, hipStream_t stream, hipEvent_t ev_start,
                                      hipEvent_t ev_stop) {
  const int B = d.batch, Hq = d.n_q_heads, Hkv = d.n_kv_heads, NG = plan.NG;
  const int heads = B * Hq, problems = B * Hkv * NG;
  const size_t coarse_bytes = (size_t)kCoarseLdsBytes;
  const size_t lut1_bytes = kExactLdsBytes;
  hipError_t err;
  static LdsSlot s_dense[16], s_exact[16], s_sample[16], s_stream[16], s_stream_r[16], s_stream_p[16], s_final[16], s_group[16], s_group_many[16],
      s_list[16];
  if (heads == 0) return hipSuccess;

  if (scores_out) {
    if ((err = allow_dynamic_lds(score_dense_kernel<M>, lut1_bytes, s_dense)) != hipSuccess) return err;
    int gx = (d.ctx_len + kStreamThreads * 8 - 1) / (kStreamThreads * 8);
    gx = gx < 1 ? 1 : gx;
    hipLaunchKernelGGL((score_dense_kernel<M>), dim3(gx, heads), dim3(kStreamThreads), lut1_bytes, stream,
                       codes, lut, lut_scale, seq_lens, scores_out, pg, B, Hq, Hkv, d.ctx_len, d.ctx_stride);
    if ((err = hipGetLastError()) != hipSuccess) return err;
  }

  const bool streams = plan.fast || (plan.wide && ws);
  if (!streams && takes_group_route(d, window, n_sink)) {
    const int heads = std::min(Hq / Hkv, kHeadsPerGroup), split = group_split(problems, heads, 0);
    const bool many = group_many(M, (long)d.ctx_len - window - n_sink, top_k, (heads + split - 1) / split);
    auto kernel = many ? group_select_kernel<M, M == 32> : group_select_kernel<M, false>;
    if ((err = allow_dynamic_lds(kernel, kGroupLdsBytes, many ? s_group_many : s_group, true)) != hipSuccess) return err;
    hipLaunchKernelGGL(kernel, dim3(problems * split), dim3(kGroupThreads), kGroupLdsBytes, stream, codes,
                       lut, lut_scale, seq_lens, topk_idx, topk_count, topk_score, make_grid_map(split, problems, NG, Hkv),
                       pg, B, Hq, Hkv, d.ctx_len, d.ctx_stride, top_k, window, n_sink, split);
    return hipGetLastError();
  }
  if (!streams) {
    if ((err = allow_dynamic_lds(select_exact_kernel<M>, lut1_bytes, s_exact)) != hipSuccess) return err;
    hipLaunchKernelGGL((select_exact_kernel<M>), dim3(heads), dim3(kExactThreads), lut1_bytes, stream,
                       codes, lut, lut_scale, seq_lens, topk_idx, topk_count, topk_score, pg, B, Hq, Hkv,
                       d.ctx_len, d.ctx_stride, top_k, window, n_sink);
    return hipGetLastError();
  }

  unsigned char* wsb = (unsigned char*)ws;
  if (plan.list) {
    if ((err = allow_dynamic_lds(list_select_kernel<M>, kListLdsBytes, s_list, true)) != hipSuccess) return err;
    const GridMap gm = make_grid_map(1, problems, NG, Hkv);
    uint32_t* stats = (uint32_t*)(wsb + plan.off_route);
    if (ev_start && ev_stop)   // (attached to the dispatch)
      hipExtLaunchKernelGGL((list_select_kernel<M>), dim3(problems), dim3(kListThreads), kListLdsBytes, stream, ev_start, ev_stop,
                            0, codes, lut, lut_scale, seq_lens, topk_idx, topk_count, topk_score, stats, gm, pg, plan.list_rows, B,
                            Hq, Hkv, NG, d.ctx_len, d.ctx_stride, top_k, window, n_sink);
    else
      hipLaunchKernelGGL((list_select_kernel<M>), dim3(problems), dim3(kListThreads), kListLdsBytes, stream, codes, lut, lut_scale,
                         seq_lens, topk_idx, topk_count, topk_score, stats, gm, pg, plan.list_rows, B, Hq, Hkv, NG, d.ctx_len,
                         d.ctx_stride, top_k, window, n_sink);
    return hipGetLastError();
  }
  int32_t* thr = (int32_t*)(wsb + plan.off_thr);
  uint32_t* counts = (uint32_t*)(wsb + plan.off_count);
  uint32_t* route = (uint32_t*)(wsb + plan.off_route);
  uint32_t* lists = (uint32_t*)(wsb + plan.off_cand);

  if (!presampled) {   // (the fused decode launch has written the thresholds already)
    if ((err = allow_dynamic_lds(sample_threshold_kernel<M>, coarse_bytes + kSampleHistBytes, s_sample, true)) != hipSuccess) return err;
    hipLaunchKernelGGL((sample_threshold_kernel<M>), dim3(plan.P0 * problems), dim3(kSampleThreads),
                       coarse_bytes + kSampleHistBytes, stream, codes, lut, seq_lens, thr, pg, B, Hq, Hkv, NG, plan.P0, plan.sample_rows,
                       problems, d.ctx_len, d.ctx_stride, top_k, window, n_sink);
    if ((err = hipGetLastError()) != hipSuccess) return err;
  }

  const bool paged = pg.table != nullptr;
  auto stream_kernel = paged ? (M == 16 ? stream_select_kernel16p : stream_select_kernel32p)
                             : (M == 16 ? (NG > 1 ? stream_select_kernel16r : stream_select_kernel16)
                                        : (NG > 1 ? stream_select_kernel32r : stream_select_kernel32));
  const int list_cap = plan.row_cap * kStreamWaves;
  const size_t stream_lds = coarse_bytes + (paged ? sizeof(StreamLds<true>) : sizeof(StreamLds<false>));
  if ((err = allow_dynamic_lds(stream_kernel, stream_lds, paged ? s_stream_p : (NG > 1 ? s_stream_r : s_stream), true)) !=
      hipSuccess)
    return err;
  // (the index arithmetic of a workgroup -- which problem, which part of it -- is prepared here:
  // its divisions would otherwise be the first thing every wave does)
  const int G = Hq / Hkv;
  const GridMap gm_stream = make_grid_map(plan.chunks, problems, NG, Hkv);
  if (ev_start && ev_stop) {
    // events attached to the dispatch itself: their difference is the kernel's own duration
    hipExtLaunchKernelGGL(stream_kernel, dim3(plan.chunks * problems), dim3(kStreamThreads), stream_lds,
                          stream, ev_start, ev_stop, 0, codes, lut, seq_lens, thr, counts, lists, gm_stream, pg, B,
                          Hq, Hkv, G, NG, plan.P0, plan.chunks, plan.rows_per_chunk,
                          list_cap, d.ctx_len, d.ctx_stride, top_k, window, n_sink);
  } else {
    hipLaunchKernelGGL(stream_kernel, dim3(plan.chunks * problems), dim3(kStreamThreads), stream_lds,
                       stream, codes, lut, seq_lens, thr, counts, lists, gm_stream, pg, B, Hq, Hkv, G, NG, plan.P0,
                       plan.chunks, plan.rows_per_chunk, list_cap,
                       d.ctx_len, d.ctx_stride, top_k, window, n_sink);
  }
  if ((err = hipGetLastError()) != hipSuccess) return err;

  const long ncand = (long)d.ctx_len - window - n_sink;
  const FinalRoom room = final_room<M>(ncand);
  // (allowed once for all contexts: threads that each raise it to their own call's size could lower one another's)
  const size_t final_most = std::max(final_room<M>(kFinalTableCand).bytes, final_room<M>(kFinalMostCand).bytes);
  if ((err = allow_dynamic_lds(final_select_kernel<M>, final_most, s_final)) != hipSuccess) return err;
  hipLaunchKernelGGL((final_select_kernel<M>), dim3(problems * kHeadsPerGroup), dim3(kExactThreads),
                     room.bytes, stream, codes, lut, lut_scale, seq_lens, thr, counts, lists, route, topk_idx,
                     topk_count, topk_score, make_grid_map(kHeadsPerGroup, problems, NG, Hkv), pg, B, Hq, Hkv, G, NG,
                     plan.P0, plan.chunks, plan.rows_per_chunk, list_cap,
                     ncand <= kFinalTableCand ? 1 : 0, room.crowd_cap, d.ctx_len, d.ctx_stride, top_k, window, n_sink);
  return hipGetLastError();
}

__global__ void codes_to_pages_kernel(const uint8_t* __restrict__ rows, uint8_t* __restrict__ pool, CodePages pg,
                                      int Hkv, int n_new, int pos0, int row_bytes, int total) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;   // one 4-byte word of one row
  const int wpr = row_bytes / 4;
  if (i >= total) return;
  const int w = i % wpr, r = i / wpr, t = r % n_new, bkv = r / n_new, kv = bkv % Hkv, b = bkv / Hkv;
  const int j = pos0 + t;
  const size_t page = (size_t)pg.table[(size_t)b * pg.pages_per_seq + (j >> pg.shift)];
  const size_t dst = ((page * Hkv + kv) << pg.shift) + (size_t)(j & ((1 << pg.shift) - 1));
  ((uint32_t*)(pool + dst * row_bytes))[w] = ((const uint32_t*)(rows + (size_t)r * row_bytes))[w];
}

hipError_t launch_codes_to_pages(const a2ats_dims& d, const uint8_t* rows, int n_new, int pos0, int row_bytes,
                                 uint8_t* pool, const CodePages& pg, hipStream_t stream) {
  const long total = (long)d.batch * d.n_kv_heads * n_new * (row_bytes / 4);
  if (total == 0) return hipSuccess;
  hipLaunchKernelGGL(codes_to_pages_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream, rows, pool,
                     pg, d.n_kv_heads, n_new, pos0, row_bytes, (int)total);
  return hipGetLastError();
}

hipError_t launch_score_topk(const a2ats_dims& d, const uint8_t* codes, const CodePages& pg, const int32_t* lut,
                             const float* lut_scale, int top_k, int window, int n_sink,
                             const int32_t* seq_lens, int32_t* topk_idx, int32_t* topk_count,
                             float* topk_score, float* scores_out, void* ws, int presampled,
                             hipStream_t stream, hipEvent_t ev_start, hipEvent_t ev_stop) {
  TopkPlan plan = make_topk_plan(d, top_k, window, n_sink, seq_lens != nullptr);
  if (presampled) plan.P0 = presampled;
  if (d.n_sub == 16)
    return launch_score_topk_m<16>(d, plan, codes, pg, lut, lut_scale, top_k, window, n_sink, seq_lens,
                                   topk_idx, topk_count, topk_score, scores_out, ws, presampled, stream,
                                   ev_start, ev_stop);
  return launch_score_topk_m<32>(d, plan, codes, pg, lut, lut_scale, top_k, window, n_sink, seq_lens,
                                 topk_idx, topk_count, topk_score, scores_out, ws, presampled, stream,
                                 ev_start, ev_stop);
}

}  // namespace a2ats
