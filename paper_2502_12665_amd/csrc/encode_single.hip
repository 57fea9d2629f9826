// Key encoder for the paper's own geometry (section 5.1: one codebook of 4096 codewords over all
// D = 128 dimensions; section 4.2: query-aware assignment with the full D x D matrix H):
//     code = argmin_c (k - c) H (k - c)^T ,  lowest c on exact ties.
//
// With the Cholesky factor of section 4.2 (H = L L^T, z = k L, c^z = c L) the distortion is the
// plain squared distance ||z - c^z||^2, and minimising it over c is minimising
//     s_c = 1/2 ||c^z||^2 - k . w_c ,   w_c = c H ,  ||c^z||^2 = c . w_c ,
// a dense [keys x 128] . [128 x 4096] contraction: 1 Mflop per key, the one matrix-core shape of
// this library.
//
// Distortions do not change when keys and codewords are moved together, but products, whose rounding goes with |k| |w|, are
// the larger the more all of them have in common.  So everything below is about keys and codewords less a centre of the
// codewords, and the matrix-core operands are balanced per dimension by powers of two t: k t . w / t.  160000 keys in all,
// 8 KV heads, all of them around 16 in every dimension: 8045 -> 381 us (nearly every key went to the float64 sweep before);
// variances 1 and 1e4 by dimension: 1297 -> 549; around the origin 375 -> 377.
//
// The kernels:
//
//   encode_single_matrix_kernel    H in float64 and the norms of its rows; in other workgroups the means that the centre is taken
//                                  from, and a copy of the codewords
//   encode_single_codewords_kernel the centre and t; w_c in float64, kept transposed for the exact decisions,
//                                  1/2 ||c^z||^2 = 1/2 c . w_c, and the largest norms
//   encode_single_operands_kernel  w_c in matrix-core operand order: rounded to f16, and as two bf16
//                                  terms (hi + lo, 16 significant bits)
//   encode_single_sample_kernel    128 keys of a KV head, which say which of the two filters it takes; of a short call all keys
//   encode_single_decide_kernel    a short call's keys: decided by the sample's products, or listed
//   encode_single_filter_kernel    every key of a longer one, by one of two filters:
//                                  - i8: scores from one product of whole numbers of 8 bits; keys that their rounding leaves
//                                  open are listed
//                                  - f16: the same with scores from one f16 product (11 significant bits per operand): the two
//                                  smallest and the code of the first are kept per key.  Where they are further apart than
//                                  the rounding of the operands can account for -- its norm is known for every key and
//                                  bounded for the codewords -- the code is decided; the other keys are listed.
//   encode_single_kernel           the listed keys, 256 at a time: three bf16 products per term
//                                  (hi.hi + hi.lo + lo.hi, float32 accumulate) give the scores to
//                                  about 2^-17 relative.  Every lane owns one key column of the
//                                  32 x 32 result tile, so the running smallest three scores (and
//                                  the codes of the first two) are per-lane registers; nothing
//                                  crosses lanes until the end.
//   encode_single_recheck_kernel   keys whose two smallest scores are closer than the rounding reach
//                                  of the bf16 products are decided in float64 between those two
//                                  codewords; keys with three that close by a float64 sweep over all
//                                  4096, and again between those that its rounding leaves open.  So the
//                                  emitted code is the float64 argmin.
//   encode_single_sweep_kernel     the few-key (decode-time append) route: one float64 pass of dot
//                                  products k . w_c decides the key; 16 workgroups per key, then
//                                  encode_single_sweep_pick_kernel.  More keys, and those of a decode
//                                  step's first launch, are swept in single_codebook.hip
//   encode_single_factor_kernel    per KV head: L in float64 (Cholesky in LDS; seeding only)
//   encode_single_transform_kernel z = k L in float64, rounded once to float32 (seeding only)
#include <algorithm>
#include "common.hpp"
#include "internal.hpp"

namespace a2ats {
namespace {

constexpr int kCW = 4096;               // codewords per KV head
constexpr int kD = 128;                 // head dimension
constexpr int kEncWaves = 4;           // two workgroups per CU: one wave of each per SIMD
constexpr int kEncThreads = 64 * kEncWaves;
constexpr int kKeysPerWave = 64;        // two 32-key column tiles
constexpr int kKeysPerWG = kKeysPerWave * kEncWaves;
constexpr int kFragBytes = 2 * 8 * 64 * 16;   // (hi, lo) x 8 k-steps x 64 lanes x 16 bytes: 32 rows of 128 dims
constexpr int kBlocks = kCW / 32;       // streamed 32-codeword blocks
static_assert(kFragBytes / 16 / kEncThreads == 4, "a thread stages four 16-byte pieces of a block");
constexpr int kFewSingle = kFewSingleKeys;   // at most this many keys per (sequence, KV head): float64 sweep only
constexpr int kSlices = kEncodeSlices;  // workgroups sharing the codewords of one such key
// Rounding reach of two scores s of the bf16 products: the split operands' (3 * 2^-18 of |k| max|w| each) and the float32
// sums', which start at 1/2 |c^z|^2 = s + k . w and take 24 products (25 * 2^-23 of s each; what they lose of k . w is in
// the slack of the first figure).  Where |k| is short against the codewords the second is all there is.
constexpr float kSplitReach = 2.5e-5f, kSumReach = 6e-6f;
constexpr int kF16Bytes = 8 * 64 * 16;  // 8 k-steps x 64 lanes x 16 bytes: 32 codewords of 128 dims in f16
constexpr int kI8Bytes = 32 * kD;       // the same in i8, a codeword after the other
constexpr int kSampleKeys = 128;        // keys of a KV head that say which filter it takes,
constexpr int kSampleSlices = 32;       // against so many slices of the codewords (16: 11.2 us, 32: 7.5)
constexpr int kSampleOpen = 4;          // and how many of them the i8 filter may leave open

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(16))) int i32x16;

// Of a KV head, over its codewords (float bits, which order like the values).
struct alignas(128) CodewordStat {   // (a cache line each: they are filled by atomics)
  uint32_t w_max, c_max, bias_max;   // largest |w / t|, |c t| and 1/2 |c^z|^2, rounded up
  uint32_t w_err;                    // largest |w - f16(w)|, in the scaled units of the f16 operands
  uint32_t w_elem, c_elem;           // largest magnitude of an element of w / t and of c t
  uint32_t w_err8;                   // largest |w - i8(w)|, in the scaled units of the i8 operands
};

// What is subtracted from every key and codeword of a KV head, and the powers of two t.
struct alignas(32) Center {
  float mu[kD], key[kD], t[kD];   // (key: t by the scale of the f16 operands)
  float key8[kD];                 // t by the scale of the i8 operands
};
__device__ __forceinline__ float inverse_of_power(float t) { return __uint_as_float((254u << 23) - __float_as_uint(t)); }
constexpr int kMeans = 16;   // shares of the codewords whose means the centre is the median of

// Smallest three scores of a listed key over a slice of the codewords, and the codes of the first two.
struct NearPart {
  float s1, s2, s3;
  uint32_t codes;
};
constexpr int kMaxSlices = 16;
constexpr int kFoundStride = 64;   // words between the counts of two KV heads' keys for float64 (a cache line each)
// Workgroups per KV head that work on its list.
inline long near_groups(const a2ats_dims& d) { return d.n_kv_heads < 512 ? 512 / d.n_kv_heads : 1; }

struct EncWs {
  size_t off_L, off_sd, off_hmat, off_means, off_center, off_copy, off_wT, off_chalf, off_cfrag, off_cbias, off_f16,
      off_fbias, off_i8, off_bias8, off_cstat, off_sample, off_norms, off_eight, off_count, off_list, off_near,
      off_near_part, off_part, bytes;
  size_t near_cap;   // keys of a KV head
};

EncWs enc_single_ws(const a2ats_dims& d) {
  const size_t Hkv = (size_t)d.n_kv_heads;
  const size_t keys_max = (size_t)d.batch * Hkv * (size_t)d.ctx_stride;
  EncWs w;
  size_t o = 0;
  auto take = [&](size_t bytes) {
    const size_t at = o;
    o += (bytes + 255) & ~(size_t)255;
    return at;
  };
  w.off_L = take(Hkv * kD * kD * sizeof(double));
  w.off_sd = take(Hkv * kD * sizeof(double));
  w.off_hmat = take(Hkv * kD * kD * sizeof(double));
  w.off_means = take(Hkv * kMeans * kD * sizeof(double));
  w.off_center = take(Hkv * sizeof(Center));
  w.off_copy = take(Hkv * kCW * kD * sizeof(double));   // (float32: the size is what callers have always brought)
  w.off_wT = take(Hkv * kD * kCW * sizeof(double));
  w.off_chalf = take(Hkv * kCW * sizeof(double));
  w.off_cfrag = take(Hkv * kBlocks * (size_t)kFragBytes);
  w.off_cbias = take(Hkv * kCW * sizeof(float));
  w.off_f16 = take(Hkv * kBlocks * (size_t)kF16Bytes);
  w.off_fbias = take(Hkv * kCW * sizeof(float));
  w.off_i8 = take(Hkv * kBlocks * (size_t)kI8Bytes);
  w.off_bias8 = take(Hkv * kCW * sizeof(int));
  w.off_cstat = take(Hkv * sizeof(CodewordStat));
  w.off_sample = take(Hkv * kSampleSlices * kSampleKeys * sizeof(int2));
  w.off_norms = take(Hkv * kSampleKeys * sizeof(float2));
  w.off_eight = take(Hkv * sizeof(uint32_t));
  // listed keys per KV head, arrivals per KV head and chunk of its list
  w.off_count = take((Hkv + Hkv * (size_t)near_groups(d)) * sizeof(uint32_t));
  w.off_list = take(keys_max * 2 * sizeof(uint32_t));   // keys for float64, by KV head; their counts are in the factor's place
  w.near_cap = (size_t)d.batch * (size_t)d.ctx_stride;
  w.off_near = take(keys_max * sizeof(uint32_t));
  w.off_near_part = take(Hkv * (size_t)near_groups(d) * kKeysPerWG * sizeof(NearPart));
  w.off_part = take((size_t)d.batch * Hkv * kFewSingle * kSlices * 2 * sizeof(double));
  w.bytes = o;
  return w;
}

// Scales of the f16 operands: powers of two that bring the largest |c| into [4, 8) -- keys up to 8000 times as
// long then fit f16 -- and the largest |w| into [64, 128).  False: out of reach of such a scale.
__device__ __forceinline__ bool f16_scales(const CodewordStat& st, float& key_scale, float& w_scale) {
  const int ec = (int)(st.c_max >> 23) - 127, ew = (int)(st.w_max >> 23) - 127;   // (inf and NaN: 128)
  const bool ok = ec > -60 && ec < 60 && ew > -60 && ew < 60;
  key_scale = ok ? __uint_as_float((uint32_t)(127 + 2 - ec) << 23) : 1.f;
  w_scale = ok ? __uint_as_float((uint32_t)(127 + 6 - ew) << 23) : 1.f;
  return ok;
}

// Scales of the i8 operands: the largest element of c becomes 100 (keys reach a little further out than their codewords; what
// is beyond 127 is cut off and counted as an error), of w 127.  False: out of reach, or 1/2 |c^z|^2 is too large against the
// products for a score of 22 bits.
__device__ __forceinline__ bool i8_scales(const CodewordStat& st, float& key_scale, float& w_scale) {
  const float c = __uint_as_float(st.c_elem), w = __uint_as_float(st.w_elem);
  const int ec = (int)(st.c_max >> 23) - 127, ew = (int)(st.w_max >> 23) - 127;
  const bool ok = ec > -60 && ec < 60 && ew > -60 && ew < 60;
  key_scale = ok ? 100.f / c : 1.f;
  w_scale = ok ? 127.f / w : 1.f;
  return ok && __uint_as_float(st.bias_max) * (key_scale * w_scale) < 2e6f;
}

// ------------------------------------------------------------------------------------------
// Per KV head: the factor L (H = L L^T) for the seeding, 16 columns at a time.  Every wave holds the 16 diagonal rows of the panel in
// lanes 0 .. 15 (all four factor them, so nothing is exchanged) and 48 of the rows below in the others, a row per
// lane; a column's pivot and multipliers come from the diagonal rows by lane reads.  The rest of the matrix is then
// updated on the float64 matrix cores.  What bounds it: the chain of square roots and divisions, 63 us (225 with a
// column at a time, three barriers each).
// ------------------------------------------------------------------------------------------
typedef __attribute__((ext_vector_type(4))) double f64x4;
constexpr int kFactorStride = kD + 1;   // (rows start on different LDS banks)

__device__ __forceinline__ double lane_value(double v, int src_lane) {   // src_lane: a constant
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)b, src_lane), hi = __builtin_amdgcn_readlane((uint32_t)(b >> 32), src_lane);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void encode_single_factor_kernel(
    const float* __restrict__ weights, int mode, double* __restrict__ Lmat, double* __restrict__ sd) {
  extern __shared__ double s_A[];   // 128 rows, lower triangle in use
  const int kv = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double* L = Lmat + (size_t)kv * kD * kD;
  if (mode != A2ATS_W_BLOCK) {
    if (tid < kD) sd[(size_t)kv * kD + tid] = mode == A2ATS_W_DIAG ? sqrt((double)weights[(size_t)kv * kD + tid]) : 1.0;
    return;
  }
  const float* H = weights + (size_t)kv * kD * kD;
  for (int e = tid; e < kD * kD; e += 256) s_A[(e / kD) * kFactorStride + e % kD] = (e % kD) <= (e / kD) ? (double)H[e] : 0.0;
  __syncthreads();
#pragma unroll 1
  for (int p = 0; p < kD / 16; ++p) {
    const int j0 = 16 * p;
    const int row = lane < 16 ? j0 + lane : j0 + 16 + wave * 48 + lane - 16;
    double* own = s_A + (row < kD ? row : kD - 1) * kFactorStride + j0;
    double a[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) a[j] = own[j];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const double s = lane_value(a[j], j), d = sqrt(s > 0.0 ? s : 0.0);
      a[j] = lane == j ? d : (d > 0.0 ? a[j] / d : 0.0);
#pragma unroll
      for (int k = j + 1; k < 16; ++k) a[k] -= a[j] * lane_value(a[j], k);
    }
    __syncthreads();   // (the diagonal rows have been read by all waves)
    if (lane < 16 ? wave == 0 : row < kD) {
#pragma unroll
      for (int j = 0; j < 16; ++j) own[j] = a[j];   // (above the diagonal: never read as part of L)
    }
    __syncthreads();
    // rest -= panel panel^T, tiles on and below the diagonal
    const int c = lane & 15, k = lane >> 4;
    int t = 0;
    for (int bi = p + 1; bi < kD / 16; ++bi)
      for (int bj = p + 1; bj <= bi; ++bj, ++t) {
        if ((t & 3) != wave) continue;
        double* tile = s_A + (16 * bi + k) * kFactorStride + 16 * bj + c;   // register r: row 4 r + k, column c
        f64x4 acc;
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[r] = tile[4 * r * kFactorStride];
#pragma unroll
        for (int u = 0; u < 4; ++u)
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-s_A[(16 * bi + c) * kFactorStride + j0 + 4 * u + k],
                                                     s_A[(16 * bj + c) * kFactorStride + j0 + 4 * u + k], acc, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) tile[4 * r * kFactorStride] = acc[r];
      }
    __syncthreads();
  }
  for (int e = tid; e < kD * kD; e += 256) L[e] = (e % kD) <= (e / kD) ? s_A[(e / kD) * kFactorStride + e % kD] : 0.0;
}

// ------------------------------------------------------------------------------------------
// What the codewords are weighed with: H in float64, mirrored from its lower triangle, and the norms of its rows (full-matrix
// mode), or the square roots of the weights.  In other workgroups the means that the centre is taken from.
// What bounds it: reading the codewords and writing the copy, 11 us for 8 KV heads.  (The Cholesky factor and L L^T stood here, 62 +
// 9 us of a chain that used 8 CUs; scores need no L, as |c^z|^2 = c H c^T = c . w, and decisions between two codewords take H.)
// ------------------------------------------------------------------------------------------
constexpr int kMatrixRows = 16, kMatrixThreads = 1024;   // rows of H a workgroup
__global__ __launch_bounds__(kMatrixThreads) void encode_single_matrix_kernel(
    const float* __restrict__ weights, int mode, double* __restrict__ hmat, double* __restrict__ sd,
    CodewordStat* __restrict__ cstat, const float* __restrict__ codebook, double* __restrict__ means, float* __restrict__ copy) {
  constexpr int kSub = kMatrixThreads / kD;
  __shared__ double s_sum[kSub][kD];
  const int kv = blockIdx.x, part = (int)blockIdx.y - kMeans, t = threadIdx.x & (kD - 1), sub = threadIdx.x / kD;
  if (part < 0) {   // the mean of one share of the codewords; and a copy of them, for calls that come with A2ATS_W_PREPARED
    constexpr int kRows = kCW / kMeans;
    const size_t at = ((size_t)kv * kCW + blockIdx.y * kRows + sub * (kRows / kSub)) * kD + t;
    double sum = 0.0;
#pragma unroll 16
    for (int r = 0; r < kRows / kSub; ++r) {
      const float c = codebook[at + (size_t)r * kD];
      copy[at + (size_t)r * kD] = c;
      sum += (double)c;
    }
    s_sum[sub][t] = sum;
    __syncthreads();
    if (sub == 0) {
#pragma unroll
      for (int i = 1; i < kSub; ++i) sum += s_sum[i][t];
      means[((size_t)kv * kMeans + blockIdx.y) * kD + t] = sum * (1.0 / kRows);
    }
    return;
  }
  if (part == 0 && threadIdx.x == 0) cstat[kv] = CodewordStat{};
  if (mode != A2ATS_W_BLOCK) {
    if (part == 0 && sub == 0) sd[(size_t)kv * kD + t] = mode == A2ATS_W_DIAG ? sqrt((double)weights[(size_t)kv * kD + t]) : 1.0;
    return;
  }
  const float* H = weights + (size_t)kv * kD * kD;
  constexpr int kPer = kMatrixRows / kSub;
  const int i0 = part * kMatrixRows + sub * kPer;
#pragma unroll
  for (int r = 0; r < kPer; ++r) {
    const double h = (double)H[t <= i0 + r ? (size_t)(i0 + r) * kD + t : (size_t)t * kD + i0 + r];
    hmat[((size_t)kv * kD + i0 + r) * kD + t] = h;
    double n = h * h;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) n += __shfl_xor(n, off);
    if ((t & 63) == 0) s_sum[sub][kPer * (t >> 6) + r] = n;   // (the two waves of a row)
  }
  __syncthreads();
  if (t < kPer) sd[(size_t)kv * kD + i0 + t] = sqrt(s_sum[sub][t] + s_sum[sub][kPer + t]);
}

// ------------------------------------------------------------------------------------------
// w = c H and |c^z|^2 = c H c^T = c . w in float64, c less the centre, and the largest norms.  A wave takes 16 codewords and all
// dimensions, on the float64 matrix cores: the matrix is the first operand (a row of the result is a dimension), the codewords the second
// (a column is a codeword), so a lane's results belong to one codeword and are written to consecutive addresses.
// The centre: every workgroup finds it again from the 16 means, which is less than one more launch takes.  (With c L for the norms
// besides, and written: 51 us; now 44, 8 KV heads, full matrix.)
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void encode_single_codewords_kernel(
    const float* __restrict__ codebook, int mode, const double* __restrict__ sd, const double* __restrict__ hmat,
    const double* __restrict__ means, Center* __restrict__ center, double* __restrict__ wT, double* __restrict__ chalf, float* __restrict__ cbias,
    CodewordStat* __restrict__ cstat) {
  __shared__ float s_mu[kD], s_t[kD];
  const int kv = blockIdx.y, lane = threadIdx.x & 63, c = lane & 15, k = lane >> 4;
  const int cg = blockIdx.x * 64 + (threadIdx.x >> 6) * 16 + c;
  const float* cw = codebook + ((size_t)kv * kCW + cg) * kD + k;
  float cv[kD / 4];   // dimensions k, 4 + k, ... of codeword cg
#pragma unroll
  for (int u = 0; u < kD / 4; ++u) cv[u] = cw[4 * u];
  if (threadIdx.x < kD) {
    // The centre of a dimension is the median of the means of the shares, so that a few codewords far out (or not finite) do
    // not draw it away from the others, whose last bits it would cost.  t: the power of two next to the square root of the
    // norm of the matrix's row, which is by how much w is longer than c in this dimension, so that k t and w / t are evenly
    // long.
    const int d = threadIdx.x;
    float m[kMeans], mu = 0.f;
#pragma unroll
    for (int i = 0; i < kMeans; ++i) {
      m[i] = (float)means[((size_t)kv * kMeans + i) * kD + d];
      if (!(fabsf(m[i]) < INFINITY)) m[i] = INFINITY;
    }
#pragma unroll
    for (int i = 0; i < kMeans; ++i) {
      int below = 0;
#pragma unroll
      for (int j = 0; j < kMeans; ++j) below += m[j] < m[i] || (m[j] == m[i] && j < i) ? 1 : 0;
      if (below == kMeans / 2) mu = m[i];
    }
    if (!(fabsf(mu) < INFINITY)) mu = 0.f;
    const double sd_d = sd[(size_t)kv * kD + d], h = mode == A2ATS_W_BLOCK ? sd_d : sd_d * sd_d;
    const int e = (int)(__float_as_uint((float)h) >> 23) - 127;   // (negative, infinite, not a number: above 100)
    const float t = e > -80 && e < 80 ? __uint_as_float((uint32_t)(127 + ((e + 1) >> 1)) << 23) : 1.f;
    s_mu[d] = mu;
    s_t[d] = t;
    if (blockIdx.x == 0) {
      center[kv].mu[d] = mu;
      center[kv].t[d] = t;
    }
  }
  __syncthreads();
  // (of c only for scales, so that float32 sums do: 128 squares of rounded differences are off by less than 1e-5; in float64 the
  // differences would stay live)
  float c2 = 0.f, c_elem = 0.f, w_elem = 0.f;
#pragma unroll
  for (int u = 0; u < kD / 4; ++u) {
    const float x = (cv[u] - s_mu[4 * u + k]) * s_t[4 * u + k];
    c2 += x * x;
    c_elem = fmaxf(c_elem, fabsf(x));
  }
  auto centred = [&](int u) { return (double)cv[u] - (double)s_mu[4 * u + k]; };
  // register r of tile t: dimension 16 t + 4 r + k of codeword cg
  f64x4 acc[8];
  auto times = [&](const double* m) {   // acc = (c m)^T, m row-major
    double row[3][8];                   // (two k-steps of the matrix in flight)
    auto request = [&](int u) {
#pragma unroll
      for (int t = 0; t < 8; ++t) row[u % 3][t] = m[(size_t)(4 * u + k) * kD + 16 * t + c];
    };
    request(0);
    request(1);
#pragma unroll
    for (int t = 0; t < 8; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int u = 0; u < kD / 4; ++u) {
      if (u + 2 < kD / 4) request(u + 2);
      __builtin_amdgcn_sched_barrier(0);
      const double b = centred(u);
#pragma unroll
      for (int t = 0; t < 8; ++t) acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(row[u % 3][t], b, acc[t], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto column_sum = [&](double n) {
    n += __shfl_xor(n, 16);
    return n + __shfl_xor(n, 32);
  };
  c2 += __shfl_xor(c2, 16);
  c2 += __shfl_xor(c2, 32);
  double z2 = 0.0, w2 = 0.0;
  if (mode == A2ATS_W_BLOCK) {
    times(hmat + (size_t)kv * kD * kD);
    // (the differences are taken again: kept in float64, they would spill)
#pragma unroll
    for (int u = 0; u < kD / 4; ++u) asm volatile("" : "+v"(cv[u]));
#pragma unroll
    for (int u = 0; u < kD / 4; ++u) z2 += acc[u / 4][u % 4] * centred(u);
  } else {
#pragma unroll
    for (int u = 0; u < kD / 4; ++u) {
      const double s = sd[(size_t)kv * kD + 4 * u + k], z = centred(u) * s;
      z2 += z * z;
      acc[u / 4][u % 4] = z * s;
    }
  }
#pragma unroll
  for (int t = 0; t < 8; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      wT[((size_t)kv * kD + 16 * t + 4 * r + k) * kCW + cg] = acc[t][r];
      const double x = acc[t][r] * (double)inverse_of_power(s_t[16 * t + 4 * r + k]);
      w2 += x * x;
      w_elem = fmaxf(w_elem, fabsf((float)x));
    }
  z2 = column_sum(z2);
  w2 = column_sum(w2);
  if (k == 0) {
    cbias[(size_t)kv * kCW + cg] = (float)(0.5 * z2);
    chalf[(size_t)kv * kCW + cg] = 0.5 * z2;
  }
  // rounded up; a float that is not negative orders like its bits (c . w is negative at times where H, rounded to float32, is
  // singular: its sign bit would stand above every magnitude)
  uint32_t most[5] = {__float_as_uint(__double2float_ru(0.5 * fabs(z2))), __float_as_uint(__double2float_ru(sqrt(w2))),
                      __float_as_uint(1.00001f * sqrtf(c2)), __float_as_uint(w_elem), __float_as_uint(c_elem)};
  __shared__ uint32_t s_most[4][5];
#pragma unroll
  for (int i = 0; i < 5; ++i) {
#pragma unroll
    for (int off = i < 3 ? 8 : 32; off >= 1; off >>= 1) most[i] = max(most[i], (uint32_t)__shfl_xor((int)most[i], off));
    if (lane == 0) s_most[threadIdx.x >> 6][i] = most[i];
  }
  __syncthreads();
  if (threadIdx.x < 5) {   // (one atomic per workgroup: one per wave, all heads in one cache line, took 100 us)
    const int i = threadIdx.x;
    const uint32_t v = max(max(s_most[0][i], s_most[1][i]), max(s_most[2][i], s_most[3][i]));
    CodewordStat* c = cstat + kv;
    atomicMax(i == 0 ? &c->bias_max : i == 1 ? &c->w_max : i == 2 ? &c->c_max : i == 3 ? &c->w_elem : &c->c_elem, v);
  }
}

// ------------------------------------------------------------------------------------------
// The matrix-core operands of 32 codewords, all -w / t (the matrix core then leaves 1/2 |c^z|^2 - k . w).
// Lane (row, g) of k-step kt holds dimensions 16 kt + 8 g .. + 8 of its codeword.
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(512) void encode_single_operands_kernel(const double* __restrict__ wT,
                                                                     Center* __restrict__ center,
                                                                     const float* __restrict__ cbias,
                                                                     uint16_t* __restrict__ cfrag,
                                                                     _Float16* __restrict__ f16,
                                                                     float* __restrict__ fbias, uint8_t* __restrict__ i8,
                                                                     int* __restrict__ bias8,
                                                                     CodewordStat* __restrict__ cstat) {
  __shared__ float s_e[16][32], s_e8[16][32];
  const int kv = blockIdx.y, cb = blockIdx.x, tid = threadIdx.x;
  const int row = tid & 31, kt = tid >> 6, g = (tid >> 5) & 1;
  float key_scale, w_scale;
  const bool ok = f16_scales(cstat[kv], key_scale, w_scale);
  float key_scale8, w_scale8;
  const bool ok8 = i8_scales(cstat[kv], key_scale8, w_scale8);
  if (cb == 0 && tid < kD) {
    center[kv].key[tid] = center[kv].t[tid] * key_scale;
    center[kv].key8[tid] = center[kv].t[tid] * key_scale8;
  }
  bf16x8 hi, lo;
  f16x8 h;
  float err = 0.f, err8 = 0.f;
  uint32_t q8[2] = {0u, 0u};
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int d = 16 * kt + 8 * g + i;
    const double neg = -wT[((size_t)kv * kD + d) * kCW + 32 * cb + row] * (double)inverse_of_power(center[kv].t[d]);
    const uint16_t b = f32_to_bf16((float)neg);
    hi[i] = __builtin_bit_cast(__bf16, b);
    lo[i] = __builtin_bit_cast(__bf16, f32_to_bf16((float)(neg - (double)bf16_to_f32(b))));
    const double x = neg * (double)w_scale;
    h[i] = (_Float16)(float)x;
    const float r = (float)(x - (double)(float)h[i]);
    err += r * r;
    const double x8 = neg * (double)w_scale8, n8 = fmin(fmax(rint(x8), -127.0), 127.0);
    q8[i / 4] |= ((uint32_t)(int)n8 & 255u) << (8 * (i % 4));
    err8 += (float)(x8 - n8) * (float)(x8 - n8);
  }
  uint16_t* blk = cfrag + ((size_t)kv * kBlocks + cb) * (kFragBytes / 2) + (kt * 64 + row + 32 * g) * 8;
  *(bf16x8*)blk = hi;
  *(bf16x8*)(blk + 8 * 64 * 8) = lo;
  *(f16x8*)(f16 + ((size_t)kv * kBlocks + cb) * (kF16Bytes / 2) + (kt * 64 + row + 32 * g) * 8) = h;
  *(uint2*)(i8 + ((size_t)kv * kCW + 32 * cb + row) * kD + 16 * kt + 8 * g) = make_uint2(q8[0], q8[1]);
  s_e[2 * kt + g][row] = err;
  s_e8[2 * kt + g][row] = err8;
  __syncthreads();
  if (tid < 32) {
    float e2 = 0.f, e28 = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      e2 += s_e[i][tid];
      e28 += s_e8[i][tid];
    }
    bias8[(size_t)kv * kCW + 32 * cb + tid] =
        ok8 ? (int)rint((double)cbias[(size_t)kv * kCW + 32 * cb + tid] * (double)(key_scale8 * w_scale8)) : 0;
    uint32_t most8 = __float_as_uint(ok8 ? 1.00001f * sqrtf(e28) : NAN);
#pragma unroll
    for (int off = 16; off >= 1; off >>= 1) most8 = max(most8, (uint32_t)__shfl_xor((int)most8, off));
    if (tid == 0) atomicMax(&cstat[kv].w_err8, most8);
    fbias[(size_t)kv * kCW + 32 * cb + tid] = cbias[(size_t)kv * kCW + 32 * cb + tid] * (key_scale * w_scale);
    uint32_t most = __float_as_uint(ok ? 1.00001f * sqrtf(e2) : NAN);   // NaN: no key is decided by the filter
#pragma unroll
    for (int off = 16; off >= 1; off >>= 1) most = max(most, (uint32_t)__shfl_xor((int)most, off));
    if (tid == 0) atomicMax(&cstat[kv].w_err, most);
  }
}

// ------------------------------------------------------------------------------------------
// z = k L for all rows (seeding), float64 accumulation, one rounding.
// A thread owns one key and 32 consecutive output dimensions; the rows of L it needs are the same
// for the whole wave.
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void encode_single_transform_kernel(
    const float* __restrict__ keys, const double* __restrict__ Lmat, float* __restrict__ z, int Hkv, int n_new) {
  __shared__ float s_k[64][kD + 1];
  const int bkv = blockIdx.y, kv = bkv % Hkv, tid = threadIdx.x;
  const int key = tid & 63, og = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int first = blockIdx.x * 64;
  const float* src = keys + (size_t)bkv * n_new * kD;
  for (int e = tid; e < 64 * (kD / 4); e += 256) {
    const int row = e / (kD / 4), c4 = e % (kD / 4);
    const float4 f = *(const float4*)(src + (size_t)min(first + row, n_new - 1) * kD + 4 * c4);
    s_k[row][4 * c4] = f.x, s_k[row][4 * c4 + 1] = f.y, s_k[row][4 * c4 + 2] = f.z, s_k[row][4 * c4 + 3] = f.w;
  }
  __syncthreads();
  double acc[32];
#pragma unroll
  for (int u = 0; u < 32; ++u) acc[u] = 0.0;
  const double* L = Lmat + (size_t)kv * kD * kD + 32 * og;
  for (int r = 32 * og; r < kD; ++r) {   // L[r][t] = 0 for r < t
    const double kr = (double)s_k[key][r];
#pragma unroll
    for (int u = 0; u < 32; ++u) acc[u] += kr * L[(size_t)r * kD + u];
  }
  if (first + key < n_new) {
    float* dst = z + ((size_t)bkv * n_new + first + key) * kD + 32 * og;
#pragma unroll
    for (int u = 0; u < 32; u += 4)
      *(float4*)(dst + u) = make_float4((float)acc[u], (float)acc[u + 1], (float)acc[u + 2], (float)acc[u + 3]);
  }
}

// ------------------------------------------------------------------------------------------
// The filter
// ------------------------------------------------------------------------------------------
// 32 NT keys per wave (B operands in registers, rounded to f16), 4 waves; the codewords stream through LDS 32 at
// a time as the A operand.  The accumulators start at 1/2 |c^z|^2 and the stored operands are -w, so the matrix
// core leaves the scores.  Ranking has no branch: the codeword's number within the lane goes into the low 11
// mantissa bits, and the two smallest are kept (2.25 vector instructions per score).
//
// With k and w now less the centre and balanced, e_k = |k - f16(k)|, e_w = max |w - f16(w)| and float32 sums, a score is off
// by at most
//   e_k max|w| + |k| e_w + 4e-6 (|k| max|w| + max 1/2 |c^z|^2)
// and by 2^-12 of itself for the number; the two smallest are told apart where they differ by more than that
// counted twice.  Of keys drawn like the codewords (normal, nothing in common with them) 2 % are not.
//
// What bounds it: the matrix cores (one product of f16; three of bf16 for every key before, and a float64 pass z = k L
// over the keys ahead of them): 96001 keys x 8 heads, full matrix: the whole call 687 us (2420 before), 1.2 PFLOP/s at
// 1.8 GHz;
// 16 keys of one head 64 us (193), whatever the matrix.
__device__ __forceinline__ void filter_insert(float a, float b, float c, float d, float& k1, float& k2) {
  // two at a time: the median of (smallest so far, two new) is the only candidate they add for second place
  float m0, m1;
  asm("v_med3_f32 %0, %1, %2, %3" : "=v"(m0) : "v"(k1), "v"(a), "v"(b));
  asm("v_min3_f32 %0, %1, %2, %3" : "=v"(k1) : "v"(k1), "v"(a), "v"(b));
  asm("v_med3_f32 %0, %1, %2, %3" : "=v"(m1) : "v"(k1), "v"(c), "v"(d));
  asm("v_min3_f32 %0, %1, %2, %3" : "=v"(k1) : "v"(k1), "v"(c), "v"(d));
  asm("v_min3_f32 %0, %1, %2, %3" : "=v"(k2) : "v"(k2), "v"(m0), "v"(m1));
}

// ------------------------------------------------------------------------------------------
// The filter in i8: whole numbers of 8 bits, keys and codewords, whose products are exact.  A score is off by at most
//   e_k max|w| + |q_k| e_w + 3/4          (in units of the two scales; q_k the key's numbers, 3/4 for 1/2 |c^z|^2)
// and about 50 times as many keys are left open as by the f16 one where keys have several codewords about equally near (of
// normal keys nearly all), but hardly any where they lie close to one: so some keys of the call say which filter a KV head
// takes (encode_single_sample_kernel).  The smallest of four scores goes on, with the number of the four in the 9 bits below
// it; the four are multiplied again at the end, which gives the same whole numbers.
//
// A product takes half the time and power of the f16 one, the ranking 17 vector instructions a tile instead of 36.  96001 keys
// x 8 heads, full matrix, codewords prepared: 707 -> 377 us (the products at 3.0 POP/s while they run, which is what this chip's
// power leaves of 5; reading and rounding keys, and the four, a quarter of the time).  With 2 % of the keys open both filters, with
// their lists, take the same time at 3 to 6 % (0.02: 872 -> 671 us, 0.06: 879 -> 848); kSampleOpen is below that.
// Tried: eight scores ranked together (13 instructions) and multiplied again 393; a wave of 32 NT keys with NT = 3 and its next
// keys read and rounded during the products 418.
// ------------------------------------------------------------------------------------------
// A lane's 64 dimensions of a key (16 g + 32 kt .. + 16), |k - q|^2 and |q|^2 over them.
__device__ __forceinline__ void quantise_key(const float* kp, const float* s_mu, const float* s_key, int g, i32x4 (&q)[4],
                                             float& e2, int& n2) {
#pragma unroll
  for (int kt = 0; kt < 4; ++kt) {
    float4 f[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) f[u] = *(const float4*)(kp + 32 * kt + 4 * u);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int d = 32 * kt + 16 * g + 4 * u;
      const float4 mu = *(const float4*)&s_mu[d], sc = *(const float4*)&s_key[d];
      const float v[4] = {(f[u].x - mu.x) * sc.x, (f[u].y - mu.y) * sc.y, (f[u].z - mu.z) * sc.z, (f[u].w - mu.w) * sc.w};
      uint32_t b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        constexpr float kRound = 12582912.f;   // 1.5 * 2^23: the sum's last bits are the whole number
        const float r = __builtin_amdgcn_fmed3f(v[i], -127.f, 127.f) + kRound, e = v[i] - (r - kRound);
        e2 += e * e;
        b[i] = __float_as_uint(r);
      }
      const uint32_t lo = __builtin_amdgcn_perm(b[1], b[0], 0x0c0c0400), hi = __builtin_amdgcn_perm(b[3], b[2], 0x0c0c0400);
      q[kt][u] = (int)(lo | hi << 16);
      n2 = __builtin_amdgcn_sdot4(q[kt][u], q[kt][u], n2, false);
    }
  }
}

// By how much two scores may be off together.
__device__ __forceinline__ float reach8(const CodewordStat& st, float key_scale, float w_scale, float e2, float n2) {
  const float w_max = __uint_as_float(st.w_max) * w_scale, w_err = __uint_as_float(st.w_err8), kn = sqrtf(n2), ke = sqrtf(e2);
  return 2.f * (1.00001f * (ke * w_max + kn * w_err) +
                4e-6f * ((kn + ke) * w_max + __uint_as_float(st.bias_max) * (key_scale * w_scale)) + 1.f);
}

__device__ __forceinline__ void insert8(int a, int b, int& k1, int& k2) {
  int m;
  asm("v_med3_i32 %0, %1, %2, %3" : "=v"(m) : "v"(k1), "v"(a), "v"(b));
  asm("v_min3_i32 %0, %1, %2, %3" : "=v"(k1) : "v"(k1), "v"(a), "v"(b));
  k2 = min(k2, m);
}

// Keys of a KV head, 128 a workgroup, against a slice of its codewords: the two smallest scores, each with its number in the slice
// in the 9 bits below it.  (And no counts yet.)  ALL: all `n_rows` keys, else 128 of them, evenly spread.
template <bool ALL>
__global__ __launch_bounds__(kEncThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void encode_single_sample_kernel(
    const float* __restrict__ keys, const Center* __restrict__ center, const uint8_t* __restrict__ i8,
    const int* __restrict__ bias8, int2* __restrict__ sample, float2* __restrict__ norms, uint32_t* __restrict__ counter,
    int n_counter, uint32_t* __restrict__ found, int n_new, long n_rows) {
  static_assert(kSampleKeys == 32 * kEncWaves, "a wave takes 32 keys");
  constexpr int kOwn = kBlocks / kSampleSlices;
  static_assert(32 * kOwn <= 512, "a number has 9 bits");
  __shared__ __align__(32) float s_mu[kD], s_key[kD];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, col = lane & 31, g = lane >> 5;
  const int slice = blockIdx.x, kv = blockIdx.y, Hkv = gridDim.y, at = blockIdx.z * kSampleKeys + wave * 32 + col;
  for (int i = (kv * kSampleSlices + slice) * kEncThreads + tid; i < n_counter; i += Hkv * kSampleSlices * kEncThreads) counter[i] = 0;
  if (slice == 0 && tid == 0) found[kv * kFoundStride] = 0;
  if (tid < kD) {
    s_mu[tid] = center[kv].mu[tid];
    s_key[tid] = center[kv].key8[tid];
  }
  const uint8_t* blk = i8 + ((size_t)kv * kBlocks + slice * kOwn) * kI8Bytes + col * kD + 16 * g;
  const int* bias = bias8 + (size_t)kv * kCW + slice * kOwn * 32 + 4 * g;
  i32x4 a[kOwn][4];
#pragma unroll
  for (int i = 0; i < kOwn; ++i)
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) a[i][kt] = *(const i32x4*)(blk + i * kI8Bytes + 32 * kt);
  __syncthreads();
  const uint32_t row = (uint32_t)(ALL ? min((long)at, n_rows - 1) : (2 * at + 1) * n_rows / (2 * kSampleKeys));
  const uint32_t seq = row / (uint32_t)n_new;   // (sequence by sequence)
  const float* kp = keys + (((size_t)seq * Hkv + kv) * n_new + (row - seq * (uint32_t)n_new)) * kD + 16 * g;
  i32x4 q[4];
  float e2 = 0.f;
  int n2 = 0, k1 = 0x7fffffff, k2 = 0x7fffffff;
  quantise_key(kp, s_mu, s_key, g, q, e2, n2);
#pragma unroll
  for (int i = 0; i < kOwn; ++i) {
    i32x16 acc;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int4 b = *(const int4*)(bias + i * 32 + 8 * v);
      acc[4 * v] = b.x, acc[4 * v + 1] = b.y, acc[4 * v + 2] = b.z, acc[4 * v + 3] = b.w;
    }
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[i][kt], q[kt], acc, 0, 0, 0);
    // register v: codeword 32 i + 8 (v / 4) + 4 g + v % 4 of the slice, number 32 i + 2 v + g
    auto numbered = [&](int v) { return (int)((uint32_t)acc[v] << 9 | (uint32_t)(32 * i + 2 * v)); };
#pragma unroll
    for (int v = 0; v < 16; v += 2) insert8(numbered(v), numbered(v + 1), k1, k2);
  }
  k1 |= g;
  k2 |= g;
  const int o1 = __shfl_xor(k1, 32), o2 = __shfl_xor(k2, 32);
  e2 += __shfl_xor(e2, 32);
  n2 += __shfl_xor(n2, 32);
  if (g == 0) {
    sample[((size_t)kv * kSampleSlices + slice) * (gridDim.z * kSampleKeys) + at] =
        make_int2(min(k1, o1), min(max(k1, o1), min(k2, o2)));
    if (slice == 0 && (!ALL || at < n_rows)) norms[(size_t)kv * (ALL ? n_rows : kSampleKeys) + at] = make_float2(e2, (float)n2);
  }
}

// The two smallest scores of key `at` over all slices, the smaller one's number and slice; two threads take a key, each half of the
// slices, and the first of them returns true.  (Of equal scores the one or the other: they leave the key open.)
struct SampleBest {
  int k1, k2, slice;
};
__device__ __forceinline__ bool best_of_slices(const int2* __restrict__ sample, int at, int stride, SampleBest& best,
                                               SampleBest (&s_half)[kSampleKeys]) {
  static_assert(kEncThreads == 2 * kSampleKeys, "two threads a key");
  const int half = threadIdx.x / kSampleKeys, first = half * (kSampleSlices / 2);
  int2 s[kSampleSlices / 2];
#pragma unroll
  for (int i = 0; i < kSampleSlices / 2; ++i) s[i] = sample[(size_t)(first + i) * stride + at];
  best = SampleBest{0x7fffffff, 0x7fffffff, 0};
  auto take = [&](int k1, int k2, int slice) {
    best.k2 = min(max(best.k1, k1), min(best.k2, k2));
    best.slice = k1 < best.k1 ? slice : best.slice;
    best.k1 = min(best.k1, k1);
  };
#pragma unroll
  for (int i = 0; i < kSampleSlices / 2; ++i) take(s[i].x, s[i].y, first + i);
  if (half == 1) s_half[threadIdx.x % kSampleKeys] = best;
  __syncthreads();
  if (half == 1) return false;
  const SampleBest o = s_half[threadIdx.x];
  take(o.k1, o.k2, o.slice);
  return true;
}
__device__ __forceinline__ bool leaves_open(const CodewordStat& st, const SampleBest& best, float2 norms) {
  float key_scale, w_scale;
  i8_scales(st, key_scale, w_scale);
  return !((float)((best.k2 >> 9) - (best.k1 >> 9)) > reach8(st, key_scale, w_scale, norms.x, norms.y));   // (also where anything is not a number)
}

// Whether a KV head takes the i8 filter: every workgroup of the filter finds it from the sample (which costs less than a launch of
// its own, or the fences with which the last workgroup of the sample could say it, 19 us).
__device__ __forceinline__ bool takes_filter8(const CodewordStat* cstat, const int2* __restrict__ sample,
                                              const float2* __restrict__ norms, int kv, SampleBest (&s_half)[kSampleKeys]) {
  const int at = threadIdx.x % kSampleKeys;
  const float2 n = norms[(size_t)kv * kSampleKeys + at];
  SampleBest best;
  bool open = false;
  if (best_of_slices(sample + (size_t)kv * kSampleSlices * kSampleKeys, at, kSampleKeys, best, s_half))
    open = leaves_open(cstat[kv], best, n);
  return __syncthreads_count(open) <= kSampleOpen;
}

// The keys of a call that are so few that a "sample" has them all: decided or listed.
__global__ __launch_bounds__(kEncThreads) void encode_single_decide_kernel(
    const CodewordStat* __restrict__ cstat, const int2* __restrict__ sample, const float2* __restrict__ norms,
    uint16_t* __restrict__ codes, uint32_t* __restrict__ near_count, uint32_t* __restrict__ near, int64_t near_cap, int n_new,
    long n_rows, int pos0, int64_t ctx_stride) {
  __shared__ SampleBest s_half[kSampleKeys];
  const int kv = blockIdx.y, Hkv = gridDim.y, at = blockIdx.x * kSampleKeys + threadIdx.x % kSampleKeys;
  const int stride = gridDim.x * kSampleKeys;
  SampleBest best;
  if (!best_of_slices(sample + (size_t)kv * kSampleSlices * stride, at, stride, best, s_half) || at >= n_rows) return;
  const int number = best.k1 & 511, v = (number >> 1) & 15;
  const int code = best.slice * (kCW / kSampleSlices) + (number >> 5) * 32 + (v >> 2) * 8 + (number & 1) * 4 + (v & 3);
  const int seq = at / n_new;
  codes[((size_t)seq * Hkv + kv) * ctx_stride + pos0 + (at - seq * n_new)] = (uint16_t)code;
  if (leaves_open(cstat[kv], best, norms[(size_t)kv * n_rows + at])) {
    const uint32_t place = atomicAdd(near_count + kv, 1u);
    near[(size_t)kv * near_cap + place] = (uint32_t)at;
  }
}

constexpr int kFilterWaves[2][5] = {{0, 2, 2, 0, 2}, {0, 4, 3, 0, 2}};   // per SIMD, of 32 NT keys each, without and with the i8 filter
constexpr int kSect = 512 + 16;   // 16 bytes of 32 codewords; a codeword's eight on different banks
constexpr int kBlk8 = 8 * kSect + 128, kBuf8 = 2 * kBlk8, kBuf16 = kF16Bytes + 128;
template <int NT>
struct FilterLds {
  __align__(16) uint8_t mem[2 * (kBuf8 > kBuf16 ? kBuf8 : kBuf16)];
  float n2[NT][kEncThreads], e2[NT][kEncThreads];   // (kept out of the registers for the main loop)
  __align__(32) float mu[kD], key[2][kD];           // (of the f16 and of the i8 operands)
  SampleBest half[kSampleKeys];
};

template <int NT>
__device__ __forceinline__ void filter8_body(
    FilterLds<NT>& lds, const float* __restrict__ keys, const uint8_t* __restrict__ i8, const int* __restrict__ bias8,
    const CodewordStat* __restrict__ cstat, uint16_t* __restrict__ codes, uint32_t* __restrict__ near_count, uint32_t* __restrict__ near, int64_t near_cap, int Hkv,
    int n_new, int pos0, int64_t ctx_stride) {
  // The codewords go through LDS two blocks at a time (with one the loads are not back when they are wanted).
  constexpr int kBlk = kBlk8, kBuf = kBuf8;
  static_assert(kI8Bytes / 16 == kEncThreads, "a thread stages 16 bytes of a block");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, col = lane & 31, g = lane >> 5;
  const int bkv = blockIdx.y, kv = bkv % Hkv, seq = bkv / Hkv;
  const long key_first = ((long)blockIdx.x * kEncWaves + wave) * (32 * NT);
  const CodewordStat st = cstat[kv];
  auto &s_n2 = lds.n2, &s_e2 = lds.e2;
  auto &s_mu = lds.mu, &s_key = lds.key[1];
  uint8_t* s_mem = lds.mem;
  const float* seq_keys = keys + (size_t)bkv * n_new * kD;
  i32x4 kq[NT][4];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    float e2 = 0.f;
    int n2 = 0;
    quantise_key(seq_keys + (size_t)min(key_first + 32 * t + col, (long)n_new - 1) * kD + 16 * g, s_mu, s_key, g, kq[t], e2, n2);
    s_n2[t][tid] = (float)n2;
    s_e2[t][tid] = e2;
    __builtin_amdgcn_sched_barrier(0);
  }

  const uint8_t* all = i8 + (size_t)kv * kBlocks * kI8Bytes;
  const uint8_t* gblk = all + tid * 16;
  const int* gbias = bias8 + (size_t)kv * kCW + (tid & 63);
  uint4 p0, p1;
  int pb;
  auto request = [&](int step) {
    step = min(step, kBlocks / 2 - 1);   // the last step loads its blocks once more, unused
    p0 = *(const uint4*)(gblk + (size_t)step * (2 * kI8Bytes));
    p1 = *(const uint4*)(gblk + (size_t)step * (2 * kI8Bytes) + kI8Bytes);
    pb = gbias[step * 64];
  };
  auto stage = [&](int step) {
    uint8_t* dst = s_mem + (step & 1) * kBuf;
    *(uint4*)(dst + (tid & 7) * kSect + (tid >> 3) * 16) = p0;   // (piece tid % 8 of codeword tid / 8)
    *(uint4*)(dst + kBlk + (tid & 7) * kSect + (tid >> 3) * 16) = p1;
    *(int*)(dst + ((tid >> 5) & 1) * kBlk + 8 * kSect + (tid & 31) * 4) = pb;   // several threads write each word, all the same
  };
  int k1[NT], k2[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) k1[t] = k2[t] = 0x7fffffff;
  i32x4 a[4];
  i32x16 bias;
  auto read_bias = [&](int cb) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int4 f = *(const int4*)(s_mem + (cb & 3) * kBlk + 8 * kSect + (8 * q + 4 * g) * 4);
      bias[4 * q] = f.x, bias[4 * q + 1] = f.y, bias[4 * q + 2] = f.z, bias[4 * q + 3] = f.w;
    }
  };
  auto operand = [&](int cb, int kt) { return *(const i32x4*)(s_mem + (cb & 3) * kBlk + (2 * kt + g) * kSect + col * 16); };
  // registers 4 q .. + 4 of a tile: codewords 32 cb + 8 q + 4 g .. + 4, number 4 cb + q
  auto least_of = [&](const i32x16& acc, int q, int cb) {
    uint32_t number = (uint32_t)(4 * cb + q);
    asm("" : "+s"(number));   // (a scalar of its own, or it is put together on the vector ALU)
    return (int)((uint32_t)min(min(acc[4 * q], acc[4 * q + 1]), min(acc[4 * q + 2], acc[4 * q + 3])) << 9 | number);
  };
  request(0);
  stage(0);
  request(1);
  __syncthreads();
  read_bias(0);
#pragma unroll
  for (int kt = 0; kt < 4; ++kt) a[kt] = operand(0, kt);
  // (products and the ranking of the tile before in turns, as in the f16 filter)
  i32x16 acc[2];
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[1][v] = 0x3fffff;   // (ranked before the first tile: above any score)
#pragma unroll 1
  for (int step = 0; step < kBlocks / 2; ++step) {
#pragma unroll
    for (int tile = 0; tile < 2 * NT; ++tile) {
      const int t = tile % NT, cb = 2 * step + tile / NT;
      i32x16& now = acc[tile & 1];
      const i32x16& done = acc[(tile + 1) & 1];
      const int prev = (t + NT - 1) % NT, prev_cb = t == 0 ? max(cb - 1, 0) : cb;
      int m0 = 0;
#pragma unroll
      for (int kt = 0; kt < 4; ++kt) {
        now = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[kt], kq[t][kt], kt == 0 ? bias : now, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (kt == 1 || kt == 2) {
          const int la = least_of(done, 2 * kt - 2, prev_cb), lb = least_of(done, 2 * kt - 1, prev_cb);
          int m;
          asm("v_med3_i32 %0, %1, %2, %3" : "=v"(m) : "v"(k1[prev]), "v"(la), "v"(lb));
          asm("v_min3_i32 %0, %1, %2, %3" : "=v"(k1[prev]) : "v"(k1[prev]), "v"(la), "v"(lb));
          if (kt == 1) m0 = m;
          else k2[prev] = min(min(k2[prev], m0), m);
        }
        if (t == NT - 1) {   // the next block's operand, each part once the last tile has taken it
          a[kt] = operand(cb + 1, kt);
          if (kt == 0) {
            asm volatile("" ::"v"(bias));   // (or the sums take the place of the bias, and both are moved about)
            read_bias(cb + 1);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (tile == 3 * NT / 2 - 1) {
        stage(step + 1);   // (its buffer was last read before the barrier of the step before)
        request(step + 2);
        __syncthreads();
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 4; i += 2)
    insert8(least_of(acc[1], i, kBlocks - 1), least_of(acc[1], i + 1, kBlocks - 1), k1[NT - 1], k2[NT - 1]);

  // The two lane halves of a key column hold disjoint codewords; both multiply the four of the smaller one again, over their
  // dimensions.
  float key_scale, w_scale;
  i8_scales(st, key_scale, w_scale);
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int o1 = __shfl_xor(k1[t], 32), o2 = __shfl_xor(k2[t], 32);
    const bool own = k1[t] < o1 || (k1[t] == o1 && g == 0);
    const int m1 = own ? k1[t] : o1, other = min(max(k1[t], o1), min(k2[t], o2)) >> 9;
    const int c0 = ((m1 & 511) >> 2) * 32 + (m1 & 3) * 8 + (own ? g : 1 - g) * 4;   // the first of the four
    const uint8_t* src = all + (size_t)c0 * kD + 16 * g;
    i32x4 w[4][4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int kt = 0; kt < 4; ++kt) w[r][kt] = *(const i32x4*)(src + r * kD + 32 * kt);
    const int4 b = *(const int4*)(bias8 + (size_t)kv * kCW + c0);
    const int half[4] = {b.x, b.y, b.z, b.w};
    int best = 0x7fffffff, second = 0x7fffffff, code = c0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      int dot = 0;
#pragma unroll
      for (int kt = 0; kt < 4; ++kt)
#pragma unroll
        for (int i = 0; i < 4; ++i) dot = __builtin_amdgcn_sdot4(kq[t][kt][i], w[r][kt][i], dot, false);
      const int score = half[r] + dot + __shfl_xor(dot, 32);
      second = min(second, max(best, score));
      code = score < best ? c0 + r : code;
      best = min(best, score);
    }
    second = min(second, other);
    const float reach = reach8(st, key_scale, w_scale, s_e2[t][tid] + s_e2[t][tid ^ 32], s_n2[t][tid] + s_n2[t][tid ^ 32]);
    const long j = key_first + 32 * t + col;
    if (g == 0 && j < n_new) {
      codes[(size_t)bkv * ctx_stride + pos0 + j] = (uint16_t)code;
      if (!((float)(second - best) > reach)) {   // (also where anything is not a number)
        const uint32_t place = atomicAdd(near_count + kv, 1u);
        near[(size_t)kv * near_cap + place] = (uint32_t)((size_t)seq * n_new + j);
      }
    }
  }
}

template <int NT>
__device__ __forceinline__ void filter16_body(
    FilterLds<NT>& lds, const float* __restrict__ keys, const uint8_t* __restrict__ f16, const float* __restrict__ fbias,
    const CodewordStat* __restrict__ cstat, uint16_t* __restrict__ codes,
    uint32_t* __restrict__ near_count, uint32_t* __restrict__ near, int64_t near_cap, int Hkv, int n_new, int pos0,
    int64_t ctx_stride) {
  constexpr int kBuf = kBuf16, kPieces = kF16Bytes / 16 / kEncThreads;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, col = lane & 31, g = lane >> 5;
  const int bkv = blockIdx.y, kv = bkv % Hkv, seq = bkv / Hkv;
  const long key_first = ((long)blockIdx.x * kEncWaves + wave) * (32 * NT);
  const float* seq_keys = keys + (size_t)bkv * n_new * kD;
  const CodewordStat st = cstat[kv];
  auto &s_n2 = lds.n2, &s_e2 = lds.e2;
  auto &s_mu = lds.mu, &s_key = lds.key[0];
  uint8_t* s_mem = lds.mem;
  float key_scale, w_scale;
  f16_scales(st, key_scale, w_scale);
  f16x8 kh[NT][8];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const float* kp = seq_keys + (size_t)min(key_first + 32 * t + col, (long)n_new - 1) * kD + 8 * g;
    float n2 = 0.f, e2 = 0.f;
#pragma unroll
    for (int k4 = 0; k4 < 8; k4 += 4) {   // four k-steps of loads in flight at a time
      float4 lo[4], hi[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        lo[u] = *(const float4*)(kp + 16 * (k4 + u));
        hi[u] = *(const float4*)(kp + 16 * (k4 + u) + 4);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        typedef __attribute__((ext_vector_type(8))) float f32x8;
        const f32x8 x = {lo[u].x, lo[u].y, lo[u].z, lo[u].w, hi[u].x, hi[u].y, hi[u].z, hi[u].w};
        const int d = 16 * (k4 + u) + 8 * g;
        const f32x8 v = (x - *(const f32x8*)&s_mu[d]) * *(const f32x8*)&s_key[d];
        kh[t][k4 + u] = __builtin_convertvector(v, f16x8);
        const f32x8 r = v - __builtin_convertvector(kh[t][k4 + u], f32x8);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          n2 += v[i] * v[i];
          e2 += r[i] * r[i];
        }
        asm volatile("" : "+v"(kh[t][k4 + u]), "+v"(n2), "+v"(e2));   // (in this order: else all of v and r stay live)
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    s_n2[t][tid] = n2;
    s_e2[t][tid] = e2;
  }

  const uint8_t* gblk = f16 + (size_t)kv * kBlocks * kF16Bytes + tid * 16;
  const float* gbias = fbias + (size_t)kv * kCW + (tid & 31);
  static_assert(kPieces == 2, "a thread stages two 16-byte pieces of a block");
  // A block is requested as soon as the one before is staged, where there are registers for that (otherwise at the top of its
  // step, which with one tile is too late: 1100 normal keys x 8 heads 188 -> 173 us).
  constexpr bool kEarly = NT <= 2;
  uint4 p0, p1;
  float pb;
  auto request = [&](int cb) {
    cb = min(cb, kBlocks - 1);   // the step of the last block loads it once more, unused
    p0 = *(const uint4*)(gblk + (size_t)cb * kF16Bytes);
    p1 = *(const uint4*)(gblk + (size_t)cb * kF16Bytes + kEncThreads * 16);
    pb = gbias[cb * 32];
  };
  auto stage = [&](int cb) {
    uint8_t* dst = s_mem + (cb & 1) * kBuf;
    *(uint4*)(dst + tid * 16) = p0;
    *(uint4*)(dst + (kEncThreads + tid) * 16) = p1;
    *(float*)(dst + kF16Bytes + (tid & 31) * 4) = pb;   // several threads write each word, all the same
  };
  float k1[NT], k2[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) k1[t] = k2[t] = INFINITY;
  uint32_t keep = ~2047u;
  asm("" : "+v"(keep));   // (a vector register: an instruction takes one scalar, and that is the number)
  // register v of a tile: codeword 32 cb + 8 (v/4) + 4 g + v%4, number 16 cb + v
  auto keys_of = [&](const f32x16& acc, int v, int cb, float (&key)[4]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      uint32_t number = (uint32_t)(cb * 16 + v + u);
      asm("" : "+s"(number));   // (a scalar of its own, or it is added up again on the vector ALU)
      key[u] = __uint_as_float((__float_as_uint(acc[v + u]) & keep) | number);
    }
  };
  f16x8 a[8];   // the operand of the block, all k-steps
  f32x16 bias;
  auto read_bias = [&](int cb) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 f = *(const float4*)(s_mem + (cb & 1) * kBuf + kF16Bytes + (8 * q + 4 * g) * 4);
      bias[4 * q] = f.x, bias[4 * q + 1] = f.y, bias[4 * q + 2] = f.z, bias[4 * q + 3] = f.w;
    }
  };
  auto operand = [&](int cb, int kt) { return *(const f16x8*)(s_mem + (cb & 1) * kBuf + kt * 1024 + lane * 16); };
  request(0);
  stage(0);
  if (kEarly) request(1);
  __syncthreads();
  read_bias(0);
#pragma unroll
  for (int kt = 0; kt < 8; ++kt) a[kt] = operand(0, kt);
  // A tile's eight products are issued with the ranking of the tile before between them (the fences keep that order):
  // a wave that first multiplies and then ranks does not overlap with its neighbour on the SIMD, which falls into the
  // same step (742 us instead of 697 for 768032 keys).
  f32x16 acc[2];
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[1][v] = 3e38f;   // (ranked before the first tile, as numbers of block 0: above any score)
#pragma unroll 1
  for (int cb = 0; cb < kBlocks; ++cb) {
    if (!kEarly) request(cb + 1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      constexpr int kOne = NT == 1 ? 0 : 1;   // (a single tile is ranked after its own products)
      f32x16& now = acc[kOne * (t & 1)];
      const f32x16& done = acc[kOne * ((t + 1) & 1)];
      const int prev = (t + NT - 1) % NT, prev_cb = t == 0 && NT > 1 ? max(cb - 1, 0) : cb;
      float key[4];
#pragma unroll
      for (int kt = 0; kt < 8; ++kt) {
        now = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[kt], kh[t][kt], kt == 0 ? bias : now, 0, 0, 0);
        if (NT > 1) {
          if (kt % 2 == 0) keys_of(done, 2 * kt, prev_cb, key);
          else filter_insert(key[0], key[1], key[2], key[3], k1[prev], k2[prev]);
          if (t == NT - 1) {   // the next block's operand, each part once the last tile has taken it
            a[kt] = operand(cb + 1, kt);
            if (kt == 0) read_bias(cb + 1);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (t == (NT - 1) / 2) {
        if (NT == 1) {
#pragma unroll
          for (int v = 0; v < 16; v += 4) {
            keys_of(now, v, cb, key);
            filter_insert(key[0], key[1], key[2], key[3], k1[0], k2[0]);
          }
        }
        stage(cb + 1);   // (its buffer was last read before the barrier of block cb - 1)
        if (kEarly) request(cb + 2);
        __syncthreads();
        if (NT == 1) {
          read_bias(cb + 1);
#pragma unroll
          for (int kt = 0; kt < 8; ++kt) a[kt] = operand(cb + 1, kt);
        }
      }
    }
  }
  if (NT > 1) {
#pragma unroll
    for (int v = 0; v < 16; v += 4) {
      float key[4];
      keys_of(acc[1], v, kBlocks - 1, key);
      filter_insert(key[0], key[1], key[2], key[3], k1[NT - 1], k2[NT - 1]);
    }
  }

  // The two lane halves of a key column hold disjoint codewords.
  const float w_max = __uint_as_float(st.w_max) * w_scale, w_err = __uint_as_float(st.w_err);
  const float bias_max = __uint_as_float(st.bias_max) * (key_scale * w_scale);
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const float o1 = __shfl_xor(k1[t], 32), o2 = __shfl_xor(k2[t], 32);
    const float kn = sqrtf(s_n2[t][tid] + s_n2[t][tid ^ 32]), ke = sqrtf(s_e2[t][tid] + s_e2[t][tid ^ 32]);   // (of this wave)
    const bool own = k1[t] <= o1;
    const float m1 = own ? k1[t] : o1, m2 = fminf(fmaxf(k1[t], o1), fminf(k2[t], o2));
    const uint32_t number = __float_as_uint(m1) & 2047u;
    const uint32_t code = (number >> 4) * 32 + ((number >> 2) & 3) * 8 + (own ? g : 1 - g) * 4 + (number & 3);
    const long j = key_first + 32 * t + col;
    if (g == 0 && j < n_new) {
      const float reach = 2.f * (1.00001f * (ke * w_max + kn * w_err) + 4e-6f * (kn * w_max + bias_max)) +
                          2.5e-4f * (fabsf(m1) + fabsf(m2));
      codes[(size_t)bkv * ctx_stride + pos0 + j] = (uint16_t)code;
      if (!(m2 - m1 > reach)) {   // (also where anything is not a number)
        const uint32_t at = atomicAdd(near_count + kv, 1u);
        near[(size_t)kv * near_cap + at] = (uint32_t)((size_t)seq * n_new + j);
      }
    }
  }
}

// I8, F16: the filters that the launch has.  Without the first, an earlier one has left its choice in `eight`.
template <int NT, bool I8, bool F16>
__global__ __launch_bounds__(kEncThreads) __attribute__((amdgpu_waves_per_eu(kFilterWaves[I8][NT], kFilterWaves[I8][NT]))) void encode_single_filter_kernel(
    const float* __restrict__ keys, const Center* __restrict__ center, const uint8_t* __restrict__ f16,
    const float* __restrict__ fbias, const uint8_t* __restrict__ i8, const int* __restrict__ bias8,
    const int2* __restrict__ sample, const float2* __restrict__ norms, uint32_t* __restrict__ eight,
    const CodewordStat* __restrict__ cstat, uint16_t* __restrict__ codes, uint32_t* __restrict__ near_count,
    uint32_t* __restrict__ near, int64_t near_cap, int Hkv, int n_new, int pos0, int64_t ctx_stride) {
  __shared__ FilterLds<NT> lds;
  const int kv = blockIdx.y % Hkv, tid = threadIdx.x;
  if (!I8 && eight[kv]) return;   // (uniform)
  if (tid < kD) {
    lds.mu[tid] = center[kv].mu[tid];
    lds.key[0][tid] = center[kv].key[tid];
    lds.key[1][tid] = center[kv].key8[tid];
  }
  bool eighth = false;
  if (I8) {   // (has barriers)
    eighth = takes_filter8(cstat, sample, norms, kv, lds.half);
    if (blockIdx.x == 0 && (int)blockIdx.y < Hkv && tid == 0) eight[kv] = eighth ? 1u : 0u;
  } else {
    __syncthreads();
  }
  if (I8 && eighth)   // (uniform)
    filter8_body<NT>(lds, keys, i8, bias8, cstat, codes, near_count, near, near_cap, Hkv, n_new, pos0, ctx_stride);
  else if (F16)
    filter16_body<NT>(lds, keys, f16, fbias, cstat, codes, near_count, near, near_cap, Hkv, n_new, pos0, ctx_stride);
}

// ------------------------------------------------------------------------------------------
// The keys the filter left open
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ void split8(const float (&z)[8], bf16x8& hi, bf16x8& lo, float& n2) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
#pragma unroll
  for (int i = 0; i < 8; i += 2) {   // two at a time: one packed conversion each for hi and lo
    const f32x2 v = {z[i], z[i + 1]};
    const bf16x2 h = __builtin_convertvector(v, bf16x2);
    const f32x2 back = __builtin_convertvector(h, f32x2);
    const bf16x2 l = __builtin_convertvector(v - back, bf16x2);
    hi[i] = h.x, hi[i + 1] = h.y;
    lo[i] = l.x, lo[i + 1] = l.y;
    n2 += z[i] * z[i] + z[i + 1] * z[i + 1];   // (the norm only scales the rounding reach)
  }
}

// Insert score s (code `c`, wave-uniform) into the running smallest three s1 <= s2 <= s3 of a lane.
__device__ __forceinline__ void top3_insert(float s, int c, float& s1, float& s2, float& s3, int& c1, int& c2) {
  s3 = __builtin_amdgcn_fmed3f(s2, s3, s);
  c2 = s < s2 ? c : c2;
  c2 = s < s1 ? c1 : c2;
  s2 = __builtin_amdgcn_fmed3f(s1, s2, s);
  c1 = s < s1 ? c : c1;
  s1 = fminf(s1, s);
}

__global__ __launch_bounds__(kEncThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void encode_single_kernel(
    const float* __restrict__ keys, const Center* __restrict__ center, const uint8_t* __restrict__ cfrag,
    const float* __restrict__ cbias, const CodewordStat* __restrict__ cstat, uint16_t* __restrict__ codes,
    const uint32_t* __restrict__ near_count, const uint32_t* __restrict__ near, int64_t near_cap,
    uint32_t* __restrict__ found, uint32_t* __restrict__ list, uint32_t* __restrict__ arrived, NearPart* parts, int Hkv,
    int n_new, int pos0, int64_t ctx_stride) {
  __shared__ __align__(16) uint8_t s_mem[2 * (kFragBytes + 128)];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, col = lane & 31, g = lane >> 5;
  const int kv = blockIdx.y;
  const long n_near = (long)near_count[kv];
  __shared__ uint32_t s_last;
  __shared__ float s_mu[kD], s_t[kD];
  if (n_near == 0) return;   // (uniform)
  if (tid < kD) {
    s_mu[tid] = center[kv].mu[tid];
    s_t[tid] = center[kv].t[tid];
  }
  __syncthreads();
  // A short list is spread over the workgroups by slices of the codewords too (a multiple of two blocks each): one
  // workgroup takes 165 us for all of them (2000 normal keys x 8 heads: 285 -> 143 us).
  const long n_chunks = (n_near + kKeysPerWG - 1) / kKeysPerWG;
  int slices = 1;
  while (slices < kMaxSlices && n_chunks * slices * 2 <= (long)gridDim.x) slices *= 2;
#pragma unroll 1
  for (long item = blockIdx.x; item < n_chunks * slices; item += gridDim.x) {
    const long chunk = item / slices, base = chunk * kKeysPerWG;
    const int cb0 = (int)(item % slices) * (kBlocks / slices), cb1 = cb0 + kBlocks / slices;
    const long key_first = base + wave * kKeysPerWave;
    auto row_of = [&](int tile) {   // of the listed key: its row in `keys`
      const uint32_t e = near[(size_t)kv * near_cap + min(key_first + 32 * tile + col, n_near - 1)];
      return ((size_t)(e / (uint32_t)n_new) * Hkv + kv) * n_new + e % (uint32_t)n_new;
    };

    bf16x8 zh[2][8], zl[2][8];
    float zn2[2] = {0.f, 0.f};
    {
      // (four k-steps of loads in flight at a time: with all sixteen the registers they land in
      // and the 128 the operands need do not fit, and the spills cost far more than the latency)
#pragma unroll
      for (int tile = 0; tile < 2; ++tile) {
        const float* kp = keys + row_of(tile) * kD + 8 * g;
#pragma unroll
        for (int k4 = 0; k4 < 8; k4 += 4) {
          float4 a[4], b[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            a[u] = *(const float4*)(kp + 16 * (k4 + u));
            b[u] = *(const float4*)(kp + 16 * (k4 + u) + 4);
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            float x[8] = {a[u].x, a[u].y, a[u].z, a[u].w, b[u].x, b[u].y, b[u].z, b[u].w};
            const int d = 16 * (k4 + u) + 8 * g;
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = (x[i] - s_mu[d + i]) * s_t[d + i];
            split8(x, zh[tile][k4 + u], zl[tile][k4 + u], zn2[tile]);
            asm volatile("" : "+v"(zn2[tile]));   // (now: else x is kept, in scratch memory, and summed up after the main loop)
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }

    // Main loop: blocks of 32 codewords (operands + their 1/2 |c^z|^2) through a double buffer in
    // LDS.  The accumulators start at 1/2 |c^z|^2 and the stored operands are -w, so the matrix
    // core leaves the score itself.  Ranking: a score only matters if it is below the lane's third
    // smallest so far, which after the first blocks is rare, so four scores at a time are tested by
    // their minimum and the insertion is skipped by the whole wave when no lane needs it.  (The
    // vector ALU issues one instruction per four cycles per SIMD and a product takes 32: ten
    // instructions per score would cost more than the products.)  Two workgroups share a CU, one wave
    // of each per SIMD, so one computes while the other waits at its barrier.
    const uint8_t* gblk = cfrag + (size_t)kv * kBlocks * kFragBytes;
    const float* gbias = cbias + (size_t)kv * kCW;
    constexpr int kBuf = kFragBytes + 128;
    float s1[2], s2[2], s3[2];
    int c1[2] = {0, 0}, c2[2] = {0, 0};
#pragma unroll
    for (int tile = 0; tile < 2; ++tile) s1[tile] = s2[tile] = s3[tile] = INFINITY;

    // The loads of the next block are issued here and waited for where they are used: without the address that the compiler
    // cannot look through and the fence behind them it sinks them past the ranking branches down to their only use, the
    // LDS store before the barrier, and every step then waits for global memory in the open.
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    typedef const __attribute__((address_space(1))) uint8_t* global_ptr;
    auto prefetch = [&](int bi, u32x4 (&p)[kFragBytes / 16 / kEncThreads], float& pb) {
      bi = min(bi, kBlocks - 1);   // the step of the last block loads it once more, unused
      global_ptr src = (global_ptr)(gblk + (size_t)bi * kFragBytes + tid * 16);
      global_ptr bsrc = (global_ptr)(gbias + bi * 32 + (tid & 31));
      asm volatile("" : "+v"(src), "+v"(bsrc));
#pragma unroll
      for (int i = 0; i < kFragBytes / 16 / kEncThreads; ++i)
        p[i] = *(const __attribute__((address_space(1))) u32x4*)(src + i * kEncThreads * 16);
      pb = *(const __attribute__((address_space(1))) float*)bsrc;
      asm volatile("" ::: "memory");
    };
    auto stage = [&](int bi, u32x4 (&p)[kFragBytes / 16 / kEncThreads], float& pb) {
      uint8_t* dst = s_mem + (bi & 1) * kBuf;
#pragma unroll
      for (int i = 0; i < kFragBytes / 16 / kEncThreads; ++i) *(u32x4*)(dst + tid * 16 + i * kEncThreads * 16) = p[i];
      *(float*)(dst + kFragBytes + (tid & 31) * 4) = pb;   // several threads write each word, all the same
    };
    {
      u32x4 p[kFragBytes / 16 / kEncThreads];
      float pb;
      prefetch(cb0, p, pb);
      stage(cb0, p, pb);
    }
    __syncthreads();
#pragma unroll 1
    for (int cb = cb0; cb < cb1; ++cb) {
      // The order of the memory operations is pinned (nothing crosses a fence): the next block is
      // requested from global memory first, and the operands of k-step kt + 1 are requested from
      // LDS before the six products of k-step kt, so neither latency is waited for in the open.
      u32x4 p[kFragBytes / 16 / kEncThreads];
      float pb;
      prefetch(cb + 1, p, pb);
      __builtin_amdgcn_sched_barrier(0);
      const uint8_t* blk = s_mem + (cb & 1) * kBuf;
      const uint8_t* fr = blk + lane * 16;
      bf16x8 a_hi = *(const bf16x8*)fr, a_lo = *(const bf16x8*)(fr + 8 * 1024);
      // register v of a tile: codeword 32 cb + 8 (v/4) + 4 g + v%4 (the 4 g is added at the end)
      f32x16 acc0, acc1;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float4 f = *(const float4*)(blk + kFragBytes + (8 * q + 4 * g) * 4);
        acc0[4 * q] = acc1[4 * q] = f.x;
        acc0[4 * q + 1] = acc1[4 * q + 1] = f.y;
        acc0[4 * q + 2] = acc1[4 * q + 2] = f.z;
        acc0[4 * q + 3] = acc1[4 * q + 3] = f.w;
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int kt = 0; kt < 8; ++kt) {
        bf16x8 n_hi = a_hi, n_lo = a_lo;
        if (kt < 7) {
          n_hi = *(const bf16x8*)(fr + (kt + 1) * 1024);
          n_lo = *(const bf16x8*)(fr + (8 + kt + 1) * 1024);
        }
        __builtin_amdgcn_sched_barrier(0);
        acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a_hi, zh[0][kt], acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a_hi, zh[1][kt], acc1, 0, 0, 0);
        acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a_hi, zl[0][kt], acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a_hi, zl[1][kt], acc1, 0, 0, 0);
        acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a_lo, zh[0][kt], acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a_lo, zh[1][kt], acc1, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        a_hi = n_hi;
        a_lo = n_lo;
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float m0 = fminf(fminf(acc0[4 * q], acc0[4 * q + 1]), fminf(acc0[4 * q + 2], acc0[4 * q + 3]));
        if (m0 < s3[0]) {
#pragma unroll
          for (int r = 0; r < 4; ++r) top3_insert(acc0[4 * q + r], cb * 32 + 8 * q + r, s1[0], s2[0], s3[0], c1[0], c2[0]);
        }
        const float m1 = fminf(fminf(acc1[4 * q], acc1[4 * q + 1]), fminf(acc1[4 * q + 2], acc1[4 * q + 3]));
        if (m1 < s3[1]) {
#pragma unroll
          for (int r = 0; r < 4; ++r) top3_insert(acc1[4 * q + r], cb * 32 + 8 * q + r, s1[1], s2[1], s3[1], c1[1], c2[1]);
        }
      }
      stage(cb + 1, p, pb);
      __syncthreads();
    }

    // The two lane halves of a key column hold disjoint codewords: merge them, then the slices, decide, flag.
    const float wmax = __uint_as_float(cstat[kv].w_max);
    // score s of code c (not tracked: 0x7fffffff, never wins a tie) into the smallest three (equal scores: lower code first)
    auto insert = [](float s, int c, float& m1, float& m2, float& m3, int& d1, int& d2) {
      const bool lt1 = s < m1 || (s == m1 && c < d1), lt2 = s < m2 || (s == m2 && c < d2);
      m3 = lt2 ? m2 : fminf(m3, s);
      d2 = lt1 ? d1 : (lt2 ? c : d2);
      m2 = lt1 ? m1 : (lt2 ? s : m2);
      d1 = lt1 ? c : d1;
      m1 = lt1 ? s : m1;
    };
    int d1[2], d2[2];
#pragma unroll
    for (int tile = 0; tile < 2; ++tile) {
      d1[tile] = c1[tile] + 4 * g;
      d2[tile] = c2[tile] + 4 * g;
      const float o1 = __shfl_xor(s1[tile], 32), o2 = __shfl_xor(s2[tile], 32), o3 = __shfl_xor(s3[tile], 32);
      const int b1 = __shfl_xor(d1[tile], 32), b2 = __shfl_xor(d2[tile], 32);
      zn2[tile] += __shfl_xor(zn2[tile], 32);
      insert(o1, b1, s1[tile], s2[tile], s3[tile], d1[tile], d2[tile]);
      insert(o2, b2, s1[tile], s2[tile], s3[tile], d1[tile], d2[tile]);
      insert(o3, 0x7fffffff, s1[tile], s2[tile], s3[tile], d1[tile], d2[tile]);
    }
    if (slices > 1) {   // (uniform) the workgroup that is last to finish a chunk decides it
      NearPart* mine = parts + ((size_t)kv * gridDim.x + item) * kKeysPerWG + wave * kKeysPerWave + col;
      if (g == 0) {
#pragma unroll
        for (int tile = 0; tile < 2; ++tile)
          mine[32 * tile] = NearPart{s1[tile], s2[tile], s3[tile], (uint32_t)d1[tile] | ((uint32_t)d2[tile] << 16)};
      }
      // Each wave's parts have arrived before the barrier, so that one fence behind it covers them all (from every wave: 5 us more).
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      if (tid == 0) __threadfence();
      if (tid == 0) s_last = atomicAdd(arrived + (size_t)kv * gridDim.x + chunk, 1u) == (uint32_t)slices - 1 ? 1u : 0u;
      __syncthreads();
      if (!s_last) continue;
      __threadfence();
      const NearPart* all = mine - (size_t)(item % slices) * kKeysPerWG;
#pragma unroll
      for (int tile = 0; tile < 2; ++tile) {
        s1[tile] = s2[tile] = s3[tile] = INFINITY;
        d1[tile] = d2[tile] = 0;
#pragma unroll 1
        for (int i = 0; i < slices; i += 4) {   // (four parts requested together; there are 2, 4, 8 or 16)
          NearPart o[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) o[u] = all[(size_t)min(i + u, slices - 1) * kKeysPerWG + 32 * tile];
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            if (i + u >= slices) break;   // (uniform)
            insert(o[u].s1, (int)(o[u].codes & 0xffffu), s1[tile], s2[tile], s3[tile], d1[tile], d2[tile]);
            insert(o[u].s2, (int)(o[u].codes >> 16), s1[tile], s2[tile], s3[tile], d1[tile], d2[tile]);
            insert(o[u].s3, 0x7fffffff, s1[tile], s2[tile], s3[tile], d1[tile], d2[tile]);
          }
        }
      }
    }
#pragma unroll
    for (int tile = 0; tile < 2; ++tile)
      if (g == 0 && key_first + 32 * tile + col < n_near) {
        const size_t row = row_of(tile);
        const float reach = kSplitReach * sqrtf(zn2[tile]) * wmax + kSumReach * fabsf(s1[tile]);
        codes[row / n_new * ctx_stride + pos0 + row % n_new] = (uint16_t)d1[tile];
        if (!(s2[tile] - s1[tile] > reach)) {
          const uint32_t full = !(s3[tile] - s1[tile] > reach) ? 0x80000000u : 0u;
          uint32_t* at = list + 2 * ((size_t)kv * near_cap + atomicAdd(&found[kv * kFoundStride], 1u));
          at[0] = (uint32_t)row | full;
          at[1] = (uint32_t)d1[tile] | ((uint32_t)d2[tile] << 16);
        }
      }
  }
}

// ------------------------------------------------------------------------------------------
// Exact decisions in float64
// ------------------------------------------------------------------------------------------
// How much further codeword c is from a key than codeword b: with e = k - c and H symmetric, e_c H e_c^T - e_b H e_b^T =
// (w_b - w_c) . (e_b + e_c).  Differences are taken first, so the error goes with the distances |e|, not with |k|.
//
// Keys with two close codewords take a wave each, two dimensions a lane, two keys requested together; keys with three, the
// whole workgroup: first the smallest 1/2 |c^z|^2 - k . w_c of all codewords, whose error goes with |k| |w|, and then every
// codeword that this leaves open against that one.
// What bounds it: for pairs the columns of wT, 256 cache lines for each (a KV head's keys are a list of their own, so that with 8
// KV heads an XCD reads the columns of one); for the others the 4 MB that one workgroup reads, 60 us.  4194304 keys drawn like
// their codewords, 8061 pairs and 14 of three: 448 -> 107 us against e H e^T of every pair and codewords one row after the other.
constexpr int kPairsAhead = 2, kRecheckBatch = 16;   // keys of a wave: requested together, between two looks at who has three
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 4))) void encode_single_recheck_kernel(
    const float* __restrict__ keys, const float* __restrict__ codebook, const Center* __restrict__ center,
    const CodewordStat* __restrict__ cstat, const double* __restrict__ wT, const double* __restrict__ chalf,
    uint16_t* __restrict__ codes, const uint32_t* __restrict__ found, const uint32_t* __restrict__ lists, int64_t near_cap, int n_new,
    int pos0, int64_t ctx_stride) {
  constexpr int kWaves = 4, kPer = kCW / 256;
  __shared__ double s_k[kD], s_x[kD], s_e[kD], s_w[kD], s_d[256], s_n[kWaves];
  __shared__ int s_i[256];
  __shared__ uint32_t s_full[kWaves], s_n_open;
  __shared__ uint16_t s_open[kCW];
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kv = blockIdx.x;
  codebook += (size_t)kv * kCW * kD;
  wT += (size_t)kv * kD * kCW;
  chalf += (size_t)kv * kCW;
  const uint32_t* list = lists + 2 * (size_t)kv * near_cap;
  const uint32_t count = found[kv * kFoundStride], n_waves = gridDim.y * kWaves;
  const uint32_t per = min((uint32_t)kRecheckBatch, (count + n_waves - 1) / n_waves);
  auto out_of = [&](uint32_t key) -> uint16_t* { return codes + (size_t)(key / (uint32_t)n_new) * ctx_stride + pos0 + key % (uint32_t)n_new; };
  for (uint32_t base = blockIdx.y * kWaves * per; base < count; base += n_waves * per) {
    const uint32_t first = base + (uint32_t)wv * per, n = first < count ? min(per, count - first) : 0u;
    uint32_t key = 0, pair = 0;   // of the wave's key `lane`
    if ((uint32_t)lane < n) {
      const uint2 e = *(const uint2*)(list + 2 * (size_t)(first + lane));
      key = e.x;
      pair = e.y;
    }
    const uint32_t full = (uint32_t)__builtin_amdgcn_ballot_w64((key >> 31) != 0u);   // (lanes past the wave's keys: 0)
    if (lane == 0) s_full[wv] = full;
    for (uint32_t i0 = 0; i0 < n; i0 += kPairsAhead) {
      double wa[kPairsAhead][2], wb[kPairsAhead][2];
      float x[kPairsAhead][2], a[kPairsAhead][2], b[kPairsAhead][2];
#pragma unroll
      for (int u = 0; u < kPairsAhead; ++u) {
        const int i = (int)min(i0 + u, n - 1);
        const uint32_t row = (uint32_t)__builtin_amdgcn_readlane((int)key, i) & 0x7fffffffu;
        const uint32_t two = (full >> i) & 1u ? 0u : (uint32_t)__builtin_amdgcn_readlane((int)pair, i);
        const uint32_t ca = two & 0xffffu, cb = two >> 16;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int t = lane + 64 * h;
          x[u][h] = keys[(size_t)row * kD + t];
          a[u][h] = codebook[ca * kD + t];
          b[u][h] = codebook[cb * kD + t];
          wa[u][h] = wT[(uint32_t)t * kCW + ca];
          wb[u][h] = wT[(uint32_t)t * kCW + cb];
        }
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < kPairsAhead; ++u) {
        double d = 0.0;
#pragma unroll
        for (int h = 0; h < 2; ++h)
          d += (wa[u][h] - wb[u][h]) * (((double)x[u][h] - (double)a[u][h]) + ((double)x[u][h] - (double)b[u][h]));
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) d += __shfl_xor(d, off);
        const int i = (int)(i0 + u);
        if (i0 + u >= n || ((full >> i) & 1u)) continue;   // (uniform)
        const uint32_t two = (uint32_t)__builtin_amdgcn_readlane((int)pair, i), ca = two & 0xffffu, cb = two >> 16;
        if (lane == 0)
          *out_of((uint32_t)__builtin_amdgcn_readlane((int)key, i)) = (uint16_t)(d < 0.0 || (d == 0.0 && cb < ca) ? cb : ca);
      }
    }
    __syncthreads();
    for (int v = 0; v < kWaves; ++v)
      for (uint32_t left = s_full[v]; left != 0u; left &= left - 1u) {   // (uniform)
        const uint32_t row = list[2 * (size_t)(base + v * per + (__ffs((int)left) - 1))] & 0x7fffffffu;
        const int t = tid & (kD - 1);
        const float x = keys[(size_t)row * kD + t];
        const double from_mu = (double)x - (double)center[kv].mu[t];
        __syncthreads();   // the arrays of the key before are still being read
        if (tid < kD) {
          s_k[t] = from_mu;
          s_x[t] = (double)x;
        }
        double kt = from_mu * (double)center[kv].t[t];
        kt *= kt;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) kt += __shfl_xor(kt, off);
        if (lane == 0) s_n[wv] = kt;
        if (__syncthreads_or(!(fabsf(x) < INFINITY))) {   // a key that is not finite is as far from all
          if (tid == 0) *out_of(row) = 0;
          continue;
        }
        double value[kPer], best = INFINITY;
        int arg = tid;
        constexpr int kGo = 8, kRows = 1;   // codewords a thread sums at a time; rows of each half requested together (2: spills)
#pragma unroll
        for (int q0 = 0; q0 < kPer; q0 += kGo) {
          double p[kGo][2] = {}, w[2][kRows][kGo][2];
          auto request = [&](int r, int buffer) {
#pragma unroll
            for (int u = 0; u < kRows; ++u)
#pragma unroll
              for (int h = 0; h < 2; ++h) {
                const double* row = wT + (size_t)(min(r + u, kD / 2 - 1) + h * (kD / 2)) * kCW + 256 * q0;
                asm volatile("" : "+s"(row));   // (else an address of every load is kept by every lane, and spilled)
#pragma unroll
                for (int q = 0; q < kGo; ++q) w[buffer][u][q][h] = row[(uint32_t)(tid + 256 * q)];
              }
            __builtin_amdgcn_sched_barrier(0);
          };
          auto add = [&](int r, int buffer) {
#pragma unroll
            for (int u = 0; u < kRows; ++u)
#pragma unroll
              for (int q = 0; q < kGo; ++q)
#pragma unroll
                for (int h = 0; h < 2; ++h) p[q][h] = __builtin_fma(s_k[r + u + h * (kD / 2)], w[buffer][u][q][h], p[q][h]);
            __builtin_amdgcn_sched_barrier(0);
          };
          request(0, 0);
#pragma unroll 1
          for (int r = 0; r < kD / 2; r += 2 * kRows) {
            request(r + kRows, 1);
            add(r, 0);
            request(r + 2 * kRows, 0);
            add(r + kRows, 1);
          }
          const double* half = chalf + 256 * q0;
          asm volatile("" : "+s"(half));
#pragma unroll
          for (int q = 0; q < kGo; ++q) {
            value[q0 + q] = half[(uint32_t)(tid + 256 * q)] - (p[q][0] + p[q][1]);
            if (value[q0 + q] < best) {   // (not if it is not a number)
              best = value[q0 + q];
              arg = tid + 256 * (q0 + q);
            }
          }
        }
        auto smallest = [&]() {   // of best, and of equal ones that of the lowest code, in s_d[0] and s_i[0]
          s_d[tid] = best;
          s_i[tid] = arg;
          __syncthreads();
          for (int s = 128; s >= 1; s >>= 1) {
            if (tid < s) {
              const double o = s_d[tid + s];
              const int oi = s_i[tid + s];
              if (o < s_d[tid] || (o == s_d[tid] && oi < s_i[tid])) {
                s_d[tid] = o;
                s_i[tid] = oi;
              }
            }
            __syncthreads();
          }
        };
        if (tid == 0) s_n_open = 0;
        smallest();
        const int cb = s_i[0];
        // What two sums of two chains of 64 products each, with half of as many for 1/2 c . w, can be off by, and some more
        const CodewordStat& st = cstat[kv];
        const double reach = 0x1p-45 * (sqrt(s_n[0] + s_n[1]) + (double)__uint_as_float(st.c_max)) * (double)__uint_as_float(st.w_max);
        const double most = s_d[0] + reach;
        if (tid < kD) {
          s_e[t] = s_x[t] - (double)codebook[cb * kD + t];
          s_w[t] = wT[(size_t)t * kCW + cb];
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kPer; ++q)
          if (value[q] <= most && tid + 256 * q != cb) s_open[atomicAdd(&s_n_open, 1u)] = (uint16_t)(tid + 256 * q);
        __syncthreads();
        best = 0.0;
        arg = cb;
        for (uint32_t i = tid; i < s_n_open; i += 256) {
          const int c = s_open[i];
          const float4* row_c = (const float4*)(codebook + c * kD);
          constexpr int kStep = 32;   // dimensions requested together
          double d = 0.0;
#pragma unroll 1
          for (int r0 = 0; r0 < kD; r0 += kStep) {
            double w[kStep];
            float4 x4[kStep / 4];
#pragma unroll
            for (int r = 0; r < kStep / 4; ++r) x4[r] = row_c[r0 / 4 + r];
#pragma unroll
            for (int r = 0; r < kStep; ++r) w[r] = wT[(uint32_t)(r0 + r) * kCW + c];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = 0; r < kStep; ++r) {
              const float cr = r % 4 == 0 ? x4[r / 4].x : (r % 4 == 1 ? x4[r / 4].y : (r % 4 == 2 ? x4[r / 4].z : x4[r / 4].w));
              d += (s_w[r0 + r] - w[r]) * (s_e[r0 + r] + (s_x[r0 + r] - (double)cr));
            }
          }
          if (d < best || (d == best && c < arg)) {
            best = d;
            arg = c;
          }
        }
        smallest();
        if (tid == 0) *out_of(row) = (uint16_t)s_i[0];
      }
    __syncthreads();   // s_full is written again
  }
}

// No counts yet, and no KV head takes the i8 filter.
__global__ void encode_single_clear_kernel(uint32_t* counter, int n, uint32_t* found, uint32_t* eight, int Hkv) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) counter[i] = 0;
  for (int i = threadIdx.x; i < Hkv; i += blockDim.x) found[i * kFoundStride] = 0;
  for (int i = threadIdx.x; i < Hkv; i += blockDim.x) eight[i] = 0;
}

// The few-key (append) route of a few keys in all: every key is decided by a float64 sweep, its 4096 codewords split
// over kSlices workgroups (one workgroup would read 4 MB by itself).  With w_c = c H the
// distortion of codeword c is |z|^2 - 2 k . w_c + |c^z|^2, so the sweep minimises
// 1/2 |c^z|^2 - k . w_c and needs neither z nor L: one pass of dot products over wT.
// part[key][slice] = {smallest value of the slice, its code as a double}.
// Each half of the dimensions is added one after the other without rounding the products, as the float64 matrix cores add them
// (build_lut_single_kernel): the codes do not depend on which of the two a call takes, whatever the rounding.
constexpr int kSweepThreads = 512;
__global__ __launch_bounds__(kSweepThreads) __attribute__((amdgpu_waves_per_eu(4, 4))) void encode_single_sweep_kernel(
    const float* __restrict__ keys, const float* __restrict__ mu, int mu_stride, const double* __restrict__ wT,
    const double* __restrict__ chalf, double* __restrict__ part, int Hkv, int n_new) {
  constexpr int PER = kCW / kSlices;   // codewords per slice
  static_assert(PER == 256 && kSweepThreads == 2 * PER, "a thread owns one codeword and half of the dimensions");
  __shared__ double s_k[kD], s_p[2][PER];
  __shared__ int s_i[PER];
  const int tid = threadIdx.x, slice = blockIdx.y, key = blockIdx.x;
  const int bkv = key / n_new, kv = bkv % Hkv;
  // thread = (codeword, half of the dimensions): the first 32 of its 64 entries are requested before
  // the key is looked at; each is replaced by its successor as it is used.  (The fences keep the
  // compiler from requesting the second half up front as well, which would not fit the registers.)
  const int cl = tid & (PER - 1), th = tid >> 8, c = slice * PER + cl;
  const double* w = wT + ((size_t)kv * kD + 64 * th) * kCW + c;
  double wv[32];
#pragma unroll
  for (int t = 0; t < 32; ++t) wv[t] = w[(size_t)t * kCW];
  const double half = chalf[(size_t)kv * kCW + c];
  if (tid < kD) s_k[tid] = (double)keys[(size_t)key * kD + tid] - (double)mu[(size_t)kv * mu_stride + tid];
  __builtin_amdgcn_sched_barrier(0);
  __syncthreads();
  double dot = 0.0;
#pragma unroll
  for (int t = 0; t < 32; t += 2) {
    dot = __builtin_fma(s_k[64 * th + t], wv[t], dot);
    dot = __builtin_fma(s_k[64 * th + t + 1], wv[t + 1], dot);
    wv[t] = w[(size_t)(32 + t) * kCW];
    wv[t + 1] = w[(size_t)(32 + t + 1) * kCW];
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int t = 0; t < 32; ++t) dot = __builtin_fma(s_k[64 * th + 32 + t], wv[t], dot);
  s_p[th][cl] = dot;
  __syncthreads();
  if (tid < PER) {   // (a value that is not a number is never the smallest, as there)
    const double value = half - (s_p[0][tid] + s_p[1][tid]);
    s_p[0][tid] = value < INFINITY ? value : INFINITY;
    s_i[tid] = c;
  }
  __syncthreads();
  for (int s = PER / 2; s >= 1; s >>= 1) {
    if (tid < s) {
      const double o = s_p[0][tid + s];
      const int oi = s_i[tid + s];
      if (o < s_p[0][tid] || (o == s_p[0][tid] && oi < s_i[tid])) {
        s_p[0][tid] = o;
        s_i[tid] = oi;
      }
    }
    __syncthreads();
  }
  if (tid == 0) {
    part[((size_t)key * kSlices + slice) * 2] = s_p[0][0];
    part[((size_t)key * kSlices + slice) * 2 + 1] = (double)s_i[0];
  }
}

__global__ void encode_single_sweep_pick_kernel(const double* __restrict__ part, uint16_t* __restrict__ codes,
                                                uint32_t n_all, int n_new, int pos0, int64_t ctx_stride) {
  const uint32_t key = blockIdx.x * blockDim.x + threadIdx.x;
  if (key >= n_all) return;
  double best = part[(size_t)key * kSlices * 2];
  int arg = (int)part[(size_t)key * kSlices * 2 + 1];
  for (int s = 1; s < kSlices; ++s) {   // slices hold ascending codes: strict < keeps the lower code
    const double d = part[((size_t)key * kSlices + s) * 2];
    if (d < best) {
      best = d;
      arg = (int)part[((size_t)key * kSlices + s) * 2 + 1];
    }
  }
  const int bkv = (int)(key / (uint32_t)n_new), j = (int)(key % (uint32_t)n_new);
  codes[(size_t)bkv * ctx_stride + pos0 + j] = (uint16_t)arg;
}

// ------------------------------------------------------------------------------------------
// k-means++ seeding under the query-aware distortion (section 4.2 initialises its k-means that
// way): the first codeword is key floor(u_0 n), every further one is drawn with probability
// proportional to the distortion to the nearest codeword chosen so far.  The draws are sequential,
// so one workgroup per KV head runs all of them; the caller supplies the uniform numbers u.
// Distortions are ||z_i - z_c||^2 in float64 over the float32 transformed keys z = k L.
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void scale_keys_kernel(const float* __restrict__ keys, const double* __restrict__ sd,
                                                         float* __restrict__ z, int Hkv, size_t n_rows_per_seq) {
  const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;   // element of [B*Hkv][n][128]
  const int bkv = blockIdx.y, kv = bkv % Hkv;
  if (e >= n_rows_per_seq * kD) return;
  const size_t at = (size_t)bkv * n_rows_per_seq * kD + e;
  z[at] = (float)((double)keys[at] * sd[(size_t)kv * kD + e % kD]);
}

constexpr int kSeedThreads = 1024;
constexpr int kSeedChunk = 4;   // consecutive rows per thread of the update kernel = rows per partial sum

// State of the draws of one KV head between the kernels of a round.
struct SeedState {
  long pick;          // row of the codeword drawn last
  float zc[kD];       // its transformed key
};

__device__ __forceinline__ const float* seed_row(const float* base, long i, int kv, int Hkv, int n_new) {
  return base + (((size_t)(i / n_new) * Hkv + kv) * n_new + i % n_new) * kD;
}

// Records draw r (st->pick): the codeword is the key itself; keeps its transformed key for the update.
__device__ __forceinline__ void seed_record(SeedState* st, const float* keys, const float* z, float* codebook_out,
                                            int32_t* picks, long pick, int r, int kv, int Hkv, int n_new, int tid) {
  if (tid < kD) {
    codebook_out[((size_t)kv * kCW + r) * kD + tid] = seed_row(keys, pick, kv, Hkv, n_new)[tid];
    st->zc[tid] = seed_row(z, pick, kv, Hkv, n_new)[tid];
  }
  if (tid == 0) {
    st->pick = pick;
    if (picks) picks[(size_t)kv * kCW + r] = (int32_t)pick;
  }
}

__global__ __launch_bounds__(128) void seed_first_kernel(const float* __restrict__ keys, const float* __restrict__ z,
                                                         const double* __restrict__ u, SeedState* __restrict__ state,
                                                         float* __restrict__ codebook_out, int32_t* __restrict__ picks,
                                                         int B, int Hkv, int n_new) {
  const int kv = blockIdx.x;
  const long rows = (long)B * n_new;
  const long pick = min(rows - 1, (long)(u[(size_t)kv * kCW] * (double)rows));
  seed_record(state + kv, keys, z, codebook_out, picks, pick, 0, kv, Hkv, n_new, threadIdx.x);
}

// Distortions of every row to the codeword drawn last, running minimum, and one partial sum per
// kSeedChunk consecutive rows (summed in row order).
__global__ __launch_bounds__(256) void seed_update_kernel(const float* __restrict__ z, const SeedState* __restrict__ state,
                                                          double* __restrict__ dmin, double* __restrict__ partial,
                                                          int B, int Hkv, int n_new, int first_round) {
  __shared__ double s_zc[kD];
  const int kv = blockIdx.y, tid = threadIdx.x;
  const long rows = (long)B * n_new, n_part = (rows + kSeedChunk - 1) / kSeedChunk;
  if (tid < kD) s_zc[tid] = (double)state[kv].zc[tid];
  __syncthreads();
  const long p = (long)blockIdx.x * 256 + tid;
  if (p >= n_part) return;
  double* d = dmin + (size_t)kv * rows;
  double own = 0.0;
  for (long i = p * kSeedChunk; i < min(rows, (p + 1) * kSeedChunk); ++i) {
    const float4* zi = (const float4*)seed_row(z, i, kv, Hkv, n_new);
    double acc = 0.0;
#pragma unroll 8
    for (int t4 = 0; t4 < kD / 4; ++t4) {
      const float4 f = zi[t4];
      const double e0 = (double)f.x - s_zc[4 * t4], e1 = (double)f.y - s_zc[4 * t4 + 1];
      const double e2 = (double)f.z - s_zc[4 * t4 + 2], e3 = (double)f.w - s_zc[4 * t4 + 3];
      acc += e0 * e0;
      acc += e1 * e1;
      acc += e2 * e2;
      acc += e3 * e3;
    }
    const double dm = first_round ? acc : fmin(d[i], acc);
    d[i] = dm;
    own += dm;
  }
  partial[(size_t)kv * n_part + p] = own;
}

// Draw r: the first row whose inclusive prefix sum of the distortions exceeds u_r times their total.
__global__ __launch_bounds__(kSeedThreads) void seed_pick_kernel(
    const float* __restrict__ keys, const float* __restrict__ z, const double* __restrict__ u,
    const double* __restrict__ dmin, const double* __restrict__ partial, SeedState* __restrict__ state,
    float* __restrict__ codebook_out, int32_t* __restrict__ picks, int B, int Hkv, int n_new, int r) {
  __shared__ double s_wave[kSeedThreads / 64];
  __shared__ long s_pick;
  __shared__ int s_owner;
  const int kv = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const long rows = (long)B * n_new, n_part = (rows + kSeedChunk - 1) / kSeedChunk;
  const long per = (n_part + kSeedThreads - 1) / kSeedThreads;
  const long p_lo = min(n_part, tid * per), p_hi = min(n_part, p_lo + per);   // this thread's contiguous partials
  const double* pk = partial + (size_t)kv * n_part;
  double own = 0.0;
  for (long p = p_lo; p < p_hi; ++p) own += pk[p];
  double inc = own;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const double o = __shfl_up(inc, off);
    if (lane >= off) inc += o;
  }
  if (lane == 63) s_wave[wave] = inc;
  __syncthreads();
  double base = 0.0, total = 0.0;
  for (int w = 0; w < kSeedThreads / 64; ++w) {
    if (w < wave) base += s_wave[w];
    total += s_wave[w];
  }
  base += inc - own;
  const double ur = u[(size_t)kv * kCW + r], target = ur * total;
  // all distortions zero (every key equals a chosen codeword): a uniform draw instead
  if (tid == 0) {
    s_pick = total > 0.0 ? 0 : min(rows - 1, (long)(ur * (double)rows));
    s_owner = -1;
  }
  __syncthreads();
  // the row belongs to the last thread whose exclusive prefix does not exceed the target
  // (prefixes do not decrease with the thread index)
  const uint64_t below = __ballot(total > 0.0 && p_lo < p_hi && base <= target);
  if (lane == 0 && below) atomicMax(&s_owner, wave * 64 + 63 - (int)__clzll((unsigned long long)below));
  __syncthreads();
  if (tid == s_owner) {
    const double* d = dmin + (size_t)kv * rows;
    double run = base;
    long found = min(rows, p_hi * kSeedChunk) - 1;   // (rounding: if the walk falls short, the thread's last row)
    bool done = false;
    for (long p = p_lo; p < p_hi && !done; ++p) {
      if (run + pk[p] > target || p == p_hi - 1) {   // the row is in this partial (or the walk ends here)
        for (long i = p * kSeedChunk; i < min(rows, (p + 1) * kSeedChunk); ++i) {
          run += d[i];
          if (run > target) {
            found = i;
            done = true;
            break;
          }
        }
        if (!done && p < p_hi - 1) continue;   // rounding: the partial fell just short; go on
        done = true;
      } else {
        run += pk[p];
      }
    }
    s_pick = found;
  }
  __syncthreads();
  seed_record(state + kv, keys, z, codebook_out, picks, s_pick, r, kv, Hkv, n_new, tid);
}

LdsSlot g_factor_lds[16];

}  // namespace

// Which products see a call's keys first.  us of whole calls, before there were products in 8 bits -> now, keys near their codewords
// (0.1) | normal keys; 8 KV heads unless stated:
//   kSampleProducts: those of the sample, which then has all keys.  100 keys 57 -> 18 | 175 -> 85, 500 78 -> 26 | 183 -> 109; one
//     KV head of 2000 57 -> 18 | 119 -> 72; 24 of 250 81 -> 35 | 211 -> 121.  By a filter that a sample chose 500 keys take 38 | 148.
//     The line is where that becomes the better one: 1024 keys 43 by the sample's products, 40 by a chosen filter.
//   kChosenFilter: 1024 keys 81 -> 40 | 187 -> 141, 12000 159 -> 75 | 333 -> 226, 96001 713 -> 402 | 1169 -> 1117.
//   kFilter16: so many KV heads that the sample, which reads all their codewords, costs what it saves.  64 of 250 keys 78 -> 57 | 264
//     -> 158 (by a chosen filter 78 | 193), 128 of 1000 156 -> 152 | 405 -> 326 (162 | 412).
// Between the two kinds of keys lie some that the f16 filter would all decide and 8 bits not.  Their list takes 35 us at the least: at
// a noise of 1.0 12000 keys 249 -> 147, 2000 81 -> 78, 500 78 -> 63, but 40 of 32 sequences 58 -> 75, one KV head of 4000 58 -> 68
// and 32 of 1100 87 -> 118.
enum Route { kSampleProducts, kChosenFilter, kFilter16 };
static Route single_route(long n_rows, int Hkv) {   // (n_rows: keys of a KV head)
  const long groups = (n_rows + kSampleKeys - 1) / kSampleKeys;
  if (Hkv > 24 && n_rows < 32l * Hkv) return kFilter16;
  return groups <= 24 && groups * Hkv <= 48 ? kSampleProducts : kChosenFilter;
}

size_t encode_single_ws_bytes(const a2ats_dims& d) { return enc_single_ws(d).bytes; }

hipError_t launch_encode_single_prepare(const a2ats_dims& d, const float* codebook, const float* weights, int mode,
                                        void* ws, hipStream_t stream) {
  const EncWs w = enc_single_ws(d);
  uint8_t* base = (uint8_t*)ws;
  double* sd = (double*)(base + w.off_sd);
  CodewordStat* cstat = (CodewordStat*)(base + w.off_cstat);
  double* means = (double*)(base + w.off_means);
  double* hmat = (double*)(base + w.off_hmat);
  Center* center = (Center*)(base + w.off_center);
  hipLaunchKernelGGL(encode_single_matrix_kernel, dim3(d.n_kv_heads, kMeans + kD / kMatrixRows), dim3(kMatrixThreads), 0, stream, weights,
                     mode, hmat, sd, cstat, codebook, means, (float*)(base + w.off_copy));
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  hipLaunchKernelGGL(encode_single_codewords_kernel, dim3(kCW / 64, d.n_kv_heads), dim3(256), 0, stream, codebook,
                     mode, sd, hmat, means, center, (double*)(base + w.off_wT), (double*)(base + w.off_chalf),
                     (float*)(base + w.off_cbias), cstat);
  if ((err = hipGetLastError()) != hipSuccess) return err;
  hipLaunchKernelGGL(encode_single_operands_kernel, dim3(kBlocks, d.n_kv_heads), dim3(512), 0, stream,
                     (const double*)(base + w.off_wT), center, (const float*)(base + w.off_cbias), (uint16_t*)(base + w.off_cfrag),
                     (_Float16*)(base + w.off_f16), (float*)(base + w.off_fbias), base + w.off_i8, (int*)(base + w.off_bias8), cstat);
  return hipGetLastError();
}

size_t encode_single_scratch_bytes(const a2ats_dims& d) {
  const EncWs w = enc_single_ws(d);
  return w.off_near_part - w.off_list;   // the lists of a call with more keys
}

hipError_t launch_encode_single_few(const a2ats_dims& d, const float* keys, int n_new, const float* codebook,
                                    const float* weights, int mode, bool prepared, void* ws, FewKeys* few, void** scratch,
                                    hipStream_t stream) {
  const EncWs w = enc_single_ws(d);
  uint8_t* base = (uint8_t*)ws;
  few->keys = keys;
  few->mu = ((const Center*)(base + w.off_center))->mu;
  few->mu_stride = sizeof(Center) / sizeof(float);
  few->wT = (const double*)(base + w.off_wT);
  few->chalf = (const double*)(base + w.off_chalf);
  few->part = (double*)(base + w.off_part);
  few->n_new = n_new;
  *scratch = base + w.off_list;
  return prepared ? hipSuccess : launch_encode_single_prepare(d, codebook, weights, mode, ws, stream);
}

// The sweep of a key at a time, whose results are in few.part.
static hipError_t launch_sweep_by_key(const a2ats_dims& d, const FewKeys& few, hipStream_t stream) {
  hipLaunchKernelGGL(encode_single_sweep_kernel, dim3((unsigned)((size_t)d.batch * d.n_kv_heads * few.n_new), kSlices),
                     dim3(kSweepThreads), 0, stream, few.keys, few.mu, few.mu_stride, few.wT, few.chalf, few.part, d.n_kv_heads,
                     few.n_new);
  return hipGetLastError();
}

static hipError_t launch_pick(const a2ats_dims& d, const FewKeys& few, void* codes, int pos0, hipStream_t stream) {
  const uint32_t n_all = (uint32_t)((size_t)d.batch * d.n_kv_heads * few.n_new);
  hipLaunchKernelGGL(encode_single_sweep_pick_kernel, dim3((n_all + 63) / 64), dim3(64), 0, stream, few.part,
                     (uint16_t*)codes, n_all, few.n_new, pos0, d.ctx_stride);
  return hipGetLastError();
}

// The keys are swept with the tables, and picked by a launch of their own.
hipError_t launch_decode_prologue_single(const a2ats_dims& d, const float* keys, int n_new, int pos0, const float* codebook,
                                         const float* weights, int mode, bool prepared, void* codes, const void* q,
                                         int q_dtype, const float* cos_b, const float* sin_b, float* q_rot, int32_t* lut,
                                         float* lut_scale, void* ws, hipStream_t stream) {
  FewKeys few{};
  void* scratch;
  hipError_t err = launch_encode_single_few(d, keys, n_new, codebook, weights, mode, prepared, ws, &few, &scratch, stream);
  if (err != hipSuccess) return err;
  err = launch_build_lut_single(d, q, q_dtype, cos_b, sin_b, codebook, q_rot, lut, lut_scale, false, few, stream);
  return err == hipSuccess ? launch_pick(d, few, codes, pos0, stream) : err;
}

hipError_t launch_encode_single(const a2ats_dims& d, const float* keys, int n_new, int pos0,
                                const float* codebook, const float* weights, int mode, bool prepared, void* codes,
                                void* ws, hipStream_t stream) {
  if (n_new == 0 || d.batch == 0) return hipSuccess;
  if (n_new <= kFewSingle) {
    FewKeys few{};
    void* scratch;
    hipError_t err = launch_encode_single_few(d, keys, n_new, codebook, weights, mode, prepared, ws, &few, &scratch, stream);
    if (err != hipSuccess) return err;
    // One sweep takes a key at a time, the other one 16 of a KV head on the matrix cores: one key of 8 KV heads 8.7 us against
    // 10.6, of 2 sequences 8.8 against 11.1, of 3 12.4 against 10.6, 8 keys of 4 sequences 70 against 13.1.  The line is where
    // the first has more workgroups than there are CUs.
    err = (long)d.batch * d.n_kv_heads * n_new * kSlices <= 256 ? launch_sweep_by_key(d, few, stream)
                                                                : launch_sweep_single(d, few, stream);
    return err == hipSuccess ? launch_pick(d, few, codes, pos0, stream) : err;
  }
  const EncWs w = enc_single_ws(d);
  uint8_t* base = (uint8_t*)ws;
  const Center* center = (const Center*)(base + w.off_center);
  uint8_t* cfrag = base + w.off_cfrag;
  float* cbias = (float*)(base + w.off_cbias);
  CodewordStat* cstat = (CodewordStat*)(base + w.off_cstat);
  uint32_t* counter = (uint32_t*)(base + w.off_count);
  uint32_t* near = (uint32_t*)(base + w.off_near);
  uint32_t* list = (uint32_t*)(base + w.off_list);
  const int Hkv = d.n_kv_heads, bkv = d.batch * Hkv;
  hipError_t err;
  if (!prepared && (err = launch_encode_single_prepare(d, codebook, weights, mode, ws, stream)) != hipSuccess)
    return err;

  const uint32_t n_all = (uint32_t)((size_t)bkv * n_new);
  uint32_t* found = (uint32_t*)(base + w.off_L);
  const int n_counter = (int)(Hkv + Hkv * near_groups(d));
  // Keys per wave: a workgroup reads all codewords whatever its keys, so 128 where that gives about the 512
  // workgroups that are resident at once, else 64 or 32 (8 KV heads, 32 / 64 / 128 a wave, us: 2000 keys 47 / 59 / 87, 12000
  // 83 / 85 / 89, 20000 122 / 119 / 134, 26000 156 / 152 / 140, 96001 479 / 415 / 395).
  const long waves = (long)bkv * (((long)n_new + 31) / 32);   // (of 32 keys)
  const int nt = waves >= 4L * kEncWaves * 400 ? 4 : (waves >= 2L * kEncWaves * 400 ? 2 : 1);
  const uint8_t *f16 = base + w.off_f16, *i8 = base + w.off_i8;
  const float* fbias = (const float*)(base + w.off_fbias);
  const int* bias8 = (const int*)(base + w.off_bias8);
  int2* sample = (int2*)(base + w.off_sample);
  float2* norms = (float2*)(base + w.off_norms);
  uint32_t* eight = (uint32_t*)(base + w.off_eight);
  const long n_rows = (long)d.batch * n_new, groups = (n_rows + kSampleKeys - 1) / kSampleKeys;
  const dim3 block(kEncThreads);
  const Route route = single_route(n_rows, Hkv);
  if (route == kSampleProducts) {
    sample = (int2*)(base + w.off_near_part);   // (used by the lists' kernels later, as the list is: 48 groups take 1.5 MB of its 2)
    norms = (float2*)list;
    hipLaunchKernelGGL(encode_single_sample_kernel<true>, dim3(kSampleSlices, Hkv, (unsigned)groups), block, 0, stream, keys, center,
                       i8, bias8, sample, norms, counter, n_counter, found, n_new, n_rows);
    if ((err = hipGetLastError()) != hipSuccess) return err;
    hipLaunchKernelGGL(encode_single_decide_kernel, dim3((unsigned)groups, Hkv), block, 0, stream, cstat, sample, norms,
                       (uint16_t*)codes, counter, near, (int64_t)w.near_cap, n_new, n_rows, pos0, d.ctx_stride);
    if ((err = hipGetLastError()) != hipSuccess) return err;
  } else {
    if (route == kFilter16)
      hipLaunchKernelGGL(encode_single_clear_kernel, dim3(1), dim3(1024), 0, stream, counter, n_counter, found, eight, Hkv);
    else
      hipLaunchKernelGGL(encode_single_sample_kernel<false>, dim3(kSampleSlices, Hkv), block, 0, stream, keys, center, i8, bias8,
                         sample, norms, counter, n_counter, found, n_new, n_rows);
    if ((err = hipGetLastError()) != hipSuccess) return err;
    const dim3 grid((n_new + 32 * nt * kEncWaves - 1) / (32 * nt * kEncWaves), bkv);
#define A2ATS_LAUNCH_FILTER(NT, I8, F16)                                                                                      \
  hipLaunchKernelGGL((encode_single_filter_kernel<NT, I8, F16>), grid, block, 0, stream, keys, center, f16, fbias, i8, bias8, sample, \
                     norms, eight, cstat, (uint16_t*)codes, counter, near, (int64_t)w.near_cap, Hkv, n_new, pos0, d.ctx_stride)
    // One launch has both filters, except with 64 keys a wave: there the i8 one has three waves per SIMD, the f16 one the
    // registers of two.
    if (route == kFilter16) {
      if (nt == 4) A2ATS_LAUNCH_FILTER(4, false, true);
      else if (nt == 2) A2ATS_LAUNCH_FILTER(2, false, true);
      else A2ATS_LAUNCH_FILTER(1, false, true);
    } else if (nt == 4) {
      A2ATS_LAUNCH_FILTER(4, true, true);
    } else if (nt == 2) {
      A2ATS_LAUNCH_FILTER(2, true, false);
      if ((err = hipGetLastError()) != hipSuccess) return err;
      A2ATS_LAUNCH_FILTER(2, false, true);
    } else {
      A2ATS_LAUNCH_FILTER(1, true, true);
    }
#undef A2ATS_LAUNCH_FILTER
    if ((err = hipGetLastError()) != hipSuccess) return err;
  }
  hipLaunchKernelGGL(encode_single_kernel, dim3((unsigned)near_groups(d), Hkv), block, 0, stream, keys, center, cfrag, cbias,
                     cstat, (uint16_t*)codes, counter, near, (int64_t)w.near_cap, found, list, counter + Hkv,
                     (NearPart*)(base + w.off_near_part), Hkv, n_new, pos0, d.ctx_stride);
  if ((err = hipGetLastError()) != hipSuccess) return err;
  // (512 workgroups are resident at once; further ones only take their time to start: 300 keys x 8 heads 20.2 -> 19.6 us with 512 instead of
  // 2048, and long lists take the same)
  const unsigned re_parts = (unsigned)std::min<long>(n_rows, std::max(1, 512 / Hkv));
  hipLaunchKernelGGL(encode_single_recheck_kernel, dim3(Hkv, re_parts), dim3(256), 0, stream, keys,
                     (const float*)(base + w.off_copy), center, cstat, (const double*)(base + w.off_wT),
                     (const double*)(base + w.off_chalf), (uint16_t*)codes, found, list, (int64_t)w.near_cap, n_new, pos0, d.ctx_stride);
  return hipGetLastError();
}

struct SeedWs {
  size_t off_z, off_d, off_partial, off_state, bytes;
};
static SeedWs seed_ws(const a2ats_dims& d) {
  const size_t rows = (size_t)d.batch * d.n_kv_heads * (size_t)d.ctx_stride;
  SeedWs w;
  size_t o = enc_single_ws(d).bytes;
  auto take = [&](size_t bytes) {
    const size_t at = o;
    o += (bytes + 255) & ~(size_t)255;
    return at;
  };
  w.off_z = take(rows * kD * sizeof(float));
  w.off_d = take(rows * sizeof(double));
  w.off_partial = take((rows / kSeedChunk + d.n_kv_heads) * sizeof(double));
  w.off_state = take((size_t)d.n_kv_heads * sizeof(SeedState));
  w.bytes = o;
  return w;
}

size_t kmeanspp_ws_bytes(const a2ats_dims& d) { return seed_ws(d).bytes; }

hipError_t launch_kmeanspp_seed(const a2ats_dims& d, const float* keys, int n_new, const float* weights, int mode,
                                const double* u, float* codebook_out, int32_t* picks, void* ws, hipStream_t stream) {
  if (d.n_kv_heads == 0) return hipSuccess;
  const EncWs w = enc_single_ws(d);
  const SeedWs sw = seed_ws(d);
  uint8_t* base = (uint8_t*)ws;
  double* Lmat = (double*)(base + w.off_L);
  double* sd = (double*)(base + w.off_sd);
  float* z = (float*)(base + sw.off_z);
  double* dmin = (double*)(base + sw.off_d);
  double* partial = (double*)(base + sw.off_partial);
  SeedState* state = (SeedState*)(base + sw.off_state);
  const int Hkv = d.n_kv_heads, bkv = d.batch * Hkv;
  const size_t factor_lds = (size_t)kD * kFactorStride * sizeof(double);
  hipError_t err = allow_dynamic_lds(encode_single_factor_kernel, factor_lds, g_factor_lds);
  if (err != hipSuccess) return err;
  hipLaunchKernelGGL(encode_single_factor_kernel, dim3(Hkv), dim3(256), factor_lds, stream, weights, mode, Lmat, sd);
  if ((err = hipGetLastError()) != hipSuccess) return err;
  if (mode == A2ATS_W_BLOCK)
    hipLaunchKernelGGL(encode_single_transform_kernel, dim3((n_new + 63) / 64, bkv), dim3(256), 0, stream, keys, Lmat,
                       z, Hkv, n_new);
  else
    hipLaunchKernelGGL(scale_keys_kernel, dim3((unsigned)(((size_t)n_new * kD + 255) / 256), bkv), dim3(256), 0,
                       stream, keys, sd, z, Hkv, (size_t)n_new);
  if ((err = hipGetLastError()) != hipSuccess) return err;
  // 4096 sequential draws: per draw one kernel over all rows (distortions to the codeword drawn
  // last) and one workgroup per KV head that turns the partial sums into the next draw
  const long rows = (long)d.batch * n_new, n_part = (rows + kSeedChunk - 1) / kSeedChunk;
  hipLaunchKernelGGL(seed_first_kernel, dim3(Hkv), dim3(128), 0, stream, keys, z, u, state, codebook_out, picks,
                     d.batch, Hkv, n_new);
  if ((err = hipGetLastError()) != hipSuccess) return err;
  for (int r = 1; r < kCW; ++r) {
    hipLaunchKernelGGL(seed_update_kernel, dim3((unsigned)((n_part + 255) / 256), Hkv), dim3(256), 0, stream, z, state,
                       dmin, partial, d.batch, Hkv, n_new, r == 1 ? 1 : 0);
    hipLaunchKernelGGL(seed_pick_kernel, dim3(Hkv), dim3(kSeedThreads), 0, stream, keys, z, u, dmin, partial, state,
                       codebook_out, picks, d.batch, Hkv, n_new, r);
    if ((err = hipGetLastError()) != hipSuccess) return err;
  }
  return hipSuccess;
}

}  // namespace a2ats
