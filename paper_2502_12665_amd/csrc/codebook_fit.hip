// Offline codebook construction (section 4.2): the second moment of the rotated queries,
//     H = E[q~^T q~]   (one D x D matrix per KV head; the G query heads of a KV head are pooled),
// and the centroid step of k-means under the query-aware distortion.  The paper runs k-means on
// z = k L and maps the centroids back with L^-1; the mean is linear, so the new codeword is the
// mean of the keys assigned to it, and a Lloyd iteration is a2ats_encode_keys (assignment under
// (k - c) H (k - c)^T) followed by a2ats_codebook_update.  Both geometries: codewords are
// [Hkv][M][L][ds], and a key contributes its subvector m to codeword codes[j][m] of subspace m.
//
//   second_moment_kernel     a workgroup accumulates the outer-product sum of its share of the samples
//                            on the float64 matrix cores, the upper triangle of 16 x 16 tiles
//   second_moment_digits_kernel  the same for many samples, by exact products of 8-bit digits
//   second_moment_sum_kernel adds the partials in a fixed order, divides, rounds once to float32
//   update_clear_kernel      zeroes the float64 sums and the counts
//   update_few_kernel        few keys: one thread per (key, dimension), float64 atomic adds into the sums
//                            (the order of the additions, and so the last bits, vary from run to run)
//   update_add_kernel        product quantiser: the sums of a subspace stay in LDS while a workgroup
//                            walks over its share of the keys, then go to memory by float64 atomic adds
//   update_count_kernel, update_scan_kernel, update_place_kernel
//                            single codebook: the keys of a KV head in the order of their codes
//   update_sorted_kernel     a wave adds up consecutive keys of that order; a codeword all of whose keys it has becomes
//                            their mean
//   update_rest_kernel       the codewords whose keys are several waves', and those without keys
//   update_mean_kernel       the other routes: sum / count, rounded once; codewords without keys keep their value
#include "common.hpp"
#include "internal.hpp"

namespace a2ats {
namespace {

constexpr int kFD = 128;
constexpr int kMomentTiles = 36;   // 16 x 16 tiles on and above the diagonal of 128 x 128
constexpr int kMomentRows = 16;    // sample rows a wave has in flight

// Partial sums per KV head: two workgroups per CU over all heads, as far as the workspace holds them.
inline int moment_parts(int Hkv) { return Hkv < 8 ? 512 / Hkv : 64; }

struct MomentPlan {
  int i[kMomentTiles], j[kMomentTiles];   // tiles row by row, j >= i; wave w takes 9 w .. 9 w + 8
  bool needs[4][8];                       // does wave w read block b of the dimensions
};
constexpr MomentPlan make_moment_plan() {
  MomentPlan p{};
  int t = 0;
  for (int i = 0; i < 8; ++i)
    for (int j = i; j < 8; ++j, ++t) {
      p.i[t] = i;
      p.j[t] = j;
      p.needs[t / 9][i] = p.needs[t / 9][j] = true;
    }
  return p;
}

// Nine tiles of one of the four waves.  Four rows x[k][..] at a time: lane = (k = lane / 16, dimension lane % 16 of
// a block) is the layout of both operands of v_mfma_f64_16x16x4_f64, so one conversion of a loaded float serves
// every tile of its block, as row and as column operand.  Register r of a result: row 4 r + lane / 16, column lane % 16
// of the tile -- or its transpose, which is the same sum.
typedef __attribute__((ext_vector_type(4))) double f64x4;
template <int W>
__device__ __forceinline__ void moment_body(const float* __restrict__ q_rot, int Hq, int G, int kv, uint32_t row0,
                                            uint32_t row1, f64x4 (&acc)[9]) {
  constexpr int kSteps = kMomentRows / 4;
  constexpr MomentPlan P = make_moment_plan();
  const int lane = threadIdx.x & 63, k = lane >> 4, c = lane & 15;
#pragma unroll
  for (int t = 0; t < 9; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
  auto row_at = [&](uint32_t r) { return q_rot + ((size_t)(r / (uint32_t)G) * Hq + (uint32_t)(kv * G) + r % (uint32_t)G) * kFD + c; };
  auto add = [&](const float (&x)[kSteps][8]) {
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {
      double f[8];
#pragma unroll
      for (int b = 0; b < 8; ++b)
        if (P.needs[W][b]) f[b] = (double)x[u][b];
#pragma unroll
      for (int t = 0; t < 9; ++t)
        acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(f[P.i[9 * W + t]], f[P.j[9 * W + t]], acc[t], 0, 0, 0);
    }
  };
  // Whole steps of 16 rows, the next one in flight.  (A vector instruction holds up the float64 products, so the rows'
  // addresses are stepped, not divided out again: 16 / G samples on and 16 % G heads, one more sample where that wraps.)
  const uint32_t n_full = (row1 - row0) / kMomentRows, head_step = kMomentRows % G;
  const ptrdiff_t step = ((ptrdiff_t)(kMomentRows / G) * Hq + head_step) * kFD, wrap = (ptrdiff_t)(Hq - G) * kFD;
  const float* at[kSteps];
  uint32_t head[kSteps];
  float x[kSteps][8];
#pragma unroll
  for (int u = 0; u < kSteps; ++u) {
    const uint32_t r = min(row0 + 4 * u + k, row1 - 1);
    at[u] = row_at(r);
    head[u] = r % (uint32_t)G;
  }
  auto request = [&]() {
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {
#pragma unroll
      for (int b = 0; b < 8; ++b)
        if (P.needs[W][b]) x[u][b] = at[u][16 * b];
      head[u] += head_step;
      const bool over = head[u] >= (uint32_t)G;
      at[u] += over ? step + wrap : step;
      head[u] -= over ? G : 0;
    }
  };
  if (n_full) request();
#pragma unroll 1
  for (uint32_t i = 0; i < n_full; ++i) {
    float now[kSteps][8];
#pragma unroll
    for (int u = 0; u < kSteps; ++u)
#pragma unroll
      for (int b = 0; b < 8; ++b)
        if (P.needs[W][b]) now[u][b] = x[u][b];
    if (i + 1 < n_full) request();   // (uniform)
    __builtin_amdgcn_sched_barrier(0);
    add(now);
  }
  const uint32_t r0 = row0 + n_full * kMomentRows;
  if (r0 < row1) {   // the last rows; those past the end are read as the last one and count as zero
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {
      const float* p = row_at(min(r0 + 4 * u + k, row1 - 1));
#pragma unroll
      for (int b = 0; b < 8; ++b)
        if (P.needs[W][b]) x[u][b] = p[16 * b];
#pragma unroll
      for (int b = 0; b < 8; ++b)
        if (P.needs[W][b]) x[u][b] = r0 + 4 * u + k < row1 ? x[u][b] : 0.f;
    }
    add(x);
  }
}

// use(place in a partial sum, sum) for each of a lane's.
template <int W, typename USE>
__device__ __forceinline__ void for_moments(const f64x4 (&acc)[9], const USE& use) {
  const int lane = threadIdx.x & 63, k = lane >> 4, c = lane & 15;
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) use(((9 * W + t) * 16 + 4 * r + k) * 16 + c, acc[t][r]);
}

// What bounds it: the float64 matrix cores, which run at the vector ALU's rate; what they save are the other half of
// the symmetric sum and the conversions and LDS reads of a register-blocked loop.  50000 samples x 32 heads:
// 1255 -> 505 us.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 3))) void second_moment_kernel(   // (at least 2: else the accumulators travel to AGPRs and back)
    const float* __restrict__ q_rot, double* __restrict__ part, int Hq, int Hkv, uint32_t rows, uint32_t rows_per_part) {
  // rows = n_samples * G row vectors of this KV head: row r is sample r / G, head kv * G + r % G
  const int kv = blockIdx.y, p = blockIdx.x, G = Hq / Hkv;
  const uint32_t row0 = p * rows_per_part, row1 = min(rows, row0 + rows_per_part);   // (host: row0 < rows)
  double* out = part + ((size_t)kv * gridDim.x + p) * (kMomentTiles * 256);
  f64x4 acc[9];
#define A2ATS_WAVE(W)                                                          \
  moment_body<W>(q_rot, Hq, G, kv, row0, row1, acc);                           \
  for_moments<W>(acc, [&](int at, double v) { out[at] = v; })
  switch (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) {
    case 0: A2ATS_WAVE(0); break;
    case 1: A2ATS_WAVE(1); break;
    case 2: A2ATS_WAVE(2); break;
    default: A2ATS_WAVE(3);
  }
#undef A2ATS_WAVE
}

// The same sums by 8-bit integer products, for many samples.  A dimension of a workgroup's rows is taken in units of a power
// of two, as an integer of 48 bits in six signed digits of 8 bits; a product of two digits is added up exactly (32 bits), the
// digits' products that have a weight in common in one sum, and from time to time the six sums go to the float64 partial sum.
// Products of digits a and b with a + b > 5 are left out.
//
// Error: with V a value in units of its upper three digits, |V| <= 2^22 (the first 64 rows get two to three bits of headroom;
// where a later row does not fit, the sums go to memory and the unit grows), V is off by at most 2^-24 and a row's product by
// at most 0.5 from that and 1.26 from what is left out (five pairs of weight 2^-16, of digits up to 2^7).  Usually 0.2, of
// either sign: for normal values 1e-14 of sqrt(H_ii H_jj) over thousands of rows.  That is fine beside products that are
// large against it, and nothing where a few rows are so large that those of all others have no upper digits; so
// the workgroup also adds up the products of the magnitudes of the upper digits, of every fourth step: a quarter of that, times
// 2^32, is no more than the sum of |V_i V_j| over all rows.  Where it shows for every i, j that a stretch of rows (in the same
// units) is off by at most 2^-26 of the sum of |x_i x_j|, half of half an ulp of a float32 result of one sign, the digits' sums
// are taken; else, and where values are not finite, the rows from the first of that stretch on go through the float64 products.
// 4096 rows, a row of 1000 times the usual size for i and another one for j: off by 7e-9 of H_ij without this, 1e6 times: 1e-3.
//
// A wave's tiles of 16 x 16 are those of two blocks of rows and two of columns, so that a digit read from LDS serves two
// products; the waves of a SIMD (w, w + 4) have nine tiles together.  One of them turns the next rows into digits before its
// products, the other after them: so one's vector instructions run beside the other's products.
//
// What bounds it: the matrix cores (756 products of 16 cycles for 64 rows, a wave by itself issues one in 36) and beside
// them, not quite hidden, the rows: 50000 samples x 32 heads 524 us by float64 products, 324 by digits (312 without the upper
// digits' products); without the products, reading and conversion take 186.  8000 samples x 64 KV heads 253 -> 112.  A sample
// 1e5 times the usual size in the middle: 549 and 364.  The vector instructions of the conversion
// between the products, one by one, changed nothing (347), nor did addresses prepared once (325).
constexpr int kDigits = 6, kDigitRows = 64, kDigitThreads = 512;
constexpr int kDigitFrag = 16 * kDigitRows;                      // bytes of one digit of a block of 16 dimensions
constexpr int kDigitBuf = 8 * kDigits * kDigitFrag;
constexpr int kTopEvery = 4, kTopFirst = 8;                      // steps whose upper digits are looked at; after which first
constexpr int kTopMags = 8 * kDigitFrag, kTopSums = kMomentTiles * 256 * 4;   // bytes of their magnitudes, and of the sums
constexpr int kDigitLds = 2 * kDigitBuf + kTopMags + kTopSums;
static_assert(kMomentTiles * 256 * sizeof(double) <= 2 * kDigitBuf, "float64 sums in the digits' place");
constexpr float kDigitLimit = 4194302.f;                         // of a value in units of its upper three digits
constexpr uint32_t kDigitFlushRows = 16384;                      // 6 x 2^14 a row: fits 31 bits
typedef __attribute__((ext_vector_type(4))) int i32x4;

struct DigitGroup {
  int n_row, n_col, row[2], col[2];   // blocks; of a row and a column equal, the tiles on and above the diagonal
};
constexpr DigitGroup digit_group(int wave, int g) {
  constexpr DigitGroup P[8][2] = {
      {{2, 2, {0, 1}, {2, 3}}, {}}, {{2, 2, {0, 1}, {4, 5}}, {}}, {{2, 2, {0, 1}, {6, 7}}, {}}, {{2, 2, {2, 3}, {4, 5}}, {}},
      {{2, 2, {2, 3}, {6, 7}}, {1, 1, {3, 3}, {3, 3}}}, {{2, 2, {4, 5}, {6, 7}}, {1, 1, {7, 7}, {7, 7}}},
      {{2, 2, {0, 1}, {0, 1}}, {1, 2, {2, 2}, {2, 3}}}, {{2, 2, {4, 5}, {4, 5}}, {1, 2, {6, 6}, {6, 7}}}};
  return P[wave][g];
}
constexpr int kDigitTiles = 5;   // of a wave, at most
struct DigitTiles {
  int n, i[kDigitTiles], j[kDigitTiles];
  int at[2][2][2];   // of (group, row, column), -1: none
};
constexpr DigitTiles digit_tiles(int wave) {
  DigitTiles t{};
  for (int g = 0; g < 2; ++g)
    for (int r = 0; r < 2; ++r)
      for (int c = 0; c < 2; ++c) {
        const DigitGroup p = digit_group(wave, g);
        t.at[g][r][c] = -1;
        if (r >= p.n_row || c >= p.n_col || p.row[r] > p.col[c]) continue;
        t.at[g][r][c] = t.n;
        t.i[t.n] = p.row[r];
        t.j[t.n++] = p.col[c];
      }
  return t;
}

struct DigitLds {
  uint32_t most[kFD];      // largest magnitude of a dimension so far (float bits)
  double unit[kFD];
  int32_t flagged, not_finite;   // the step whose rows do not fit; whether any value is not finite
  int32_t coarse;                // whether the digits are too coarse for the products of some i, j
};

template <int W>
__device__ __forceinline__ void digit_products(const uint8_t* buf, i32x4 (&acc)[kDigitTiles][kDigits]) {
  constexpr DigitTiles T = digit_tiles(W);
  const int lane = threadIdx.x & 63;
  auto digit = [&](int block, int a) { return *(const i32x4*)(buf + (block * kDigits + a) * kDigitFrag + lane * 16); };
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    constexpr DigitGroup P0 = digit_group(W, 0), P1 = digit_group(W, 1);
    const DigitGroup& P = g ? P1 : P0;
    i32x4 col[2][kDigits];
#pragma unroll
    for (int c = 0; c < 2; ++c)
      if (c < P.n_col) {
#pragma unroll
        for (int b = 0; b < kDigits; ++b) col[c][b] = digit(P.col[c], b);
      }
    // the rows' digits one after the other, the next one on its way (the fences bound the registers)
    auto row_digit = [&](int at) {
      const int block = P.row[at / kDigits], a = at % kDigits;
      return block == P.col[0] ? col[0][a] : (P.n_col > 1 && block == P.col[1] ? col[1][a] : digit(block, a));
    };
    i32x4 row = {0, 0, 0, 0};
    if (P.n_row) row = row_digit(0);
#pragma unroll
    for (int at = 0; at < 2 * kDigits; ++at)
      if (at < P.n_row * kDigits) {
        const int r = at / kDigits, a = at % kDigits;
        const i32x4 next = at + 1 < P.n_row * kDigits ? row_digit(at + 1) : row;
#pragma unroll
        for (int b = 0; a + b < kDigits; ++b)
#pragma unroll
          for (int c = 0; c < 2; ++c)
            if (T.at[g][r][c] >= 0)
              acc[T.at[g][r][c]][a + b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(row, col[c][b], acc[T.at[g][r][c]][a + b], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        row = next;
      }
  }
}

constexpr int tile_index(int i, int j) { return i * 8 - i * (i - 1) / 2 + j - i; }

// Adds the products of a step's magnitudes to this lane's sums.
template <int W>
__device__ __forceinline__ void top_products(const uint8_t* mags, i32x4* sums) {
  constexpr DigitTiles T = digit_tiles(W);
  const int lane = threadIdx.x & 63;
  i32x4 s[kDigitTiles];   // (read ahead of the stores, which the compiler would not pass)
#pragma unroll
  for (int t = 0; t < kDigitTiles; ++t)
    if (t < T.n) s[t] = sums[tile_index(T.i[t], T.j[t]) * 64 + lane];
#pragma unroll
  for (int t = 0; t < kDigitTiles; ++t)
    if (t < T.n) {
      const i32x4 row = *(const i32x4*)(mags + T.i[t] * kDigitFrag + lane * 16);
      const i32x4 col = *(const i32x4*)(mags + T.j[t] * kDigitFrag + lane * 16);
      s[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(row, col, s[t], 0, 0, 0);
    }
#pragma unroll
  for (int t = 0; t < kDigitTiles; ++t)
    if (t < T.n) sums[tile_index(T.i[t], T.j[t]) * 64 + lane] = s[t];
}

// Whether this lane's sums are large enough for `rows` rows.  (A dimension that has been zero so far has exact products.)
template <int W>
__device__ __forceinline__ bool top_suffices(const i32x4* sums, const DigitLds& L, uint32_t rows) {
  constexpr DigitTiles T = digit_tiles(W);
  const int lane = threadIdx.x & 63;
  bool ok = true;
#pragma unroll
  for (int t = 0; t < kDigitTiles; ++t)
    if (t < T.n) {
      const int i = T.i[t], j = T.j[t];
      const i32x4 s = sums[tile_index(i, j) * 64 + lane];
      const uint4 m = *(const uint4*)&L.most[16 * i + 4 * (lane >> 4)];
      const uint32_t most[4] = {m.x, m.y, m.z, m.w}, col = L.most[16 * j + (lane & 15)];
#pragma unroll
      for (int r = 0; r < 4; ++r) ok &= 8u * (uint32_t)s[r] >= rows || col == 0u || most[r] == 0u;
    }
  return ok;
}

// The sums to the partial sum in memory (`first`: which holds nothing yet).
template <int W>
__device__ __forceinline__ void digit_flush(const i32x4 (&acc)[kDigitTiles][kDigits], const DigitLds& L, double* __restrict__ out,
                                            bool first) {
  constexpr DigitTiles T = digit_tiles(W);
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane), "+s"(out));   // (else the addresses are formed before the loop over the rows, and its registers spilled)
#pragma unroll
  for (int t = 0; t < kDigitTiles; ++t) {
    if (t < T.n) {
      const int i = T.i[t], j = T.j[t], tile = tile_index(i, j);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 4 * (lane >> 4) + r, c = lane & 15;
        double v = (double)acc[t][0][r];
#pragma unroll
        for (int l = 1; l < kDigits; ++l) v = v * 256.0 + (double)acc[t][l][r];
        v *= L.unit[16 * i + row] * L.unit[16 * j + c] * (1.0 / 256.0);
        double* p = out + ((size_t)tile * 16 + row) * 16 + c;
        *p = first ? v : *p + v;
        __builtin_amdgcn_sched_barrier(0);   // (registers)
      }
    }
  }
}

// Wave W of a workgroup (every wave passes the same barriers).
template <int W>
__device__ __forceinline__ void digit_body(const float* __restrict__ q_rot, double* __restrict__ out, int Hq, int kv,
                                           const FastDiv& G, uint32_t row0, uint32_t row1, uint8_t* s_buf, DigitLds& L) {
  const int tid = threadIdx.x;
  // this thread's dimension, and its 16 rows of a step (the same for the wave)
  const int d = tid & (kFD - 1), rg = W >> 1;
  const int n_steps = (int)((row1 - row0 + kDigitRows - 1) / kDigitRows);
  // (a row's address is the same for the wave: the first one of 16 in a buffer descriptor, the others by a scalar offset)
  const int64_t sample_bytes = (int64_t)Hq * kFD * 4;
  const uint32_t wrap_bytes = (uint32_t)(Hq - (int)G.d) * kFD * 4u, small_div = (65535u + G.d) / G.d;   // n / G = n small_div >> 16, n < 4096
  auto load = [&](int step, float (&x)[16]) {
    const uint32_t r0 = row0 + (uint32_t)(step * kDigitRows + rg * 16), in = min(r0, row1 - 1), sample = fast_div(in, G);
    const uint32_t head = in - sample * G.d, last = min(15u, row1 - 1 - in);
    const char* at = (const char*)q_rot + (int64_t)sample * sample_bytes + (int64_t)(kv * (int)G.d + (int)head) * (kFD * 4);
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)at, 0, 0x7fffffff, 0x00027000);
#pragma unroll
    for (int u = 0; u < 16; ++u) {   // (past the last row: that one again)
      const uint32_t n = min((uint32_t)u, last), off = n * (kFD * 4) + ((head + n) * small_div >> 16) * wrap_bytes;
      x[u] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, d * 4, (int)off, 0));
    }
  };
  auto drop_past_end = [&](int step, float (&x)[16]) {   // (when they are used: a load is not waited for before)
    const uint32_t r0 = row0 + (uint32_t)(step * kDigitRows + rg * 16);
    if (r0 + 16 > row1) {   // (uniform over the wave)
#pragma unroll
      for (int u = 0; u < 16; ++u) x[u] = r0 + u < row1 ? x[u] : 0.f;
    }
  };
  auto most_of = [&](const float (&x)[16]) {   // not a number if any of them is not
    float m = 0.f;
#pragma unroll
    for (int u = 0; u < 16; u += 2) asm("v_maximum3_f32 %0, %1, |%2|, |%3|" : "=v"(m) : "v"(m), "v"(x[u]), "v"(x[u + 1]));
    return m;
  };
  float scale = 1.f;
  auto set_scale = [&]() {   // from L.most, between two barriers; the largest value becomes less than 2^20
    const uint32_t bits = L.most[d];
    const int e = bits ? min(max(19 - ((int)(bits >> 23) - 127), -126), 126) : 126;
    scale = __uint_as_float((uint32_t)(127 + e) << 23);
    if (rg == 0) L.unit[d] = (double)__uint_as_float((uint32_t)(127 - e) << 23);
    if (bits >= 0x7f800000u) L.not_finite = 1;
  };
  // Six digits of each of 16 values.  Value times scale = hi + lo 2^-24, hi its nearest integer (23 bits), lo the nearest even
  // one (25 bits): adding 1.5 2^23 (2^24) leaves them in the mantissa.  With 128 added at every digit but the first, digits are
  // bytes, the carry of lo's first goes to hi, and the top bit of those bytes turned makes them signed.
  uint8_t* mags = s_buf + 2 * kDigitBuf;
  i32x4* top_sums = (i32x4*)(mags + kTopMags);   // (a lane's own, as is what it reads of them)
  // top: also the magnitudes of the upper digits, one less for those below zero.
  auto convert = [&](const float (&x)[16], uint8_t* buf, bool top) {
    uint32_t w[kDigits][4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      uint32_t h[4], l[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const float v = x[4 * q + u], hm = __builtin_fmaf(v, scale, 12582912.f), hi = hm - 12582912.f;
        const float rem = __builtin_fmaf(v, scale, -hi), lm = __builtin_fmaf(rem, 16777216.f, 25165824.f);
        l[u] = (__float_as_uint(lm) << 1) + (0x808080u - 0x97800000u);
        h[u] = __float_as_uint(hm) + (0x8080u - 0x4B400000u) + (l[u] >> 24);
      }
      auto transpose = [&](const uint32_t (&t)[4], int a, uint32_t first_sign) {
        const uint32_t p01 = __builtin_amdgcn_perm(t[1], t[0], 0x05010400u), p23 = __builtin_amdgcn_perm(t[3], t[2], 0x05010400u);
        const uint32_t q01 = __builtin_amdgcn_perm(t[1], t[0], 0x0c0c0602u), q23 = __builtin_amdgcn_perm(t[3], t[2], 0x0c0c0602u);
        w[a][q] = __builtin_amdgcn_perm(q23, q01, 0x05040100u) ^ first_sign;
        w[a + 1][q] = __builtin_amdgcn_perm(p23, p01, 0x07060302u) ^ 0x80808080u;
        w[a + 2][q] = __builtin_amdgcn_perm(p23, p01, 0x05040100u) ^ 0x80808080u;
      };
      transpose(h, 0, 0u);
      transpose(l, 3, 0x80808080u);
      __builtin_amdgcn_sched_barrier(0);
    }
    uint8_t* dst = buf + (d >> 4) * (kDigits * kDigitFrag) + ((d & 15) + 16 * rg) * 16;
#pragma unroll
    for (int a = 0; a < kDigits; ++a) *(uint4*)(dst + a * kDigitFrag) = make_uint4(w[a][0], w[a][1], w[a][2], w[a][3]);
    if (top) {   // (uniform)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint32_t below = w[0][q] & 0x80808080u;
        w[0][q] ^= (below << 1) - (below >> 7);   // (all bits of those bytes)
      }
      *(uint4*)(mags + (d >> 4) * kDigitFrag + ((d & 15) + 16 * rg) * 16) = make_uint4(w[0][0], w[0][1], w[0][2], w[0][3]);
    }
  };
  auto clear_top = [&]() {
    constexpr DigitTiles T = digit_tiles(W);
#pragma unroll
    for (int t = 0; t < kDigitTiles; ++t)
      if (t < T.n) top_sums[tile_index(T.i[t], T.j[t]) * 64 + (tid & 63)] = i32x4{0, 0, 0, 0};
  };
  auto fine_enough = [&](int steps) {
    if (!top_suffices<W>(top_sums, L, (uint32_t)steps * kDigitRows)) L.coarse = 1;
    __syncthreads();
    return L.coarse == 0;
  };
  float x[16], most;
  if (tid < kFD) L.most[tid] = 0u;
  if (tid == 0) {
    L.flagged = -1;
    L.not_finite = 0;
    L.coarse = 0;
  }
  load(0, x);
  drop_past_end(0, x);
  __syncthreads();
  atomicMax(&L.most[d], __float_as_uint(most_of(x)) & 0x7fffffffu);
  __syncthreads();
  set_scale();
  convert(x, s_buf, true);
  load(min(1, n_steps - 1), x);
  __syncthreads();
  bool good = L.not_finite == 0, first = true;
  int step = 0, start = 0;   // what comes before row `start` is in the partial sum
#pragma unroll 1
  while (good && step < n_steps) {   // (uniform, as the conditions below) a stretch of rows in the same units
    i32x4 acc[kDigitTiles][kDigits];
#pragma unroll
    for (int t = 0; t < kDigitTiles; ++t)
#pragma unroll
      for (int l = 0; l < kDigits; ++l) acc[t][l] = i32x4{0, 0, 0, 0};
    clear_top();
    const int stop = min(n_steps, step + (int)(kDigitFlushRows / kDigitRows));
    bool fits = true;
#pragma unroll 1
    do {
      const uint8_t* now = s_buf + (step & 1) * kDigitBuf;
      uint8_t* next = s_buf + ((step + 1) & 1) * kDigitBuf;
      const bool more = step + 1 < n_steps;
      auto prepare_next = [&]() {
        drop_past_end(step + 1, x);
        most = most_of(x);
        convert(x, next, (step + 1 - start) % kTopEvery == 0);
        if (!(most * scale <= kDigitLimit)) L.flagged = step + 1;
        load(min(step + 2, n_steps - 1), x);
      };
      if (W < 4 && more) prepare_next();
      digit_products<W>(now, acc);
      if ((step - start) % kTopEvery == 0) top_products<W>(mags, top_sums);
      if (W >= 4 && more) prepare_next();
      __syncthreads();
      ++step;
      fits = L.flagged != step;
      if (fits && step - start == kTopFirst && stop - step >= kTopFirst) good = fine_enough(kTopFirst);
    } while (fits && good && step < stop);
    if (!good || !(good = fine_enough(step - start))) break;
    digit_flush<W>(acc, L, out, first);
    first = false;
    start = step;
    if (!fits) {   // a larger unit from here on
      __syncthreads();   // (the units have been read)
      atomicMax(&L.most[d], __float_as_uint(most) & 0x7fffffffu);
      __syncthreads();
      set_scale();
      float again[16];
      load(step, again);
      drop_past_end(step, again);
      convert(again, s_buf + (step & 1) * kDigitBuf, true);
      __syncthreads();
      good = L.not_finite == 0;
    }
  }
  if (start == n_steps) return;
  // what is left, by float64 products: one half of the rows each for waves 0 to 3 and 4 to 7
  const uint32_t from = row0 + (uint32_t)(start * kDigitRows), mid = from + (row1 - from + 1) / 2;
  f64x4 sums[9];
  moment_body<W & 3>(q_rot, Hq, (int)G.d, kv, W < 4 ? from : mid, W < 4 ? mid : row1, sums);
  double* other = (double*)s_buf;
  if (W >= 4) for_moments<W & 3>(sums, [&](int at, double v) { other[at] = v; });
  __syncthreads();
  if (W < 4)
    for_moments<W & 3>(sums, [&](int at, double v) {
      v += other[at];
      out[at] = first ? v : out[at] + v;
    });
}

__global__ __launch_bounds__(kDigitThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void second_moment_digits_kernel(
    const float* __restrict__ q_rot, double* __restrict__ part, int Hq, int Hkv, FastDiv G, uint32_t rows,
    uint32_t rows_per_part) {
  extern __shared__ __align__(16) uint8_t s_buf[];   // two buffers of digits, the upper digits' magnitudes and sums, DigitLds
  DigitLds& L = *(DigitLds*)(s_buf + kDigitLds);
  const int kv = blockIdx.y, p = blockIdx.x;
  const uint32_t row0 = p * rows_per_part, row1 = min(rows, row0 + rows_per_part);   // (host: row0 < rows)
  double* out = part + ((size_t)kv * gridDim.x + p) * (kMomentTiles * 256);
#define A2ATS_WAVE(W) \
  case W: digit_body<W>(q_rot, out, Hq, kv, G, row0, row1, s_buf, L); break
  switch (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) {
    A2ATS_WAVE(0);
    A2ATS_WAVE(1);
    A2ATS_WAVE(2);
    A2ATS_WAVE(3);
    A2ATS_WAVE(4);
    A2ATS_WAVE(5);
    A2ATS_WAVE(6);
    A2ATS_WAVE(7);
    default: break;
  }
#undef A2ATS_WAVE
}

__global__ __launch_bounds__(256) void second_moment_sum_kernel(const double* __restrict__ part, float* __restrict__ h,
                                                                double inv_rows, int n_parts) {
  const int kv = blockIdx.y, t = blockIdx.x, e = threadIdx.x;   // an element of tile t
  const double* p = part + (size_t)kv * n_parts * (kMomentTiles * 256) + t * 256 + e;
  double s = 0.0;
#pragma unroll 8
  for (int i = 0; i < n_parts; ++i) s += p[(size_t)i * (kMomentTiles * 256)];
  const float v = (float)(s * inv_rows);
  int bi = 0, bj = t;
  while (bj >= 8 - bi) bj -= 8 - bi++;
  bj += bi;
  const int i = 16 * bi + (e >> 4), j = 16 * bj + (e & 15);
  float* o = h + (size_t)kv * kFD * kFD;
  o[(size_t)i * kFD + j] = v;
  if (bi != bj) o[(size_t)j * kFD + i] = v;   // (a diagonal tile holds both)
}

__global__ void update_clear_kernel(double* __restrict__ sums, uint32_t* __restrict__ counts, size_t n_sums,
                                    size_t n_counts) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_sums; i += (size_t)gridDim.x * blockDim.x)
    sums[i] = 0.0;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_counts; i += (size_t)gridDim.x * blockDim.x)
    counts[i] = 0u;
}

template <typename CODE>
__global__ __launch_bounds__(256) void update_few_kernel(const float* __restrict__ keys, const CODE* __restrict__ codes,
                                                         double* __restrict__ sums, uint32_t* __restrict__ counts,
                                                         int Hkv, int M, int L, int ds, int n_new, int pos0,
                                                         int64_t ctx_stride) {
  const int bkv = blockIdx.y, kv = bkv % Hkv, tid = threadIdx.x;
  const long j = (long)blockIdx.x * 2 + (tid >> 7);   // two keys per workgroup
  const int t = tid & 127;
  if (j >= n_new) return;
  const int m = t / ds;
  const int c = (int)codes[((size_t)bkv * ctx_stride + pos0 + j) * M + m] & (L - 1);   // L is a power of two
  const size_t cw = ((size_t)kv * M + m) * L + c;
  unsafeAtomicAdd(&sums[cw * ds + t % ds], (double)keys[((size_t)bkv * n_new + j) * kFD + t]);
  if (t % ds == 0) atomicAdd(&counts[cw], 1u);
}

// Product quantiser.  A workgroup takes kAddSub subspaces (64 dimensions at ds = 8, 32 at ds = 4) of a share of the
// keys of a KV head; their sums fill 128 KB (64 KB) of LDS.  What bounds it: the LDS atomics; in memory every key would
// cost 128 float64 atomics (24001 keys x 32: M = 16 1056 -> 239 us, M = 32 1950 -> 240 us).
constexpr int kAddThreads = 1024, kAddSub = 8;
template <int DS>
__global__ __launch_bounds__(kAddThreads) void update_add_kernel(const float* __restrict__ keys,
                                                                 const uint8_t* __restrict__ codes,
                                                                 double* __restrict__ sums, uint32_t* __restrict__ counts,
                                                                 int B, int Hkv, int M, int n_new, int pos0,
                                                                 int64_t ctx_stride, long rows_per_wg) {
  constexpr int L = 256, kRow = kAddSub * DS, kPerStep = kAddThreads / kRow;   // floats of a key, keys per step
  extern __shared__ double s_sum[];              // [subspace][code][ds]
  uint32_t* s_n = (uint32_t*)(s_sum + kAddSub * L * DS);   // [subspace][code]
  const int kv = blockIdx.z, sub0 = blockIdx.y * kAddSub, tid = threadIdx.x;
  for (int i = tid; i < kAddSub * L * DS; i += kAddThreads) s_sum[i] = 0.0;
  for (int i = tid; i < kAddSub * L; i += kAddThreads) s_n[i] = 0u;
  __syncthreads();
  const long rows = (long)B * n_new;   // of the KV head: row r is key r % n_new of sequence r / n_new
  const long r0 = blockIdx.x * rows_per_wg, r1 = min(rows, r0 + rows_per_wg);
  const int e = tid % kRow, sub = e / DS, t = e % DS;
#pragma unroll 4
  for (long r = r0 + tid / kRow; r < r1; r += kPerStep) {
    const uint32_t b = (uint32_t)r / (uint32_t)n_new, j = (uint32_t)r % (uint32_t)n_new;   // (rows < 2^31)
    const size_t bkv = (size_t)b * Hkv + kv;
    const int c = codes[(bkv * ctx_stride + pos0 + j) * M + sub0 + sub];
    const float x = keys[(bkv * n_new + j) * kFD + sub0 * DS + e];
    unsafeAtomicAdd(&s_sum[(sub * L + c) * DS + t], (double)x);
    if (t == 0) atomicAdd(&s_n[sub * L + c], 1u);
  }
  __syncthreads();
  const size_t cw0 = ((size_t)kv * M + sub0) * L;
  for (int i = tid; i < kAddSub * L * DS; i += kAddThreads)
    if (s_n[i / DS]) unsafeAtomicAdd(&sums[cw0 * DS + i], s_sum[i]);
  for (int i = tid; i < kAddSub * L; i += kAddThreads)
    if (s_n[i]) atomicAdd(&counts[cw0 + i], s_n[i]);
}

// Single codebook: 4096 codewords of 128 dimensions do not fit LDS, but the keys can be read in the order of their codes.
// The keys of a KV head are cut into slices, of which a workgroup counts the codes in LDS; from the counts
// hist[kv][slice][c] follow the first place start[kv][c] of a code and, in the place of the counts, that of a slice's keys of
// it; a workgroup then puts the keys of its slice there: order[kv][place] = (row, code).  768032 keys, 8 KV heads, all three
// 28 us; 52 with a counter per codeword in memory, to be cleared first, whose atomics return a key's rank.  16 slices a KV
// head, which the scan reads at once, and 32 where they are long, whatever the number of heads: the whole update with 16, 24,
// 32, 48, one KV head, 300000 keys 66 us, 67, 67, 72, 800000 169, 159, 153, 153 (163 with the counters in memory); 2 heads of
// 400000 144, 142, 142, 145; 4 of 200000 132, 133, 136, 141; 8 of 200000 226, 230, 233, 240.
constexpr int kFL = 4096, kOrderThreads = 1024;
struct OrderSlices {
  int n;        // per KV head
  long per;     // rows of one
};
inline OrderSlices order_slices(long rows) {   // (at most as many as a word per row holds counts of, but at least one)
  OrderSlices s;
  const long most = rows >= 400000 ? 32 : 16;
  s.n = (int)(rows / kFL < 1 ? 1 : (rows / kFL > most ? most : rows / kFL));
  s.per = (rows + s.n - 1) / s.n;
  return s;
}

// use(row, code) for every key of the workgroup's slice: row r of a KV head is key r % n_new of sequence r / n_new.
template <typename USE>
__device__ __forceinline__ void for_slice(const uint16_t* __restrict__ codes, int Hkv, int n_new, int pos0,
                                          int64_t ctx_stride, long rows, long per, const USE& use) {
  const int kv = blockIdx.y;
  const long r0 = blockIdx.x * per, r1 = min(rows, r0 + per);
#pragma unroll 4
  for (long r = r0 + threadIdx.x; r < r1; r += kOrderThreads) {
    const uint32_t b = (uint32_t)r / (uint32_t)n_new, j = (uint32_t)r % (uint32_t)n_new;
    const size_t bkv = (size_t)b * Hkv + kv;
    use((uint32_t)(bkv * n_new + j), codes[bkv * ctx_stride + pos0 + j] & (uint32_t)(kFL - 1));
  }
}

__global__ __launch_bounds__(kOrderThreads) void update_count_kernel(const uint16_t* __restrict__ codes,
                                                                     uint32_t* __restrict__ hist, int Hkv, int n_new,
                                                                     int pos0, int64_t ctx_stride, long rows, long per) {
  __shared__ uint32_t s_n[kFL];
  for (int i = threadIdx.x; i < kFL; i += kOrderThreads) s_n[i] = 0u;
  __syncthreads();
  for_slice(codes, Hkv, n_new, pos0, ctx_stride, rows, per, [&](uint32_t, uint32_t c) { atomicAdd(&s_n[c], 1u); });
  __syncthreads();
  uint32_t* out = hist + ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * kFL;
  for (int i = threadIdx.x; i < kFL; i += kOrderThreads) out[i] = s_n[i];
}

constexpr int kScanAhead = 16;   // slices whose counts are on their way together
// With one slice `hist` is `counts`, and the slice's first places are `start`.
__global__ __launch_bounds__(1024) void update_scan_kernel(uint32_t* hist, uint32_t* counts, uint32_t* __restrict__ start,
                                                           int slices) {
  __shared__ uint32_t s_wave[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint4* mine = (uint4*)(hist + (size_t)blockIdx.x * slices * kFL) + tid;   // four codes, kFL / 4 apart by slice
  uint4 n = make_uint4(0u, 0u, 0u, 0u), h[kScanAhead];
  auto request = [&](int s0) {   // (conditions on slices are uniform)
#pragma unroll
    for (int u = 0; u < kScanAhead; ++u)
      if (s0 + u < slices) h[u] = mine[(size_t)(s0 + u) * (kFL / 4)];
  };
  for (int s0 = 0; s0 < slices; s0 += kScanAhead) {
    request(s0);
#pragma unroll
    for (int u = 0; u < kScanAhead; ++u)
      if (s0 + u < slices) n = make_uint4(n.x + h[u].x, n.y + h[u].y, n.z + h[u].z, n.w + h[u].w);
  }
  const uint32_t own = n.x + n.y + n.z + n.w;
  uint32_t inc = own;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t o = __shfl_up(inc, off);
    if (lane >= off) inc += o;
  }
  if (lane == 63) s_wave[wave] = inc;
  __syncthreads();
  uint32_t before = inc - own;
  for (int w = 0; w < wave; ++w) before += s_wave[w];
  uint4 at = make_uint4(before, before + n.x, before + n.x + n.y, before + n.x + n.y + n.z);
  ((uint4*)(counts + (size_t)blockIdx.x * kFL))[tid] = n;
  ((uint4*)(start + (size_t)blockIdx.x * kFL))[tid] = at;
  if (slices == 1) return;
  for (int s0 = 0; s0 < slices; s0 += kScanAhead) {
    if (slices > kScanAhead) request(s0);   // (else they are still there)
#pragma unroll
    for (int u = 0; u < kScanAhead; ++u)
      if (s0 + u < slices) {
        mine[(size_t)(s0 + u) * (kFL / 4)] = at;
        at = make_uint4(at.x + h[u].x, at.y + h[u].y, at.z + h[u].z, at.w + h[u].w);
      }
  }
}

__global__ __launch_bounds__(kOrderThreads) void update_place_kernel(const uint16_t* __restrict__ codes,
                                                                     const uint32_t* __restrict__ first,
                                                                     uint2* __restrict__ order, int Hkv, int n_new,
                                                                     int pos0, int64_t ctx_stride, long rows, long per) {
  __shared__ uint32_t s_at[kFL];
  const uint32_t* in = first + ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * kFL;
  for (int i = threadIdx.x; i < kFL; i += kOrderThreads) s_at[i] = in[i];
  __syncthreads();
  uint2* out = order + (size_t)blockIdx.y * rows;
  for_slice(codes, Hkv, n_new, pos0, ctx_stride, rows, per,
            [&](uint32_t row, uint32_t c) { out[atomicAdd(&s_at[c], 1u)] = make_uint2(row, c); });   // (512 bytes a key: fewer than 2^32 rows fit the card)
}

// A wave takes `chunk` consecutive keys of the order, two dimensions per lane, and adds up every run of equal codes.  A run
// that holds all keys of its codeword becomes the mean at once; of the others, the one that goes on from the wave before and
// the one that goes on into the next, the sums are left in the wave's two places for update_rest_kernel.  So no sums are
// cleared, added to or read again in memory.  What bounds it: reading the keys, 512 bytes at a time in no order of theirs
// (768032 keys, 8 KV heads: 80 us, 4.9 TB/s, and 6 for the rest; 104 with atomics of every run and a division of all sums).
// Chunks: 64 keys, and 128 where that still makes the waves that keep the memory busy (fewer runs are cut); longer only where
// the places would not fit the sums' part of the workspace.
constexpr int kPlaces = 2048;   // waves per KV head whose places fit there
inline int sum_chunk(long rows, int Hkv) {
  const long fits = (rows + 64L * kPlaces - 1) / (64L * kPlaces), busy = rows * Hkv >= 300000 ? 2 : 1;
  return (int)(64 * (fits > busy ? fits : busy));
}

__global__ __launch_bounds__(256) void update_sorted_kernel(const float* __restrict__ keys, const uint2* __restrict__ order,
                                                            double* __restrict__ sums, float* __restrict__ new_cb, long rows,
                                                            int chunk) {
  const int kv = blockIdx.y, lane = threadIdx.x & 63;
  const long w = (long)blockIdx.x * 4 + (threadIdx.x >> 6), first = w * chunk;
  if (first >= rows) return;
  const long last = min(rows, first + chunk);   // (uniform in the wave, as all that follows)
  const uint2* ord = order + (size_t)kv * rows;
  double* places = sums + ((size_t)kv * kPlaces + w) * 2 * kFD + 2 * lane;
  float* out = new_cb + (size_t)kv * kFL * kFD + 2 * lane;
  const uint32_t none = ~0u;
  const uint32_t code_before = first > 0 ? __builtin_amdgcn_readfirstlane(ord[first - 1].y) : none;
  const uint32_t code_after = last < rows ? __builtin_amdgcn_readfirstlane(ord[last].y) : none;
  double a0 = 0.0, a1 = 0.0;
  uint32_t run = __builtin_amdgcn_readfirstlane(ord[first].y), n_run = 0;
  bool cut = run == code_before;   // the run has keys in the wave before
  auto finish = [&](bool goes_on) {
    if (cut || goes_on) {
      *(double2*)(places + (cut ? 0 : kFD)) = make_double2(a0, a1);
    } else {
      out[(size_t)run * kFD] = (float)(a0 / (double)n_run);
      out[(size_t)run * kFD + 1] = (float)(a1 / (double)n_run);
    }
  };
  constexpr int U = 8;
#pragma unroll 1
  for (long p = first; p < last; p += 64) {
    const int n = (int)min(64L, last - p);
    const uint2 mine = ord[p + min(lane, n - 1)];
#pragma unroll 1
    for (int i0 = 0; i0 < n; i0 += U) {
      float2 x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t row = __builtin_amdgcn_readlane(mine.x, min(i0 + u, n - 1));
        x[u] = *(const float2*)(keys + (size_t)row * kFD + 2 * lane);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (i0 + u >= n) break;
        const uint32_t c = __builtin_amdgcn_readlane(mine.y, i0 + u);
        if (c != run) {
          finish(false);
          a0 = a1 = 0.0;
          run = c;
          n_run = 0;
          cut = false;
        }
        a0 += (double)x[u].x;
        a1 += (double)x[u].y;
        ++n_run;
      }
    }
  }
  finish(run == code_after);
}

// The codewords whose keys more than one wave added up, those without keys, and the counts: four codewords a wave, one after the
// other (48000 keys of one KV head 31.3 -> 29.9 us against 16 a wave, 800000 152.9 -> 150.4).
constexpr int kRestPerWave = 4;
__global__ __launch_bounds__(256) void update_rest_kernel(const double* __restrict__ sums, const uint32_t* __restrict__ counts,
                                                          const uint32_t* __restrict__ start, const float* __restrict__ old_cb,
                                                          float* __restrict__ new_cb, int32_t* __restrict__ counts_out,
                                                          int chunk) {
  const int kv = blockIdx.y, lane = threadIdx.x & 63;
  const int c0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * kRestPerWave;
  const size_t cw = (size_t)kv * kFL + c0 + lane % kRestPerWave;
  const uint32_t n = counts[cw], at = start[cw];
  if (counts_out && lane < kRestPerWave) counts_out[cw] = (int32_t)n;
  const uint32_t w0 = at / (uint32_t)chunk, w1 = n ? (at + n - 1) / (uint32_t)chunk : w0;
  uint64_t todo = __builtin_amdgcn_ballot_w64(lane < kRestPerWave && (n == 0 || w1 > w0));
  while (todo) {   // (uniform)
    const int i = (int)__builtin_ctzll(todo);
    todo &= todo - 1;
    const uint32_t ni = __builtin_amdgcn_readlane(n, i), a = __builtin_amdgcn_readlane(w0, i), z = __builtin_amdgcn_readlane(w1, i);
    const size_t o = ((size_t)kv * kFL + c0 + i) * kFD + 2 * lane;
    if (ni == 0) {
      new_cb[o] = old_cb[o];   // (codebooks are aligned to their elements, no more)
      new_cb[o + 1] = old_cb[o + 1];
      continue;
    }
    const double* places = sums + (size_t)kv * kPlaces * 2 * kFD + 2 * lane;
    double2 s = *(const double2*)(places + ((size_t)a * 2 + 1) * kFD);
#pragma unroll 8
    for (uint32_t w = a + 1; w <= z; ++w) {
      const double2 x = *(const double2*)(places + (size_t)w * 2 * kFD);
      s.x += x.x;
      s.y += x.y;
    }
    new_cb[o] = (float)(s.x / (double)ni);
    new_cb[o + 1] = (float)(s.y / (double)ni);
  }
}

__global__ __launch_bounds__(256) void update_mean_kernel(const double* __restrict__ sums,
                                                          const uint32_t* __restrict__ counts,
                                                          const float* __restrict__ old_cb, float* __restrict__ new_cb,
                                                          int32_t* __restrict__ counts_out, int ds, size_t n_elems) {
  const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= n_elems) return;
  const size_t cw = e / ds;
  const uint32_t n = counts[cw];
  new_cb[e] = n ? (float)(sums[e] / (double)n) : old_cb[e];
  if (counts_out && e % ds == 0) counts_out[cw] = (int32_t)n;
}

}  // namespace

struct FitWs {
  size_t off_counts, off_start, off_hist, off_order, update_bytes;   // of the update; its sums come first
  size_t bytes;
};
// The second moment is taken from digits where the rows are more than a step for each CU (its look at the upper digits pays
// from the second on): float64 -> digits, 16500 rows of one KV head 41.9 -> 30.9 us, 8000 26.9 -> 28.8; 8 KV heads, 2400 rows each
// 27.6 -> 22.6, 2048 22.2 -> 24.5; 4 of 4200 28.7 -> 22.1.  And from 2048 rows of a KV head: fewer leave more of a digit sum's
// error in the mean.
inline bool moment_by_digits(long rows, int Hkv) { return rows >= 2048 && rows * Hkv > 256L * kDigitRows; }
constexpr size_t kMomentPart = kMomentTiles * 256 * sizeof(double);   // a partial sum of the second moment
static FitWs fit_ws(const a2ats_dims& d) {
  const size_t cws = (size_t)d.n_kv_heads * d.n_sub * d.n_centroids;
  size_t o = 0;
  auto take = [&](size_t bytes) {
    const size_t at = o;
    o += (bytes + 255) & ~(size_t)255;
    return at;
  };
  FitWs w;
  take(cws * d.sub_dim * sizeof(double));
  w.off_counts = take(cws * sizeof(uint32_t));
  const bool single = single_codebook(d);
  w.off_start = take(single ? cws * sizeof(uint32_t) : 0);
  w.off_hist = take(single ? (size_t)d.batch * d.n_kv_heads * (size_t)d.ctx_stride * sizeof(uint32_t) : 0);
  w.off_order = take(single ? (size_t)d.batch * d.n_kv_heads * (size_t)d.ctx_stride * sizeof(uint2) : 0);
  w.update_bytes = o;
  const size_t moment = (size_t)d.n_kv_heads * moment_parts(d.n_kv_heads) * kMomentPart;
  w.bytes = ((moment > o ? moment : o) + 255) & ~(size_t)255;
  return w;
}

size_t fit_ws_bytes(const a2ats_dims& d) { return fit_ws(d).bytes; }

// What either call can do with: 113 partial sums per KV head, or the sums and counts of the update (4.3 MB at most).
size_t fit_ws_least_bytes(const a2ats_dims& d) {
  const size_t least = (size_t)d.n_kv_heads << 23, all = fit_ws(d).bytes;
  return least < all ? least : all;
}

hipError_t launch_second_moment(const a2ats_dims& d, const float* q_rot, int64_t n_samples, float* h_out, void* ws,
                                size_t ws_bytes, hipStream_t stream) {
  if (d.n_kv_heads == 0) return hipSuccess;
  const int G = d.n_q_heads / d.n_kv_heads;
  const long rows = (long)n_samples * G;   // (512 bytes each: fewer than 2^32 fit the card)
  // at least 64 rows a workgroup: the partials are 72 KB each
  const long held = (long)(ws_bytes / kMomentPart) / d.n_kv_heads, wanted = moment_parts(d.n_kv_heads);
  long most = held < wanted ? held : wanted;
  const bool digits = moment_by_digits(rows, d.n_kv_heads);
  if (digits && most > 256 / d.n_kv_heads && d.n_kv_heads <= 256) most = 256 / d.n_kv_heads;   // one workgroup a CU
  long per = (rows + most - 1) / most;
  per = ((per < 64 ? 64 : per) + kDigitRows - 1) / kDigitRows * kDigitRows;
  const int parts = (int)((rows + per - 1) / per);
  hipError_t e;
  if (digits) {
    const size_t lds = kDigitLds + sizeof(DigitLds);
    static LdsSlot s_lds[16];
    if ((e = allow_dynamic_lds(second_moment_digits_kernel, lds, s_lds)) != hipSuccess) return e;
    hipLaunchKernelGGL(second_moment_digits_kernel, dim3(parts, d.n_kv_heads), dim3(kDigitThreads), lds, stream, q_rot,
                       (double*)ws, d.n_q_heads, d.n_kv_heads, make_fastdiv((uint32_t)G), (uint32_t)rows, (uint32_t)per);
  } else if (parts > 0) {
    hipLaunchKernelGGL(second_moment_kernel, dim3(parts, d.n_kv_heads), dim3(256), 0, stream, q_rot, (double*)ws,
                       d.n_q_heads, d.n_kv_heads, (uint32_t)rows, (uint32_t)per);
  }
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  hipLaunchKernelGGL(second_moment_sum_kernel, dim3(kMomentTiles, d.n_kv_heads), dim3(256), 0, stream,
                     (const double*)ws, h_out, rows > 0 ? 1.0 / (double)rows : 0.0, parts);
  return hipGetLastError();
}

hipError_t launch_codebook_update(const a2ats_dims& d, const float* keys, int n_new, int pos0, const void* codes,
                                  const float* codebook, float* codebook_out, int32_t* counts_out, void* ws,
                                  size_t ws_bytes, hipStream_t stream) {
  const size_t cws = (size_t)d.n_kv_heads * d.n_sub * d.n_centroids, n_elems = cws * d.sub_dim;
  if (n_elems == 0) return hipSuccess;
  const FitWs w = fit_ws(d);
  uint8_t* base = (uint8_t*)ws;
  double* sums = (double*)base;
  uint32_t* counts = (uint32_t*)(base + w.off_counts);
  const int Hkv = d.n_kv_heads, bkv = d.batch * Hkv;
  const long rows = (long)d.batch * n_new, n_keys = rows * Hkv;
  // Few keys are added one by one: below these counts the further launches, or filling and emptying the sums in LDS,
  // cost more than the atomics they save (one by one -> otherwise, us: single codebook 16000 keys 33 -> 50, 20000 24 ->
  // 29, 80000 75 -> 51; M = 16, 8000 keys 18 -> 21, 16000 29 -> 24; M = 32, 2000 keys 13 -> 14, 8000 28 -> 15).
  // So are those of a single codebook whose order the workspace has no room for.
  const bool one_by_one = n_keys < (single_codebook(d) ? 48000 : 192000 / d.n_sub) || (single_codebook(d) && ws_bytes < w.update_bytes);
  hipError_t err;
  if (n_keys > 0 && single_codebook(d) && !one_by_one) {
    uint32_t* start = (uint32_t*)(base + w.off_start);
    uint2* order = (uint2*)(base + w.off_order);
    const uint16_t* c16 = (const uint16_t*)codes;
    const OrderSlices sl = order_slices(rows);
    uint32_t* hist = sl.n > 1 ? (uint32_t*)(base + w.off_hist) : counts;
    const int chunk = sum_chunk(rows, Hkv);
    const long waves = (rows + chunk - 1) / chunk;
    hipLaunchKernelGGL(update_count_kernel, dim3(sl.n, Hkv), dim3(kOrderThreads), 0, stream, c16, hist, Hkv, n_new, pos0,
                       d.ctx_stride, rows, sl.per);
    if ((err = hipGetLastError()) != hipSuccess) return err;
    hipLaunchKernelGGL(update_scan_kernel, dim3(Hkv), dim3(1024), 0, stream, hist, counts, start, sl.n);
    if ((err = hipGetLastError()) != hipSuccess) return err;
    hipLaunchKernelGGL(update_place_kernel, dim3(sl.n, Hkv), dim3(kOrderThreads), 0, stream, c16, sl.n > 1 ? hist : start, order,
                       Hkv, n_new, pos0, d.ctx_stride, rows, sl.per);
    if ((err = hipGetLastError()) != hipSuccess) return err;
    hipLaunchKernelGGL(update_sorted_kernel, dim3((unsigned)((waves + 3) / 4), Hkv), dim3(256), 0, stream, keys, order, sums,
                       codebook_out, rows, chunk);
    if ((err = hipGetLastError()) != hipSuccess) return err;
    hipLaunchKernelGGL(update_rest_kernel, dim3(kFL / (4 * kRestPerWave), Hkv), dim3(256), 0, stream, sums, counts, start,
                       codebook, codebook_out, counts_out, chunk);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(update_clear_kernel, dim3(1024), dim3(256), 0, stream, sums, counts, n_elems, cws);
  if ((err = hipGetLastError()) != hipSuccess) return err;
  if (n_new > 0 && d.batch > 0 && one_by_one) {
    const dim3 grid((n_new + 1) / 2, bkv);
    if (single_codebook(d))
      hipLaunchKernelGGL(update_few_kernel<uint16_t>, grid, dim3(256), 0, stream, keys, (const uint16_t*)codes, sums,
                         counts, Hkv, d.n_sub, d.n_centroids, d.sub_dim, n_new, pos0, d.ctx_stride);
    else
      hipLaunchKernelGGL(update_few_kernel<uint8_t>, grid, dim3(256), 0, stream, keys, (const uint8_t*)codes, sums,
                         counts, Hkv, d.n_sub, d.n_centroids, d.sub_dim, n_new, pos0, d.ctx_stride);
    if ((err = hipGetLastError()) != hipSuccess) return err;
  } else if (n_new > 0 && d.batch > 0) {
    // One workgroup per CU: as many shares of the keys as fill the CUs once, of 512 keys or more (a share ends with
    // up to 16384 atomics).
    const long groups = (long)Hkv * (d.n_sub / kAddSub);
    const long shares = groups < 256 ? 256 / groups : 1;
    long per = (rows + shares - 1) / shares;
    if (per < 512) per = 512;
    const dim3 grid((unsigned)((rows + per - 1) / per), d.n_sub / kAddSub, Hkv);
    const size_t lds = (size_t)kAddSub * 256 * (d.sub_dim * sizeof(double) + sizeof(uint32_t));
    static LdsSlot s_lds[2][16];
    if (d.sub_dim == 8) {
      if ((err = allow_dynamic_lds(update_add_kernel<8>, lds, s_lds[0])) != hipSuccess) return err;
      hipLaunchKernelGGL(update_add_kernel<8>, grid, dim3(kAddThreads), lds, stream, keys, (const uint8_t*)codes, sums,
                         counts, d.batch, Hkv, d.n_sub, n_new, pos0, d.ctx_stride, per);
    } else {
      if ((err = allow_dynamic_lds(update_add_kernel<4>, lds, s_lds[1])) != hipSuccess) return err;
      hipLaunchKernelGGL(update_add_kernel<4>, grid, dim3(kAddThreads), lds, stream, keys, (const uint8_t*)codes, sums,
                         counts, d.batch, Hkv, d.n_sub, n_new, pos0, d.ctx_stride, per);
    }
    if ((err = hipGetLastError()) != hipSuccess) return err;
  }
  hipLaunchKernelGGL(update_mean_kernel, dim3((unsigned)((n_elems + 255) / 256)), dim3(256), 0, stream, sums, counts,
                     codebook, codebook_out, counts_out, d.sub_dim, n_elems);
  return hipGetLastError();
}

}  // namespace a2ats
