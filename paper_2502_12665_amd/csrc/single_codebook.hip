// The paper's own vector-quantisation geometry (section 5.1): ONE codebook of 4096 codewords per
// head over all D = 128 dimensions (M = 1), a 16-bit code per token.  The approximate score of a
// token is then a single table entry, u^_j = q~ . C[s_j] (section 2.2 eq. "attention weights
// approximation", section 4.2 last equation), so the code stream is 2 bytes per token and there
// are at most 4096 distinct scores per head: selection is dominated by exact ties.
//
//   build_lut_single_kernel    q~ = q R_b and the 4096 scores q~ . c per head, float64 inner
//                              products rounded once to float32 and stored as order-preserving
//                              32-bit keys (no fixed-point scale is needed: a score is one entry);
//                              in other workgroups the same sweep for a few appended keys, and the
//                              candidates per codeword
//   select_chunks_single_kernel  exact top-K of a head from those counts, by a workgroup per chunk of
//                              the sequence (a2ats_decode_select)
//   select_single_kernel       exact top-K per head without them: candidates counted per codeword, a
//                              weighted selection over the 4096 codewords, then one ordered pass that
//                              emits the winners in ascending position, equal scores to the lower position
// (the key encoder of this geometry lives in encode_single.hip)
#include <algorithm>

#include "common.hpp"
#include "internal.hpp"

namespace a2ats {

constexpr int kCodewords = 4096;
constexpr int kSD = 128;   // head dimension = subspace dimension
constexpr int kLutChunk = kCodewords / kEncodeSlices;   // codewords of a table workgroup
static_assert(kLutChunk == 256, "a thread per codeword of the chunk writes the entries");
constexpr int kMaxChunk = 16384;   // tokens of a chunk of a sequence whose codewords are counted, at most (16-bit counts)
struct CodeCount {
  uint16_t* counts;   // [B * Hkv][chunks][codeword]
  uint2* ranges;      // [B * Hq][table workgroup]: the largest of the complements of the keys, and of the keys
  GridMap gm;         // of (sequence and KV head, chunk)
  int tokens;         // of a chunk: a power of two, 4096 .. kMaxChunk
  int aligned;        // the codes of every (sequence, KV head) start on 16 bytes
};

// float32 score <-> signed 32-bit key with the same order (so that the integer selection
// machinery of the product-quantised path applies unchanged).
__device__ __forceinline__ int32_t float_to_key(float f) {
  const int32_t b = __float_as_int(f);
  return b ^ ((b >> 31) & 0x7fffffff);
}
__device__ __forceinline__ float key_to_float(int32_t k) {
  return __int_as_float(k ^ ((k >> 31) & 0x7fffffff));
}

// ------------------------------------------------------------------------------------------
// Candidates per codeword
// ------------------------------------------------------------------------------------------
constexpr int kPerThread = 8;                       // consecutive tokens of one load
constexpr int kCountThreads = 512;

// The codes of tokens [j0, j0 + 8) of a sequence.  Branch-free: a start beyond the row is moved
// back into it (the caller masks such tokens by position), so every load is unconditional and a
// thread's loads are all in flight together.  ALIGNED rows (16-byte aligned, a multiple of 8
// codes long) take one 16-byte load, others eight 2-byte loads.
template <bool ALIGNED>
__device__ __forceinline__ uint4 load_codes8(const uint16_t* __restrict__ seq_codes, int j0, int row_len) {
  if (ALIGNED) return *(const uint4*)(seq_codes + min(j0, row_len - kPerThread));
  uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int i = 0; i < kPerThread; ++i) w[i >> 1] |= (uint32_t)seq_codes[min(j0 + i, row_len - 1)] << (16 * (i & 1));
  return make_uint4(w[0], w[1], w[2], w[3]);
}
__device__ __forceinline__ uint32_t code_of(const uint4& v, int i) {
  const uint32_t w = i < 2 ? v.x : (i < 4 ? v.y : (i < 6 ? v.z : v.w));
  return (w >> (16 * (i & 1))) & (kCodewords - 1);   // the mask keeps a bad code inside the table
}
// Bit i set when token j0 + i is a candidate, i.e. lies in [lo, hi).
__device__ __forceinline__ uint32_t valid_mask8(int j0, int lo, int hi) {
  const int a = min(max(lo - j0, 0), kPerThread), e = min(max(hi - j0, 0), kPerThread);
  return ((1u << e) - 1u) & ~((1u << a) - 1u);
}

// Whether every load of 8 codes may be one of 16 bytes.
static bool codes_aligned(const a2ats_dims& d, const void* codes) {
  return (((uintptr_t)codes) & 15u) == 0 && d.ctx_stride % kPerThread == 0 && d.ctx_stride >= kPerThread;
}

// Where the candidates of a sequence start being counted: rounds start on a multiple of 8 tokens.
__device__ __forceinline__ int first_token(const SeqRange& sr) { return sr.sink_end & ~(kPerThread - 1); }

// The sequence of a KV head in chunks of cc.tokens tokens, one workgroup (kCountThreads threads) each: counts[bkv][chunk][codeword].
// Chunks past the candidates and those of sequences that select everything are left out.
__device__ __forceinline__ void count_codes_body(int block, const CodeCount& cc, uint32_t* s_count,
                                                 const uint16_t* __restrict__ codes, const int32_t* __restrict__ seq_lens,
                                                 int Hkv, int ctx_len, int64_t ctx_stride, int top_k, int window,
                                                 int n_sink) {
  constexpr int NT = kCountThreads, kRounds = kMaxChunk / (NT * kPerThread);
  int bkv, chunk;
  map_block((uint32_t)block, cc.gm, bkv, chunk);
  const int tid = threadIdx.x, b = bkv / Hkv;
  const SeqRange sr = seq_range(ctx_len, seq_lens, b, window, n_sink, top_k);
  const int lo = sr.sink_end, hi = sr.win_start, s0 = first_token(sr) + chunk * cc.tokens;
  if (s0 >= hi || sr.kk == 0 || sr.kk >= sr.ncand) return;
  const uint16_t* seq_codes = codes + (size_t)bkv * ctx_stride;
  const int row_len = (int)ctx_stride, rounds = cc.tokens / (NT * kPerThread);
  uint4 cv[kRounds];
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const int j0 = s0 + (min(r, rounds - 1) * NT + tid) * kPerThread;
    cv[r] = cc.aligned ? load_codes8<true>(seq_codes, j0, row_len) : load_codes8<false>(seq_codes, j0, row_len);
  }
  for (int i = tid; i < kCodewords / 4; i += NT) ((uint4*)s_count)[i] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    if (r >= rounds) break;   // (uniform)
    const uint32_t vm = valid_mask8(s0 + (r * NT + tid) * kPerThread, lo, hi);
#pragma unroll
    for (int i = 0; i < kPerThread; ++i)
      if ((vm >> i) & 1u) atomicAdd(&s_count[code_of(cv[r], i)], 1u);
  }
  __syncthreads();
  uint4* out = (uint4*)(cc.counts + ((size_t)bkv * cc.gm.parts.d + chunk) * kCodewords);
  for (int i = tid; i < kCodewords / 8; i += NT) {   // (at most kMaxChunk tokens: 16 bits)
    const uint4 x = ((const uint4*)s_count)[2 * i], y = ((const uint4*)s_count)[2 * i + 1];
    out[i] = make_uint4(x.x | x.y << 16, x.z | x.w << 16, y.x | y.y << 16, y.z | y.w << 16);
  }
}

// ------------------------------------------------------------------------------------------
// Tables
// ------------------------------------------------------------------------------------------
// The sweep of 256 codewords against up to 16 vectors on the float64 matrix cores (16 x 16 x 4): a row of the product is a
// vector, from LDS, a column a codeword, from memory.  The inner dimension is taken in the order 16 i + 4 k + e (lane quarter
// k, step 4 i + e), so that a lane's share of a codeword is eight 16-byte loads; a wave takes two tiles of 16 codewords.
//
// Tables: the vectors are rotated queries, of any sequences (they have the codebook in common); `shared`: one table per KV
// head, from the float32 sum of its heads' rotated queries (the table array is then laid out for Hq = Hkv).
// Appended keys: up to a constant of the key, the distortion of codeword c is 1/2 |c^z|^2 - (k - mu) . w_c, so a key is the vector
// k - mu and the columns are the prepared w_c = (c - mu) H; each half of the dimensions one after the other, as
// encode_single_sweep_kernel has them, so that either finds the same code.  part[key][chunk] = {smallest value, its code}.
// Counts: candidates per codeword of the chunks of the sequences.
// The three kinds of workgroup have nothing to do with each other.
//
// What bounds it: latency.  4 sequences of 131072 tokens, 8 KV heads, one key each, tables, keys and counts: 16 us (a launch
// for the keys 11.5 and one for the tables 11.0 before, the counting in the selection), of which a sweep of 16 vectors takes 4.6
// (64 products of a wave, two waves a SIMD; a thread's dimensions on the vector ALU, eight lanes a codeword, took 10), the
// first loads 2.5 to 3.8.  Tables alone: 32 sequences of 32 heads 52 -> 28 us.  Up to four vectors of a KV head: products of four
// rows, and without keys and counts a wave takes one tile, twice as many workgroups: 4 heads 8.1 -> 5.1 us (eight lanes a
// codeword: 6.4), 8 KV heads of 4 8.6 -> 5.6.  Keys from the prepared columns instead of (k - mu) H, a product more, and the
// codewords: 8 keys of 4 sequences, a launch to pick them included, 18.2 -> 13.1 us.
constexpr int kTabThreads = 512, kTabTiles = kLutChunk / (16 * kTabThreads / 64);
static_assert(kTabTiles == 2, "a wave's codewords");
typedef __attribute__((ext_vector_type(4))) double f64x4;

constexpr int kFewVectors = 4;   // of a KV head: see add_product

struct TabLds {
  union {
    double v[kSD * 16];               // [dimension][vector], see tab_slot
    uint32_t count[kCodewords];
  };
  uint32_t range[2][16];            // of the vectors
  uint64_t best[16];                // of the keys: the smallest value, and the lowest code that has it
  int32_t arg[16];
};
// Where dimension d of vector `row` lies: the dimensions that the quarters of a wave read together are on different halves of
// the banks.
__device__ __forceinline__ int tab_slot(int d, int row) { return ((d ^ ((d >> 2) & 1)) << 4) | row; }

// Adds a step of the product to acc: rows 4 r + k (register r), column lane & 15; a: of row lane & 15.  FEW: there are no rows
// but the first four (four products of 4 x 4 x 4, of the same rows; a is of row lane & 3).  Their sums are the same bit for bit:
// either form adds the dimensions one after the other, without rounding the products.
template <bool FEW>
__device__ __forceinline__ void add_product(double a, double b, f64x4& acc) {
  if (FEW) acc[0] = __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, acc[0], 0, 0, 0);
  else acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc, 0, 0, 0);
}

// acc[t]: as above, of tile t.
template <bool FEW, int TILES>
__device__ __forceinline__ void tab_product(const float* __restrict__ cw, const TabLds& L, f64x4 (&acc)[TILES]) {
  const int lane = threadIdx.x & 63, j = lane & 15, k = lane >> 4, wave = threadIdx.x >> 6;
  float4 c[TILES][8];
#pragma unroll
  for (int t = 0; t < TILES; ++t)
#pragma unroll
    for (int i = 0; i < 8; ++i)
      c[t][i] = *(const float4*)(cw + (size_t)((wave * TILES + t) * 16 + j) * kSD + 16 * i + 4 * k);
#pragma unroll
  for (int t = 0; t < TILES; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int d = 16 * i + 4 * k + e;
      const double a = L.v[tab_slot(d, FEW ? j & 3 : j)];
#pragma unroll
      for (int t = 0; t < TILES; ++t) {
        const float4 f = c[t][i];
        add_product<FEW>(a, (double)(e == 0 ? f.x : (e == 1 ? f.y : (e == 2 ? f.z : f.w))), acc[t]);
      }
    }
}

// The same with the prepared columns of a KV head, the first half of which is in wv; each is replaced by its successor as it is
// used.  `at`: bytes to this lane's column and quarter of a step's dimensions.  (By descriptor: the steps are 128 KB apart, and
// an address in registers for each would not fit.)
constexpr int kKeySteps = kSD / 4;
__device__ __forceinline__ double load_column(__amdgpu_buffer_rsrc_t w, int at, int step, int tile) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(w, at + tile * 16 * (int)sizeof(double),
                                                                         step * 4 * kCodewords * (int)sizeof(double), 0));
}
template <bool FEW, int TILES>
__device__ __forceinline__ void key_product(__amdgpu_buffer_rsrc_t w, int at, double (&wv)[TILES][kKeySteps / 2], const TabLds& L,
                                            f64x4 (&acc)[TILES]) {
  const int lane = threadIdx.x & 63, j = lane & 15, k = lane >> 4;
  f64x4 second[TILES];
#pragma unroll
  for (int t = 0; t < TILES; ++t) acc[t] = second[t] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int i = 0; i < kKeySteps; ++i) {
    const double a = L.v[tab_slot(4 * i + k, FEW ? j & 3 : j)];
#pragma unroll
    for (int t = 0; t < TILES; ++t) {
      double& x = wv[t][i % (kKeySteps / 2)];
      add_product<FEW>(a, x, i < kKeySteps / 2 ? acc[t] : second[t]);
      if (i < kKeySteps / 2) x = load_column(w, at, i + kKeySteps / 2, t);
    }
    __builtin_amdgcn_sched_barrier(0);   // (else the second half is requested before the first has been used: registers)
  }
#pragma unroll
  for (int t = 0; t < TILES; ++t) acc[t] += second[t];
}

// A number that is not a NaN as an unsigned integer of the same order (0 and -0 are one).
__device__ __forceinline__ uint64_t ordered_bits(double x) {
  const uint64_t b = __builtin_bit_cast(uint64_t, x + 0.0);
  return b ^ ((uint64_t)((int64_t)b >> 63) | 0x8000000000000000ull);
}
// The largest of 16 lanes, in all of them.
__device__ __forceinline__ uint32_t row16_most(uint32_t v) {
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xf, 0xf, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xf, 0xf, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xf, 0xf, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xf, 0xf, false));
  return v;
}

// Workgroups of build_lut_single_kernel: those of the appended keys, the tables, the counts, in this order.
struct TabPlan {
  int n_key, n_table;        // workgroups
  FastDiv key_groups, table_groups;   // of 16 vectors, of a KV head
  int per_seq;               // table heads of a sequence and KV head
  FastDiv per_seq_div, n_new_div;
};

// The code of key `key` of all: the smallest of its slices (they hold ascending codes: strict < keeps the lower code on equal
// values).
__device__ __forceinline__ uint16_t pick_code(const double* __restrict__ part, size_t key) {
  const double* mine = part + key * kEncodeSlices * 2;
  double best = mine[0];
  int arg = (int)mine[1];
#pragma unroll
  for (int sl = 1; sl < kEncodeSlices; ++sl) {
    const double dv = mine[2 * sl];
    const int code = (int)mine[2 * sl + 1];
    arg = dv < best ? code : arg;
    best = dv < best ? dv : best;
  }
  return (uint16_t)arg;
}

// TILES 1: no more than kFewVectors tables of a KV head, and neither keys nor counts.  FEW_KEYS: no more than that many keys.
template <bool QBF16, int TILES, bool FEW_KEYS>
__global__ __launch_bounds__(kTabThreads) __attribute__((amdgpu_waves_per_eu(4, 4))) void build_lut_single_kernel(
    const void* __restrict__ q_in, const float* __restrict__ cos_b, const float* __restrict__ sin_b,
    const float* __restrict__ codebook, float* __restrict__ q_rot, int32_t* __restrict__ lut,
    float* __restrict__ lut_scale, int B, int Hq, int Hkv, int shared, TabPlan tp, FewKeys few, CodeCount cc,
    const uint16_t* __restrict__ codes, const int32_t* __restrict__ seq_lens, int ctx_len, int64_t ctx_stride, int top_k,
    int window, int n_sink) {
  constexpr int HALF = kSD / 2, NT = kTabThreads, CHUNK = 16 * (NT / 64) * TILES, CHUNKS = kCodewords / CHUNK;
  static_assert(TILES == 1 || CHUNKS == kEncodeSlices, "the slices of the keys, and those of the ranges");
  __shared__ __align__(16) TabLds L;
  const int tid = threadIdx.x, lane = tid & 63, j = lane & 15, k = lane >> 4, wave = tid >> 6;
  int block = blockIdx.x;
  if (block >= tp.n_key + tp.n_table) {
    count_codes_body(block - tp.n_key - tp.n_table, cc, L.count, codes, seq_lens, Hkv, ctx_len, ctx_stride, top_k, window,
                     n_sink);
    return;
  }
  const bool is_key = block < tp.n_key;
  if (!is_key) block -= tp.n_key;
  const int chunk = block % CHUNKS, unit = block / CHUNKS;
  const FastDiv& groups = is_key ? tp.key_groups : tp.table_groups;
  const int kv = (int)fast_div((uint32_t)unit, groups), v0 = (unit - kv * (int)groups.d) * 16;   // first vector of the group
  f64x4 acc[TILES];

  if (!is_key) {
    const int G = Hq / Hkv, per = tp.per_seq, n_vec = B * per;
    for (int i = tid; i < 16 * HALF; i += NT) {
      const int row = i / HALF, t = i % HALF, vec = v0 + row;
      double s1 = 0.0, s2 = 0.0;
      if (vec < n_vec) {
        const int b = (int)fast_div((uint32_t)vec, tp.per_seq_div), g0 = vec - b * per;
        const double c = (double)cos_b[t], s = (double)sin_b[t];
        for (int g = shared ? 0 : g0; g < (shared ? G : g0 + 1); ++g) {
          const size_t base = ((size_t)b * Hq + kv * G + g) * kSD;
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
          const float o1 = (float)(x1 * c - x2 * s), o2 = (float)(x2 * c + x1 * s);
          s1 += (double)o1;
          s2 += (double)o2;
          if (chunk == 0) {
            q_rot[base + t] = o1;
            q_rot[base + t + HALF] = o2;
          }
        }
        if (chunk == 0 && t == 0) lut_scale[((size_t)b * Hkv + kv) * per + g0] = 1.f;
      }
      L.v[tab_slot(t, row)] = (double)(float)s1;
      L.v[tab_slot(t + HALF, row)] = (double)(float)s2;
    }
    __syncthreads();
    const float* cw = codebook + ((size_t)kv * kCodewords + chunk * CHUNK) * kSD;
    if (cc.ranges && tid < 32) L.range[tid >> 4][tid & 15] = 0u;
    if (TILES == 1 || n_vec <= kFewVectors) tab_product<true>(cw, L, acc);
    else tab_product<false>(cw, L, acc);
    if (cc.ranges) __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int vec = v0 + 4 * r + k;
      uint32_t key[TILES];
#pragma unroll
      for (int t = 0; t < TILES; ++t) key[t] = (uint32_t)float_to_key((float)acc[t][r]);
      if (vec < n_vec) {   // (uniform over 16 lanes)
        const int b = (int)fast_div((uint32_t)vec, tp.per_seq_div), g = vec - b * per;
        int32_t* out = lut + (((size_t)b * Hkv + kv) * per + g) * kCodewords + chunk * CHUNK + wave * TILES * 16 + j;
#pragma unroll
        for (int t = 0; t < TILES; ++t) out[16 * t] = (int32_t)key[t];
      }
      if (cc.ranges) {
        uint32_t least = 0, most = 0;
#pragma unroll
        for (int t = 0; t < TILES; ++t) {
          least = max(least, ~score_key((int32_t)key[t]));
          most = max(most, score_key((int32_t)key[t]));
        }
        least = row16_most(least);
        most = row16_most(most);
        if (j == 0) {
          atomicMax(&L.range[0][4 * r + k], least);
          atomicMax(&L.range[1][4 * r + k], most);
        }
      }
    }
    if (cc.ranges) {
      __syncthreads();
      const int vec = v0 + tid;
      if (tid < 16 && vec < n_vec) {
        const int b = (int)fast_div((uint32_t)vec, tp.per_seq_div), g = vec - b * per;
        cc.ranges[(((size_t)b * Hkv + kv) * per + g) * kEncodeSlices + chunk] = make_uint2(L.range[0][tid], L.range[1][tid]);
      }
    }
    return;
  }

  // --- appended keys
  if (TILES == 1) return;
  const int n_vec = B * few.n_new;
  const float* mu = few.mu + (size_t)kv * few.mu_stride;
  auto key_index = [&](int vec) {   // among all keys
    const int b = (int)fast_div((uint32_t)vec, tp.n_new_div);
    return (size_t)(b * Hkv + kv) * few.n_new + (vec - b * few.n_new);
  };
  constexpr int PER = 16 * kSD / NT;   // of the vectors' entries
  float x[PER], m[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int row = (tid + i * NT) / kSD, d = tid % kSD, vec = min(v0 + row, n_vec - 1);
    x[i] = few.keys[key_index(vec) * kSD + d];
    m[i] = mu[d];
  }
  const int col = chunk * CHUNK + wave * TILES * 16 + j, at = (k * kCodewords + col) * (int)sizeof(double);
  const auto w = __builtin_amdgcn_make_buffer_rsrc((void*)(few.wT + (size_t)kv * kSD * kCodewords), 0,
                                                   kSD * kCodewords * (int)sizeof(double), 0x00027000);
  double wv[TILES][kKeySteps / 2], chalf[TILES];
#pragma unroll
  for (int i = 0; i < kKeySteps / 2; ++i)
#pragma unroll
    for (int t = 0; t < TILES; ++t) wv[t][i] = load_column(w, at, i, t);
#pragma unroll
  for (int t = 0; t < TILES; ++t) chalf[t] = few.chalf[(size_t)kv * kCodewords + col + 16 * t];
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int row = (tid + i * NT) / kSD, d = tid % kSD;
    L.v[tab_slot(d, row)] = v0 + row < n_vec ? (double)x[i] - (double)m[i] : 0.0;
  }
  if (tid < 16) {
    L.best[tid] = ~0ull;
    L.arg[tid] = CHUNK;
  }
  __syncthreads();
  key_product<FEW_KEYS>(w, at, wv, L, acc);
  // the smallest of a key's values, the lower code on equal ones (a value that is not a number is never smaller)
  double best[4];
  int arg[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    best[r] = INFINITY;
    arg[r] = 0;
#pragma unroll
    for (int t = 0; t < TILES; ++t) {
      const double s = chalf[t] - acc[t][r];
      if (s < best[r]) {
        best[r] = s;
        arg[r] = (wave * TILES + t) * 16 + j;
      }
    }
  }
  uint64_t mine[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    mine[r] = ordered_bits(best[r]);
    atomicMin((unsigned long long*)&L.best[4 * r + k], (unsigned long long)mine[r]);
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 4; ++r)
    if (mine[r] == L.best[4 * r + k]) atomicMin(&L.arg[4 * r + k], arg[r]);
  __syncthreads();
  if (tid < 16 && v0 + tid < n_vec) {
    double* out = few.part + (key_index(v0 + tid) * kEncodeSlices + chunk) * 2;
    const uint64_t o = L.best[tid];
    out[0] = __builtin_bit_cast(double, o ^ (o >> 63 ? 0x8000000000000000ull : ~0ull));
    out[1] = (double)(chunk * CHUNK + L.arg[tid]);
  }
}

// Tables (q), appended keys (few.keys) and counts (n_count workgroups), any of them or all.
static hipError_t launch_tables_single(const a2ats_dims& d, const void* q, int q_dtype, const float* cos_b,
                                       const float* sin_b, const float* codebook, float* q_rot, int32_t* lut,
                                       float* lut_scale, bool shared, const FewKeys& few, const CodeCount& cc, int n_count,
                                       const void* codes, const int32_t* seq_lens, int top_k, int window, int n_sink,
                                       hipStream_t stream) {
  if (d.batch == 0) return hipSuccess;
  TabPlan tp;
  const int n_new = few.keys ? few.n_new : 0;
  tp.per_seq = shared ? 1 : d.n_q_heads / d.n_kv_heads;
  tp.per_seq_div = make_fastdiv((uint32_t)tp.per_seq);
  tp.n_new_div = make_fastdiv((uint32_t)n_new);
  const int key_groups = (d.batch * n_new + 15) / 16, table_groups = q ? (d.batch * tp.per_seq + 15) / 16 : 0;
  tp.key_groups = make_fastdiv((uint32_t)key_groups);
  tp.table_groups = make_fastdiv((uint32_t)table_groups);
  tp.n_key = key_groups * d.n_kv_heads * kEncodeSlices;
  const bool small = n_new == 0 && !cc.counts && d.batch * tp.per_seq <= kFewVectors;
  tp.n_table = table_groups * d.n_kv_heads * kEncodeSlices * (small ? kTabTiles : 1);
  const dim3 grid(tp.n_key + tp.n_table + n_count), block(kTabThreads);
  if (grid.x == 0) return hipSuccess;
#define A2ATS_LAUNCH_TABLES(BF, TILES, FEW_KEYS)                                                                          \
  hipLaunchKernelGGL((build_lut_single_kernel<BF, TILES, FEW_KEYS>), grid, block, 0, stream, q, cos_b, sin_b, codebook,  \
                     q_rot, lut, lut_scale, d.batch, d.n_q_heads, d.n_kv_heads, shared ? 1 : 0, tp, few, cc,             \
                     (const uint16_t*)codes, seq_lens, d.ctx_len, d.ctx_stride, top_k, window, n_sink)
#define A2ATS_LAUNCH_TABLES2(BF)                                                          \
  do {                                                                                    \
    if (small) A2ATS_LAUNCH_TABLES(BF, 1, true);                                          \
    else if (d.batch * n_new <= kFewVectors) A2ATS_LAUNCH_TABLES(BF, kTabTiles, true);    \
    else A2ATS_LAUNCH_TABLES(BF, kTabTiles, false);                                       \
  } while (0)
  if (q_dtype == A2ATS_BF16) A2ATS_LAUNCH_TABLES2(true);
  else A2ATS_LAUNCH_TABLES2(false);
#undef A2ATS_LAUNCH_TABLES2
#undef A2ATS_LAUNCH_TABLES
  return hipGetLastError();
}

hipError_t launch_build_lut_single(const a2ats_dims& d, const void* q, int q_dtype, const float* cos_b,
                                   const float* sin_b, const float* codebook, float* q_rot, int32_t* lut,
                                   float* lut_scale, bool shared, const FewKeys& few, hipStream_t stream) {
  return launch_tables_single(d, q, q_dtype, cos_b, sin_b, codebook, q_rot, lut, lut_scale, shared, few, CodeCount{}, 0,
                              nullptr, nullptr, 0, 0, 0, stream);
}

hipError_t launch_sweep_single(const a2ats_dims& d, const FewKeys& few, hipStream_t stream) {
  return launch_tables_single(d, nullptr, A2ATS_F32, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, false, few,
                              CodeCount{}, 0, nullptr, nullptr, 0, 0, 0, stream);
}

// ------------------------------------------------------------------------------------------
// Selection
// ------------------------------------------------------------------------------------------
constexpr int kSelThreads = 512;
constexpr int kRound = kSelThreads * kPerThread;    // tokens per round

constexpr int kSpan = 32;                           // rounds a thread keeps in registers
constexpr int kSpanTokens = kSpan * kRound;         // 131072
constexpr int kSelWaves = kSelThreads / 64;
constexpr int kSmallSel = 128;                      // a K-th-key bin of at most this many codewords is finished by counting

struct SelLds {
  int32_t table[kCodewords];    // the head's scores as order-preserving keys
  uint32_t count[kCodewords];   // candidate tokens per codeword
  uint32_t hist[kHistBins];
  uint32_t wave_tot[kSpan][kSelWaves];   // packed (above, equal) counts per round and wave
  uint32_t wave_pre[kSpan][kSelWaves];   // ... exclusive over the waves of a round
  uint32_t round_tot[kSpan];
  uint32_t wave_a[kSelWaves];
  uint32_t res[2];
  uint32_t kmin, kmax;
  uint32_t small_n;                 // codewords in the bin of the K-th key after a radix level
  uint32_t small_key[kSmallSel], small_w[kSmallSel];
  uint8_t cls[kCodewords];          // per codeword: 1 = above the K-th key, 2 = equal to it, 0 = below
};

// Bit 2i set when bit i of an 8-bit mask is.
__device__ __forceinline__ uint32_t spread8(uint32_t m) {
  m = (m | (m << 4)) & 0x0f0fu;
  m = (m | (m << 2)) & 0x3333u;
  return (m | (m << 1)) & 0x5555u;
}

// One workgroup per head.  A score is one table entry, so the K-th largest score over the
// candidate tokens is a weighted selection over the 4096 codewords: (1) count the candidates per
// codeword (one pass over the 2-byte codes), (2) find the K-th key over the 4096 keys weighted by
// those counts, (3) a pass that emits the winners in ascending position, equal scores going to
// the lower position.  A thread keeps the codes of kSpan rounds of 8 consecutive tokens in
// registers (one span = 131072 tokens per workgroup): all its loads are in flight together, a
// context of one span is read once and serves both passes, and the rounds share one scan of their
// packed (above, equal) counts over the waves instead of one scan and two barriers per round.
template <bool ALIGNED>
__global__ __launch_bounds__(kSelThreads) void select_single_kernel(
    const uint16_t* __restrict__ codes, const int32_t* __restrict__ lut, const int32_t* __restrict__ seq_lens,
    int32_t* __restrict__ topk_idx, int32_t* __restrict__ topk_count, float* __restrict__ topk_score,
    int Hq, int Hkv, int ctx_len, int64_t ctx_stride, int top_k, int window, int n_sink) {
  constexpr int NT = kSelThreads;
  __shared__ SelLds L;
  const int bh = blockIdx.x, b = bh / Hq, h = bh % Hq, G = Hq / Hkv, kv = h / G, tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6, wave_u = __builtin_amdgcn_readfirstlane(wave);
  const SeqRange sr = seq_range(ctx_len, seq_lens, b, window, n_sink, top_k);
  int32_t* oi = topk_idx + (size_t)bh * top_k;
  float* os = topk_score ? topk_score + (size_t)bh * top_k : nullptr;
  if (tid == 0) topk_count[bh] = sr.kk;
  for (int t = sr.kk + tid; t < top_k; t += NT) {
    oi[t] = -1;
    if (os) os[t] = 0.f;
  }
  if (sr.kk == 0) return;

  const uint16_t* seq_codes = codes + ((size_t)b * Hkv + kv) * ctx_stride;
  const int row_len = (int)ctx_stride;
  const int lo = sr.sink_end, hi = sr.win_start;
  const int first = lo & ~(kPerThread - 1);   // rounds start on a multiple of 8 tokens
  const int n_span = (hi - first + kSpanTokens - 1) / kSpanTokens;
  const bool take_all = sr.kk >= sr.ncand;

  // Requests in the order their data is needed last-to-first is wrong for in-order returns: the
  // table is asked for first (it is small), the codes after it, so the count pass can start on the
  // first round's codes while the later rounds are still arriving.
  constexpr int kTablePer = kCodewords / NT;
  const int32_t* head_table = lut + (size_t)bh * kCodewords;
  int32_t tv[kTablePer];
#pragma unroll
  for (int i = 0; i < kTablePer; ++i) tv[i] = head_table[i * NT + tid];
  uint4 cv[kSpan];
  if (!take_all || n_span == 1) {
#pragma unroll
    for (int r = 0; r < kSpan; ++r) cv[r] = load_codes8<ALIGNED>(seq_codes, first + r * kRound + tid * kPerThread, row_len);
  }
  uint32_t kmin = 0xffffffffu, kmax = 0u;
#pragma unroll
  for (int i = 0; i < kTablePer; ++i) {
    L.table[i * NT + tid] = tv[i];
    L.count[i * NT + tid] = 0;
    kmin = min(kmin, score_key(tv[i]));
    kmax = max(kmax, score_key(tv[i]));
  }
  if (tid == 0) {
    L.kmin = 0xffffffffu;
    L.kmax = 0u;
  }
  __syncthreads();

  uint32_t kth = 0, k_rem = (uint32_t)sr.kk;
  if (!take_all) {
    // (1) candidates per codeword
#pragma unroll 1
    for (int sp = 0; sp < n_span; ++sp) {
      const int s0 = first + sp * kSpanTokens;
      if (sp > 0) {
#pragma unroll
        for (int r = 0; r < kSpan; ++r) cv[r] = load_codes8<ALIGNED>(seq_codes, s0 + r * kRound + tid * kPerThread, row_len);
      }
#pragma unroll
      for (int r = 0; r < kSpan; ++r) {
        const int jw = s0 + r * kRound + wave_u * (64 * kPerThread);   // first token of this wave's share
        if (jw >= lo && jw + 64 * kPerThread <= hi) {   // (wave-uniform) every token is a candidate
#pragma unroll
          for (int i = 0; i < kPerThread; ++i) atomicAdd(&L.count[code_of(cv[r], i)], 1u);
        } else if (jw < hi) {   // (a spare bin for the others is one address for all that lies past the end: 122 us, not 18, at 4096 tokens)
          const uint32_t vm = valid_mask8(s0 + r * kRound + tid * kPerThread, lo, hi);
#pragma unroll
          for (int i = 0; i < kPerThread; ++i)
            if ((vm >> i) & 1u) atomicAdd(&L.count[code_of(cv[r], i)], 1u);
        }
      }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      kmin = min(kmin, __shfl_xor(kmin, off));
      kmax = max(kmax, __shfl_xor(kmax, off));
    }
    if (lane == 0) {
      atomicMin(&L.kmin, kmin);
      atomicMax(&L.kmax, kmax);
    }
    __syncthreads();
    // (2) the K-th largest key over the codewords weighted by those counts.  First a level of
    // 2048 bins LINEAR in the score between the smallest and the largest table entry (the bit
    // pattern of a float spends its leading digits on the exponent: a level on those would put
    // every score of one binade into one bin); the mapping is monotone, so the bin of the K-th
    // key is exact.  That bin usually holds a handful of codewords: they are listed, and every
    // member adds up the candidates above and at its own key -- the member whose range contains
    // k_rem is the K-th key.  A crowded bin (many equal or nearly equal scores), or a table whose
    // range is empty or not finite, is finished by an MSB-first radix select on the keys.
    const uint32_t k_lo = L.kmin;
    const float s_lo = key_to_float(key_score(k_lo)), span = key_to_float(key_score(L.kmax)) - s_lo;
    const bool use_lin = span >= 1e-30f && span < INFINITY;
    const float lin_scale = use_lin ? (float)kHistBins / span : 0.f;
    auto lin_bin = [&](int32_t entry) {
      return (uint32_t)min((int)((key_to_float(entry) - s_lo) * lin_scale), kHistBins - 1);
    };
    uint32_t bin1 = 0;
    bool found = false;
    if (use_lin) {
      // this thread's 8 codewords, read once (the loops below would otherwise wait for LDS per codeword)
      uint32_t w8[kTablePer], b8[kTablePer];
#pragma unroll
      for (int i = 0; i < kTablePer; ++i) {
        w8[i] = L.count[i * NT + tid];
        b8[i] = lin_bin(tv[i]);
      }
      for (int i = tid; i < kHistBins; i += NT) L.hist[i] = 0;
      if (tid == 0) L.small_n = 0;
      __syncthreads();
#pragma unroll
      for (int i = 0; i < kTablePer; ++i)
        if (w8[i]) atomicAdd(&L.hist[b8[i]], w8[i]);
      __syncthreads();
      block_find_rank_desc<NT, kHistBins>([&](int i) { return L.hist[i]; }, k_rem, L.wave_a, L.res);
      bin1 = L.res[0];
      k_rem -= L.res[1];
#pragma unroll
      for (int i = 0; i < kTablePer; ++i) {
        if (w8[i] && b8[i] == bin1) {
          const uint32_t at = atomicAdd(&L.small_n, 1u);
          if (at < (uint32_t)kSmallSel) {
            L.small_key[at] = score_key(tv[i]);
            L.small_w[at] = w8[i];
          }
        }
      }
      __syncthreads();
      const uint32_t n_small = L.small_n;
      if (n_small <= (uint32_t)kSmallSel) {
        if ((uint32_t)tid < n_small) {
          const uint32_t key = L.small_key[tid];
          uint32_t gt = 0, eq = 0;
          for (uint32_t u = 0; u < n_small; ++u) {
            const uint32_t ku = L.small_key[u], wu = L.small_w[u];
            gt += ku > key ? wu : 0u;
            eq += ku == key ? wu : 0u;
          }
          if (gt < k_rem && k_rem <= gt + eq) {   // every member at the K-th key writes the same two words
            L.res[0] = key;
            L.res[1] = k_rem - gt;
          }
        }
        __syncthreads();
        kth = L.res[0];
        k_rem = L.res[1];
        found = true;
      }
    }
    if (!found) {
      int remaining = 32 - __clz(L.kmax - k_lo);
      uint32_t prefix = 0, mask = 0;
#pragma unroll 1
      while (remaining > 0) {
        const int bits = remaining < 11 ? remaining : 11;
        const int shift = remaining - bits;
        const uint32_t dmask = (1u << bits) - 1u;
        __syncthreads();   // the histogram may still be read
        for (int i = tid; i < kHistBins; i += NT) L.hist[i] = 0;
        __syncthreads();
        for (int e = tid; e < kCodewords; e += NT) {
          const int32_t entry = L.table[e];
          const uint32_t rel = score_key(entry) - k_lo, w = L.count[e];
          if (w && (!use_lin || lin_bin(entry) == bin1) && (rel & mask) == prefix)
            atomicAdd(&L.hist[(rel >> shift) & dmask], w);
        }
        __syncthreads();
        block_find_rank_desc<NT, kHistBins>([&](int i) { return L.hist[i]; }, k_rem, L.wave_a, L.res);
        const uint32_t bin = L.res[0], above = L.res[1];
        k_rem -= above;
        prefix |= bin << shift;
        mask |= dmask << shift;
        remaining = shift;
      }
      kth = prefix + k_lo;
    }
  }
  // class of every codeword, one byte each: the emission pass then costs one byte read per token
#pragma unroll
  for (int i = 0; i < kTablePer; ++i) {
    const uint32_t key = score_key(tv[i]);
    L.cls[i * NT + tid] = take_all ? 1 : (key > kth ? 1 : (key == kth ? 2 : 0));
  }
  __syncthreads();

  // (3) ordered emission: keys above the K-th, plus the first k_rem positions that equal it
  uint32_t out_n = 0, eq_seen = 0;
#pragma unroll 1
  for (int sp = 0; sp < n_span; ++sp) {
    const int s0 = first + sp * kSpanTokens;
    if (n_span > 1) {
      __syncthreads();   // the scan arrays of the span before are still being read
#pragma unroll
      for (int r = 0; r < kSpan; ++r) cv[r] = load_codes8<ALIGNED>(seq_codes, s0 + r * kRound + tid * kPerThread, row_len);
    }
    // two bits per token (bit 2i: above the K-th key, bit 2i + 1: equal to it), two rounds per word
    uint32_t cbits[kSpan / 2];
    uint32_t pre[kSpan];   // packed (above, equal) counts of the lanes before this one, per round
#pragma unroll
    for (int i = 0; i < kSpan / 2; ++i) cbits[i] = 0;
#pragma unroll
    for (int r = 0; r < kSpan; ++r) {
      uint32_t c2 = 0;
#pragma unroll
      for (int i = 0; i < kPerThread; ++i) c2 |= (uint32_t)L.cls[code_of(cv[r], i)] << (2 * i);
      const int jw = s0 + r * kRound + wave_u * (64 * kPerThread);
      if (!(jw >= lo && jw + 64 * kPerThread <= hi)) {   // (wave-uniform) some tokens are not candidates
        const uint32_t vm = spread8(valid_mask8(s0 + r * kRound + tid * kPerThread, lo, hi));
        c2 &= vm | (vm << 1);
      }
      cbits[r / 2] |= c2 << (16 * (r % 2));
      const uint32_t own = (uint32_t)__popc(c2 & 0x5555u) | ((uint32_t)__popc(c2 & 0xaaaau) << 16);
      const uint32_t v = wave_inclusive_scan(own);
      pre[r] = v - own;
      if (lane == 63) L.wave_tot[r][wave] = v;
    }
    __syncthreads();
    if (tid < kSpan * kSelWaves) {   // exclusive scan over the 16 waves of each round (16-lane groups)
      const int r = tid / kSelWaves, w = tid % kSelWaves;
      const uint32_t own = L.wave_tot[r][w];
      uint32_t v = own;
#pragma unroll
      for (int off = 1; off < kSelWaves; off <<= 1) {
        const uint32_t n = __shfl_up(v, off, kSelWaves);
        if (w >= off) v += n;
      }
      L.wave_pre[r][w] = v - own;
      if (w == kSelWaves - 1) L.round_tot[r] = v;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSpan; ++r) {
      const uint32_t c2 = (cbits[r / 2] >> (16 * (r % 2))) & 0xffffu;
      const uint32_t g = c2 & 0x5555u, e = (c2 >> 1) & 0x5555u;   // token i at bit 2i
      const uint32_t tot = L.round_tot[r];
      const uint32_t own_pre = pre[r];
      if (g | e) {
        const int j0 = s0 + r * kRound + tid * kPerThread;
        const uint32_t p = own_pre + L.wave_pre[r][wave];
        // winners of this thread: everything above the K-th, and the equal ones whose rank among
        // the equal ones is below k_rem
        const uint32_t gt_before = p & 0xffffu, eq_before = eq_seen + (p >> 16);
        uint32_t e_take = 0;
        if (e && eq_before < k_rem) {
          const uint32_t room = k_rem - eq_before;   // >= 1
          e_take = e;
          if ((uint32_t)__popc(e) > room) {          // keep the lowest `room` set bits
#pragma unroll 1
            for (uint32_t drop = (uint32_t)__popc(e) - room; drop; --drop) e_take &= ~(0x80000000u >> __clz(e_take));
          }
        }
        uint32_t m = g | e_take;
#pragma unroll 1
        while (m) {
          const int bit = __ffs(m) - 1, i = bit >> 1;
          const uint32_t below = (1u << bit) - 1u;
          const uint32_t slot = out_n + gt_before + (uint32_t)__popc(g & below) + min(eq_before, k_rem) + (uint32_t)__popc(e_take & below);
          oi[slot] = j0 + i;
          if (os) os[slot] = key_to_float(L.table[seq_codes[j0 + i] & (kCodewords - 1)]);
          m &= m - 1;
        }
      }
      out_n += tot & 0xffffu;
      eq_seen += tot >> 16;
    }
    if (out_n + min(eq_seen, k_rem) >= (uint32_t)sr.kk) break;   // uniform over the workgroup
  }
}

// ------------------------------------------------------------------------------------------
// Selection from counts that an earlier launch has made (a2ats_decode_select)
// ------------------------------------------------------------------------------------------
// One workgroup per chunk of a sequence and H query heads of a KV head.  Every workgroup adds up the chunks' counts (8 KB
// each) and finds the K-th key of its heads by itself; what the chunks before its own hold above that key and at it gives
// the place of its first winner, so the workgroups of a head need nothing from each other.
//
// What bounds it: its phases one after the other; 4 sequences of 131072 tokens, 32 heads: 14.5 us, of which counts, keys and
// codes take 4.5 to arrive, bins and K-th keys 4.5, flags and places 3.  A workgroup a head, which counts by itself and holds
// the codes meanwhile (select_single_kernel), takes 32.5.  Steps: 90.1 -> 63.9 us.
constexpr int kCsThreads = 512, kCsWaves = kCsThreads / 64;
constexpr int kCsPer = kCodewords / kCsThreads;                       // codewords of a thread
static_assert(kCsPer == 8, "a thread's counts are one 16-byte load");
template <int H>
struct ChunkLds {
  uint32_t hist[H][kHistBins];
  uint32_t flags[kCodewords];   // bit (16 / H) h: above the K-th key of head h, 16 bits further: equal to it
  uint32_t small_key[H][kSmallSel], small_w[H][kSmallSel];
  uint32_t bin[H], kth[H], k_rem[H], small_n[H];
  uint32_t before_gt[H], before_eq[H];
  uint32_t wave_tot[H][kCsWaves];
  uint32_t wave_a[kCsWaves], res[2];
};

// The bin that holds the k-th largest of the values counted in a 2048-bin histogram, and how many lie above it, by one wave.
__device__ __forceinline__ void wave_rank(const uint32_t* hist, uint32_t k, int lane, uint32_t& bin, uint32_t& above) {
  uint32_t sum = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) {   // (rotated: the lanes of a read hit different banks)
    const uint4 v = *(const uint4*)(hist + 32 * lane + 4 * ((i + lane) & 7));
    sum += v.x + v.y + v.z + v.w;
  }
  const uint32_t pre = wave_inclusive_scan(sum);
  const uint32_t inc = (uint32_t)__builtin_amdgcn_readlane((int)pre, 63) - pre + sum, higher = inc - sum;
  const uint64_t owner = __builtin_amdgcn_ballot_w64(higher < k && k <= inc);
  const int src = owner ? (int)__builtin_ctzll(owner) : 0;
  const uint32_t base = (uint32_t)__builtin_amdgcn_readlane((int)higher, src);
  const uint32_t c = lane < 32 ? hist[32 * src + 31 - lane] : 0u;
  const uint32_t incl = wave_inclusive_scan(c);
  const uint64_t reach = __builtin_amdgcn_ballot_w64(lane < 32 && base + incl >= k);
  const int at = reach ? (int)__builtin_ctzll(reach) : 31;
  bin = (uint32_t)(32 * src + 31 - at);
  above = base + (uint32_t)__builtin_amdgcn_readlane((int)(incl - c), at);
}

template <int H>
__global__ __launch_bounds__(kCsThreads) __attribute__((amdgpu_waves_per_eu(4, 4))) void select_chunks_single_kernel(
    uint16_t* __restrict__ codes, const int32_t* __restrict__ lut, const int32_t* __restrict__ seq_lens,
    int32_t* __restrict__ topk_idx, int32_t* __restrict__ topk_count, float* __restrict__ topk_score, CodeCount cc,
    GridMap gm, const double* __restrict__ part, int n_new, int pos0, int Hq, int Hkv, int ctx_len,
    int64_t ctx_stride, int top_k, int window, int n_sink) {
  constexpr int NT = kCsThreads, kLoads = kMaxChunk / (kCsThreads * kPerThread);
  constexpr int kBits = 16 / H, kAcc = kLoads * kPerThread / kBits, kWords = kLoads * kPerThread / 32;   // tokens of a word of flags
  __shared__ ChunkLds<H> L;
  int prob, chunk, b, kv, g4;
  map_block(blockIdx.x, gm, prob, chunk);
  split_problem(prob, gm, b, kv, g4);
  const int G = Hq / Hkv, n_real = min(H, G - g4 * H), bkv = b * Hkv + kv, head0 = b * Hq + kv * G + g4 * H;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const SeqRange sr = seq_range(ctx_len, seq_lens, b, window, n_sink, top_k);
  if (chunk == 0) {
    if (tid < n_real) topk_count[head0 + tid] = sr.kk;
    for (int h = 0; h < n_real; ++h)
      for (int t = sr.kk + tid; t < top_k; t += NT) {
        topk_idx[(size_t)(head0 + h) * top_k + t] = -1;
        if (topk_score) topk_score[(size_t)(head0 + h) * top_k + t] = 0.f;
      }
    // The codes of the keys appended in this step, which the launch before has swept.  No candidate is among them.
    if (g4 == 0 && tid < n_new)
      codes[(size_t)bkv * ctx_stride + pos0 + tid] = pick_code(part, (size_t)bkv * n_new + tid);
  }
  const int lo = sr.sink_end, hi = sr.win_start, first = first_token(sr), s0 = first + chunk * cc.tokens;
  if (sr.kk == 0 || s0 >= hi) return;
  const uint16_t* seq_codes = codes + (size_t)bkv * ctx_stride;
  const int row_len = (int)ctx_stride, loads = cc.tokens / (NT * kPerThread);   // 1 .. kLoads
  const int j0 = s0 + tid * loads * kPerThread;   // this thread's tokens follow each other
  const bool take_all = sr.kk >= sr.ncand;
  uint4 cv[kLoads];
  uint32_t k_rem[H], acc[kAcc];
#pragma unroll
  for (int q = 0; q < kAcc; ++q) acc[q] = 0u;
#pragma unroll
  for (int h = 0; h < H; ++h) k_rem[h] = 0u;

  if (!take_all) {   // (uniform, as the conditions on n_real and n_part below)
    // --- this thread's 8 codewords: their counts in all chunks and in those before this one, and their keys
    const int n_part = (hi - first + cc.tokens - 1) / cc.tokens;
    const uint4* cnt = (const uint4*)(cc.counts + (size_t)bkv * cc.gm.parts.d * kCodewords) + tid;
    int32_t tv[H][kCsPer];
    uint2 range[H];
#pragma unroll
    for (int h = 0; h < H; ++h) {
      if (h >= n_real) break;
      range[h] = cc.ranges[(size_t)(head0 + h) * kEncodeSlices + (lane & (kEncodeSlices - 1))];
      const int4* t = (const int4*)(lut + (size_t)(head0 + h) * kCodewords) + 2 * tid;
      const int4 x = t[0], y = t[1];
      tv[h][0] = x.x, tv[h][1] = x.y, tv[h][2] = x.z, tv[h][3] = x.w;
      tv[h][4] = y.x, tv[h][5] = y.y, tv[h][6] = y.z, tv[h][7] = y.w;
    }
    uint32_t tot[kCsPer], before[kCsPer];
#pragma unroll
    for (int i = 0; i < kCsPer; ++i) tot[i] = before[i] = 0u;
#pragma unroll 1
    for (int p0 = 0; p0 < n_part; p0 += 4) {
      uint4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = cnt[(size_t)min(p0 + u, n_part - 1) * (kCodewords / 8)];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t w[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
        const uint32_t in = p0 + u < n_part ? 0xffffu : 0u, pre = p0 + u < chunk ? 0xffffu : 0u;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          tot[2 * i] += w[i] & in;
          tot[2 * i + 1] += (w[i] >> 16) & in;
          before[2 * i] += w[i] & pre;
          before[2 * i + 1] += (w[i] >> 16) & pre;
        }
      }
    }
#pragma unroll
    for (int r = 0; r < kLoads; ++r)
      if (r < loads)
        cv[r] = cc.aligned ? load_codes8<true>(seq_codes, j0 + r * kPerThread, row_len)
                           : load_codes8<false>(seq_codes, j0 + r * kPerThread, row_len);
    for (int i = tid; i < H * kHistBins / 4; i += NT) ((uint4*)&L.hist[0][0])[i] = make_uint4(0u, 0u, 0u, 0u);
    if (tid < H) {
      L.small_n[tid] = 0u;
      L.before_gt[tid] = 0u;
      L.before_eq[tid] = 0u;
    }
    __syncthreads();
    // --- a level of 2048 bins linear in the score, as in select_single_kernel
    float s_lo[H], lin_scale[H];
    uint32_t use_lin = 0, k_lo[H], k_hi[H];
#pragma unroll
    for (int h = 0; h < H; ++h) {
      if (h >= n_real) break;
      const uint2 mine = range[h];
      k_lo[h] = ~(uint32_t)__builtin_amdgcn_readfirstlane((int)row16_most(mine.x));
      k_hi[h] = (uint32_t)__builtin_amdgcn_readfirstlane((int)row16_most(mine.y));
      s_lo[h] = key_to_float(key_score(k_lo[h]));
      const float span = key_to_float(key_score(k_hi[h])) - s_lo[h];
      const bool ok = span >= 1e-30f && span < INFINITY;
      lin_scale[h] = ok ? (float)kHistBins / span : 0.f;
      use_lin |= ok ? 1u << h : 0u;
    }
    auto lin_bin = [&](int h, int i) {
      return (uint32_t)min((int)((key_to_float(tv[h][i]) - s_lo[h]) * lin_scale[h]), kHistBins - 1);
    };
#pragma unroll
    for (int h = 0; h < H; ++h) {
      if (h >= n_real) break;
      if ((use_lin >> h) & 1u) {
#pragma unroll
        for (int i = 0; i < kCsPer; ++i)
          if (tot[i]) atomicAdd(&L.hist[h][lin_bin(h, i)], tot[i]);
      }
    }
    __syncthreads();
    if (wave < n_real && ((use_lin >> wave) & 1u)) {
      uint32_t bin, above;
      wave_rank(L.hist[wave], (uint32_t)sr.kk, lane, bin, above);
      if (lane == 0) {
        L.bin[wave] = bin;
        L.k_rem[wave] = (uint32_t)sr.kk - above;
      }
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < H; ++h) {
      if (h >= n_real) break;
      if ((use_lin >> h) & 1u) {
        const uint32_t bin = L.bin[h];
#pragma unroll
        for (int i = 0; i < kCsPer; ++i)
          if (tot[i] && lin_bin(h, i) == bin) {
            const uint32_t at = atomicAdd(&L.small_n[h], 1u);
            if (at < (uint32_t)kSmallSel) {
              L.small_key[h][at] = score_key(tv[h][i]);
              L.small_w[h][at] = tot[i];
            }
          }
      }
    }
    __syncthreads();
    if (wave < n_real && ((use_lin >> wave) & 1u)) {
      const uint32_t n_small = L.small_n[wave], rem = L.k_rem[wave];
      if (n_small <= (uint32_t)kSmallSel) {
        for (uint32_t m = lane; m < n_small; m += 64) {
          const uint32_t key = L.small_key[wave][m];
          uint32_t gt = 0, eq = 0;
          for (uint32_t u = 0; u < n_small; ++u) {
            const uint32_t ku = L.small_key[wave][u], wu = L.small_w[wave][u];
            gt += ku > key ? wu : 0u;
            eq += ku == key ? wu : 0u;
          }
          if (gt < rem && rem <= gt + eq) {   // every member at the K-th key writes the same two words
            L.kth[wave] = key;
            L.k_rem[wave] = rem - gt;   // (read by all lanes above)
          }
        }
      }
    }
    __syncthreads();
    // --- a crowded bin, or a table whose range is empty or not finite: an MSB-first radix select on the keys
#pragma unroll
    for (int h = 0; h < H; ++h) {
      if (h >= n_real) break;
      const bool lin = (use_lin >> h) & 1u;
      if (lin && L.small_n[h] <= (uint32_t)kSmallSel) continue;   // (uniform)
      const uint32_t bin1 = lin ? L.bin[h] : 0u;
      uint32_t rem = lin ? L.k_rem[h] : (uint32_t)sr.kk, prefix = 0, mask = 0;
      int remaining = 32 - __clz(k_hi[h] - k_lo[h]);
#pragma unroll 1
      while (remaining > 0) {
        const int bits = remaining < 11 ? remaining : 11, shift = remaining - bits;
        const uint32_t dmask = (1u << bits) - 1u;
        __syncthreads();   // the histogram may still be read
        for (int i = tid; i < kHistBins; i += NT) L.hist[h][i] = 0;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kCsPer; ++i) {
          const uint32_t rel = score_key(tv[h][i]) - k_lo[h];
          if (tot[i] && (!lin || lin_bin(h, i) == bin1) && (rel & mask) == prefix)
            atomicAdd(&L.hist[h][(rel >> shift) & dmask], tot[i]);
        }
        __syncthreads();
        block_find_rank_desc<NT, kHistBins>([&](int i) { return L.hist[h][i]; }, rem, L.wave_a, L.res);
        rem -= L.res[1];
        prefix |= L.res[0] << shift;
        mask |= dmask << shift;
        remaining = shift;
      }
      __syncthreads();
      if (tid == 0) {
        L.kth[h] = prefix + k_lo[h];
        L.k_rem[h] = rem;
      }
      __syncthreads();
    }
    // --- flags of the codewords, and the candidates above and at the K-th key in the chunks before
    uint32_t fl[kCsPer];
#pragma unroll
    for (int i = 0; i < kCsPer; ++i) fl[i] = 0u;
#pragma unroll
    for (int h = 0; h < H; ++h) {
      if (h >= n_real) break;
      const uint32_t kth = L.kth[h];
      k_rem[h] = L.k_rem[h];
      uint32_t gt = 0, eq = 0;
#pragma unroll
      for (int i = 0; i < kCsPer; ++i) {
        const uint32_t key = score_key(tv[h][i]);
        fl[i] |= key > kth ? 1u << (kBits * h) : (key == kth ? 0x10000u << (kBits * h) : 0u);
        gt += key > kth ? before[i] : 0u;
        eq += key == kth ? before[i] : 0u;
      }
      if (chunk > 0) {
        gt = wave_inclusive_scan(gt);
        eq = wave_inclusive_scan(eq);
        if (lane == 63) {
          if (gt) atomicAdd(&L.before_gt[h], gt);
          if (eq) atomicAdd(&L.before_eq[h], eq);
        }
      }
    }
    ((uint4*)L.flags)[2 * tid] = make_uint4(fl[0], fl[1], fl[2], fl[3]);
    ((uint4*)L.flags)[2 * tid + 1] = make_uint4(fl[4], fl[5], fl[6], fl[7]);
    __syncthreads();
    // --- flags of this thread's tokens, kBits of them to a word
#pragma unroll
    for (int r = 0; r < kLoads; ++r)
      if (r < loads) {
#pragma unroll
        for (int i = 0; i < kPerThread; ++i)
          acc[(r * kPerThread + i) / kBits] |= L.flags[code_of(cv[r], i)] << ((r * kPerThread + i) % kBits);
      }
  }
  // which of them are candidates, above the K-th key, equal to it: 32 tokens a word
  uint32_t above[H][kWords], equal[H][kWords], pre[H];
#pragma unroll
  for (int w = 0; w < kWords; ++w) {
    const int a = min(max(lo - j0 - 32 * w, 0), 32), e = min(max(min(hi - j0, loads * kPerThread) - 32 * w, 0), 32);
    const uint32_t valid = e > a ? (uint32_t)((1ull << e) - (1ull << a)) : 0u;
#pragma unroll
    for (int h = 0; h < H; ++h) {
      uint32_t g = 0, q_ = 0;
#pragma unroll
      for (int q = 0; q < 32 / kBits; ++q) {
        const uint32_t word = acc[w * (32 / kBits) + q];
        g |= ((word >> (kBits * h)) & ((1u << kBits) - 1u)) << (kBits * q);
        q_ |= ((word >> (16 + kBits * h)) & ((1u << kBits) - 1u)) << (kBits * q);
      }
      above[h][w] = take_all ? valid : g & valid;
      equal[h][w] = take_all ? 0u : q_ & valid;
    }
  }
#pragma unroll
  for (int h = 0; h < H; ++h) {
    if (h >= n_real) break;
    uint32_t own = 0;
#pragma unroll
    for (int w = 0; w < kWords; ++w) own += (uint32_t)__popc(above[h][w]) | (uint32_t)__popc(equal[h][w]) << 16;
    const uint32_t inc = wave_inclusive_scan(own);   // (a chunk's counts fit 16 bits)
    pre[h] = inc - own;
    if (lane == 63) L.wave_tot[h][wave] = inc;
  }
  __syncthreads();
  // --- the winners of this chunk in ascending position
#pragma unroll
  for (int h = 0; h < H; ++h) {
    if (h >= n_real) break;
    uint32_t p = pre[h];
    for (int w = 0; w < wave; ++w) p += L.wave_tot[h][w];
    uint32_t gt_before = (take_all ? (uint32_t)max(s0 - lo, 0) : L.before_gt[h]) + (p & 0xffffu);
    uint32_t eq_before = (take_all ? 0u : L.before_eq[h]) + (p >> 16);
    int32_t* oi = topk_idx + (size_t)(head0 + h) * top_k;
#pragma unroll
    for (int w = 0; w < kWords; ++w) {
      uint32_t e_take = 0;
      if (equal[h][w] && eq_before < k_rem[h]) {
        const uint32_t room = k_rem[h] - eq_before;
        e_take = equal[h][w];
        if ((uint32_t)__popc(e_take) > room) {   // keep the lowest `room` set bits
#pragma unroll 1
          for (uint32_t drop = (uint32_t)__popc(e_take) - room; drop; --drop) e_take &= ~(0x80000000u >> __clz(e_take));
        }
      }
      uint32_t m = above[h][w] | e_take, slot = gt_before + min(eq_before, k_rem[h]);
#pragma unroll 1
      for (; m; m &= m - 1, ++slot) {
        const int at = j0 + 32 * w + __ffs(m) - 1;
        if (slot < (uint32_t)sr.kk) {   // (always, of consistent counts)
          oi[slot] = at;
          if (topk_score)
            topk_score[(size_t)(head0 + h) * top_k + slot] =
                key_to_float(lut[(size_t)(head0 + h) * kCodewords + (seq_codes[at] & (kCodewords - 1))]);
        }
      }
      gt_before += (uint32_t)__popc(above[h][w]);
      eq_before += (uint32_t)__popc(equal[h][w]);
    }
  }
}

// How many heads a workgroup of the selection takes and how long the chunks are.  What a workgroup does whatever its chunk
// (adding up the counts, the K-th keys) costs more than the chunk's own tokens, but less for a further head than for a first
// one.  So the chunks are long and the heads of a workgroup few, while there are CUs for all, and shorter only where CUs
// would be idle.  Steps of 32 query and 8 KV heads, us, heads / tokens of a workgroup: 4 sequences of 131072 tokens 1 / 8192
// 86, 1 / 16384 69.5, 2 / 16384 64.7, 4 / 16384 66.7; one of 131072 1 / 8192 43.4, 1 / 16384 39.7, 2 / 16384 42.3; one of
// 32768 1 / 4096 38.7, 1 / 16384 61; 64 of 16384 1 / 16384 232, 2 / 16384 228, 4 / 16384 224.
struct ChunkPlan {
  int heads, tokens, n;
  size_t off_ranges, bytes;   // of the counts; of counts and ranges
};
static ChunkPlan plan_chunks(const a2ats_dims& d, int window, int n_sink) {
  const int G = d.n_q_heads / d.n_kv_heads;
  const long rows = (long)d.batch * d.n_kv_heads, win = d.ctx_len > window ? d.ctx_len - window : 0;
  const long span = std::max<long>(1, win - (std::min<long>(n_sink, win) & ~(long)(kPerThread - 1)));
  ChunkPlan p;
  auto groups = [&](int heads, int tokens) { return rows * ((G + heads - 1) / heads) * ((span + tokens - 1) / tokens); };
  p.heads = groups(1, kMaxChunk) <= 256 ? 1 : (groups(2, kMaxChunk) <= 512 ? 2 : 4);
  p.tokens = kMaxChunk / 4;
  while (p.tokens < kMaxChunk && groups(p.heads, p.tokens) > 256) p.tokens *= 2;
  p.n = (int)((span + p.tokens - 1) / p.tokens);
  p.off_ranges = (size_t)rows * p.n * kCodewords * sizeof(uint16_t);
  p.bytes = p.off_ranges + (size_t)d.batch * d.n_q_heads * kEncodeSlices * sizeof(uint2);
  return p;
}

// Every workgroup adds up the counts of all chunks, so the work grows with the square of the context, and with many heads at long
// contexts a workgroup a head, which counts by itself, is the faster way (two calls).  Both times but for what they have in
// common, us, from steps without the attention of 1 to 128 sequences, 8 to 1024 heads, 16384 to 1048576 tokens; a workgroup
// by itself holds the codes of 131072 tokens and reads those of more again.  Two calls -> by chunk: 32 sequences of 8 KV heads
// with one query head each, 65536 tokens 49.8 -> 45.2, 131072 59.2 -> 69.0, 1048576 259 -> 759; 128 of these 158 -> 151, 208 -> 263;
// 16 of them 262144 tokens 74 -> 68, 524288 116 -> 138; four heads each, 16 sequences, 524288 256 -> 205, 1048576 457 -> 514;
// one sequence 1048576 181 -> 47.
bool select_chunks_single_fits(const a2ats_dims& d, int window, int n_sink, size_t scratch_bytes) {
  const ChunkPlan p = plan_chunks(d, window, n_sink);
  const int G = d.n_q_heads / d.n_kv_heads;
  const double wgs = (double)d.batch * d.n_kv_heads * ((G + p.heads - 1) / p.heads) * p.n;
  const double by_chunk = wgs * (0.0215 + 0.004 * (std::min(G, p.heads) - 1) + 0.0003 * p.n);
  const double heads = (double)d.batch * d.n_q_heads, n = (double)p.n * p.tokens / kMaxChunk;
  const double by_head = 10 + 0.06 * heads + n * (n <= 8 ? 1.6 : 3.0) * std::max(1.0, heads / 256);
  return p.bytes <= scratch_bytes && by_chunk <= by_head;
}

hipError_t launch_decode_select_single(const a2ats_dims& d, const void* q, int q_dtype, const float* cos_b,
                                       const float* sin_b, const float* codebook, float* q_rot, int32_t* lut,
                                       float* lut_scale, const FewKeys& few, int pos0, void* codes, int top_k, int window,
                                       int n_sink, const int32_t* seq_lens, int32_t* topk_idx, int32_t* topk_count,
                                       float* topk_score, void* scratch, hipStream_t stream) {
  const int G = d.n_q_heads / d.n_kv_heads, rows = d.batch * d.n_kv_heads;
  if (rows == 0) return hipSuccess;
  const ChunkPlan p = plan_chunks(d, window, n_sink);
  CodeCount cc;
  cc.counts = (uint16_t*)scratch;
  cc.ranges = (uint2*)((unsigned char*)scratch + p.off_ranges);
  cc.gm = make_grid_map(p.n, rows, 1, d.n_kv_heads);
  cc.tokens = p.tokens;
  cc.aligned = codes_aligned(d, codes);
  const hipError_t err = launch_tables_single(d, q, q_dtype, cos_b, sin_b, codebook, q_rot, lut, lut_scale, false, few,
                                              cc, rows * p.n, codes, seq_lens, top_k, window, n_sink, stream);
  if (err != hipSuccess) return err;
  const int groups = (G + p.heads - 1) / p.heads;
#define A2ATS_LAUNCH_CHUNKS(H)                                                                                          \
  hipLaunchKernelGGL(select_chunks_single_kernel<H>, dim3(rows * groups * p.n), dim3(kCsThreads), 0, stream,            \
                     (uint16_t*)codes, lut, seq_lens, topk_idx, topk_count, topk_score, cc,                             \
                     make_grid_map(p.n, rows * groups, groups, d.n_kv_heads), few.part, few.keys ? few.n_new : 0, pos0, \
                     d.n_q_heads, d.n_kv_heads, d.ctx_len, d.ctx_stride, top_k, window, n_sink)
  if (p.heads == 1) A2ATS_LAUNCH_CHUNKS(1);
  else if (p.heads == 2) A2ATS_LAUNCH_CHUNKS(2);
  else A2ATS_LAUNCH_CHUNKS(4);
#undef A2ATS_LAUNCH_CHUNKS
  return hipGetLastError();
}

// Debug / parity: every token's score as float.
__global__ __launch_bounds__(256) void score_dense_single_kernel(
    const uint16_t* __restrict__ codes, const int32_t* __restrict__ lut, const int32_t* __restrict__ seq_lens,
    float* __restrict__ scores_out, int Hq, int Hkv, int ctx_len, int64_t ctx_stride) {
  const int bh = blockIdx.y, b = bh / Hq, h = bh % Hq, G = Hq / Hkv, kv = h / G;
  int n = seq_lens ? seq_lens[b] : ctx_len;
  n = n < 0 ? 0 : (n > ctx_len ? ctx_len : n);
  const uint16_t* seq_codes = codes + ((size_t)b * Hkv + kv) * ctx_stride;
  const int32_t* table = lut + (size_t)bh * kCodewords;
  for (int j = blockIdx.x * 256 + threadIdx.x; j < n; j += gridDim.x * 256)
    scores_out[(size_t)bh * ctx_stride + j] = key_to_float(table[seq_codes[j] & (kCodewords - 1)]);
}

hipError_t launch_score_topk_single(const a2ats_dims& d, const void* codes, const int32_t* lut, int top_k,
                                    int window, int n_sink, const int32_t* seq_lens, int32_t* topk_idx,
                                    int32_t* topk_count, float* topk_score, float* scores_out,
                                    hipStream_t stream) {
  const int heads = d.batch * d.n_q_heads;
  if (heads == 0) return hipSuccess;
  if (scores_out) {
    int gx = (d.ctx_len + 256 * 8 - 1) / (256 * 8);
    if (gx < 1) gx = 1;
    hipLaunchKernelGGL(score_dense_single_kernel, dim3(gx, heads), dim3(256), 0, stream,
                       (const uint16_t*)codes, lut, seq_lens, scores_out, d.n_q_heads, d.n_kv_heads,
                       d.ctx_len, d.ctx_stride);
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
  }
  const bool aligned = codes_aligned(d, codes);
  if (aligned)
    hipLaunchKernelGGL(select_single_kernel<true>, dim3(heads), dim3(kSelThreads), 0, stream,
                       (const uint16_t*)codes, lut, seq_lens, topk_idx, topk_count, topk_score, d.n_q_heads,
                       d.n_kv_heads, d.ctx_len, d.ctx_stride, top_k, window, n_sink);
  else
    hipLaunchKernelGGL(select_single_kernel<false>, dim3(heads), dim3(kSelThreads), 0, stream,
                       (const uint16_t*)codes, lut, seq_lens, topk_idx, topk_count, topk_score, d.n_q_heads,
                       d.n_kv_heads, d.ctx_len, d.ctx_stride, top_k, window, n_sink);
  return hipGetLastError();
}

}  // namespace a2ats
