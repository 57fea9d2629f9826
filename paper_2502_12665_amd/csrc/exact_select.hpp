// Exact scores of code rows from a head's 32-bit table in LDS, and the exact route of a2ats_score_topk:
// the top-K of one head by one workgroup (select_exact_kernel, and the fallback of the other routes).
#pragma once
#include "common.hpp"

namespace a2ats {

constexpr int kExactThreads = 1024;
constexpr int kSmallList = 1024;     // members of the K-th key's bin ranked by brute force

// ------------------------------------------------------------------------------------------
// Scoring primitives
// ------------------------------------------------------------------------------------------

// Exact score of one token for one head.  The head's table sits in LDS with one 256-byte row per
// centroid id c; the 4-byte entry of subspace m is at byte m << 2 of the row (M = 32), or, for
// M = 16, twice: at m << 2 and at 64 + (m << 2).  LDS serves a 4-byte read 32 lanes at a time.
// Lane L visits the subspaces of its row in the order m = t ^ (L & 15) within a 16-byte half row,
// and lanes 16..31 of each half-wave use the second copy (M = 16) or take the two half rows in the
// other order (M = 32): the 32 lanes served together then touch 32 different banks whatever the
// code bytes are (a [m][c] table would spread them at random: ~3.5 lanes on the busiest bank).
// The visiting order does not change the result because the scores are integer sums.
constexpr int kExactLdsBytes = kCentroids * 256;

template <int M, int NT>
__device__ __forceinline__ void load_exact_table(const int32_t* __restrict__ head_table, unsigned char* tbl) {
  const int4* src = (const int4*)head_table;   // [256 c][M] int32
#pragma unroll 4
  for (int e = threadIdx.x; e < kCentroids * M / 4; e += NT) {
    const int c = e / (M / 4), mq = e % (M / 4);
    const int4 v = src[e];
    *(int4*)(tbl + (c << 8) + (mq << 4)) = v;
    if (M == 16) *(int4*)(tbl + (c << 8) + 64 + (mq << 4)) = v;
  }
}

template <int M>
struct ExactSwizzle {
  uint32_t mc[M / 4];   // byte t&3 of mc[t>>2]: low address byte for step t of this lane
  uint32_t sel[4];      // v_perm selectors: address byte 1 <- code byte (k ^ b), byte 0 <- mc byte k
  bool swap1, swap2;    // dword index inside a half row is XORed with (rho >> 2)
  bool swaph;           // M = 32: this lane takes the two half rows in the other order
  __device__ __forceinline__ void init(int lane) {
    const uint32_t rho = lane & 15, b = rho & 3, hi = (lane >> 4) & 1;
#pragma unroll
    for (int d = 0; d < M / 4; ++d) {
      uint32_t v = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t t = 4 * d + k;
        const uint32_t m_low = (t ^ rho) & 15u, half = t >> 4;
        const uint32_t byte = M == 16 ? ((hi << 6) | (m_low << 2)) : ((((half ^ hi) << 4) | m_low) << 2);
        v |= byte << (8 * k);
      }
      mc[d] = v;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) sel[k] = 0x0c0c0000u | ((4u + ((uint32_t)k ^ b)) << 8) | (uint32_t)k;
    swap1 = (rho >> 2) & 1;
    swap2 = (rho >> 3) & 1;
    swaph = M == 32 && hi;
  }
};

template <int M>
__device__ __forceinline__ int32_t score_exact(const uint4 (&w)[M / 16], const unsigned char* tbl,
                                               const ExactSwizzle<M>& sw) {
  int32_t s = 0;
#pragma unroll
  for (int qd = 0; qd < M / 16; ++qd) {
    uint4 h = w[qd];
    if (M == 32) {
      const uint4 o = w[(M / 16 - 1) - qd];
      h = make_uint4(sw.swaph ? o.x : h.x, sw.swaph ? o.y : h.y, sw.swaph ? o.z : h.z, sw.swaph ? o.w : h.w);
    }
    const uint32_t x0 = sw.swap1 ? h.y : h.x, x1 = sw.swap1 ? h.x : h.y;
    const uint32_t x2 = sw.swap1 ? h.w : h.z, x3 = sw.swap1 ? h.z : h.w;
    const uint32_t z[4] = {sw.swap2 ? x2 : x0, sw.swap2 ? x3 : x1, sw.swap2 ? x0 : x2, sw.swap2 ? x1 : x3};
#pragma unroll
    for (int t = 0; t < 16; ++t) {
      const uint32_t off = __builtin_amdgcn_perm(z[t >> 2], sw.mc[qd * 4 + (t >> 2)], sw.sel[t & 3]);
      s += *(const int32_t*)(tbl + off);
    }
  }
  return s;
}

template <int M>
__device__ __forceinline__ int32_t score_exact_row(const uint8_t* row, const unsigned char* tbl,
                                                   const ExactSwizzle<M>& sw) {
  uint4 w[M / 16];
#pragma unroll
  for (int qd = 0; qd < M / 16; ++qd) w[qd] = *(const uint4*)(row + qd * 16);
  return score_exact<M>(w, tbl, sw);
}

// ------------------------------------------------------------------------------------------
// Exact route (also the fallback of the fast route)
// ------------------------------------------------------------------------------------------
constexpr int kKeepRows = 16;   // rows per thread the exact route keeps in registers (16384 candidates)
struct ExactLds {
  uint32_t hist[kHistBins];
  uint32_t wave_a[kExactThreads / 64];
  uint32_t wave_b[kExactThreads / 64];
  uint32_t res[2];
  // emission with resident keys: packed (above, equal) counts per round and wave, their exclusive
  // prefixes over the waves of a round, and the rounds' totals
  uint32_t round_wave[kKeepRows][kExactThreads / 64];
  uint32_t round_pre[kKeepRows][kExactThreads / 64];
  uint32_t round_tot[kKeepRows];
  // the keys of the K-th key's bin after a select level, when they are few enough to rank by counting
  uint32_t small_n;
  uint32_t small_key[kSmallList];
};

// One count more in hist[bin] for every lane that is `in`, where few bins hold most of a wave (what lies below the bounds,
// above them, and the tied scores): the lanes of three bins are added up, as atomics of a wave on one address take their
// turns.
__device__ __forceinline__ void count_shared_bins(uint32_t* hist, uint32_t bin, bool in) {
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const uint64_t left = __builtin_amdgcn_ballot_w64(in);
    if (!left) return;
    const int leader = (int)__builtin_ctzll(left);
    const uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int)bin, leader);
    const bool same = in && bin == first;
    const uint32_t n = (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(same));
    if (lane_id() == leader) atomicAdd(&hist[first], n);
    in = in && !same;
  }
  if (in) atomicAdd(&hist[bin], 1u);
}

// Exact top-K for one head by the whole workgroup.  `head_table` is the head's [c][m] table in
// global memory, s_lo and s_hi bounds of any score, `tbl` kExactLdsBytes of LDS.  Writes
// out_idx[0..kk) ascending (and out_score); the caller has written the count and the -1 padding.
// Requires sr.kk >= 1.
// TIES: many rows are expected to have one score, and s_lo and s_hi are bounds of the K-th; out_score is not written.
// TABLE_IN_LDS: the caller has put the head's table at `tbl` (a barrier follows here).
// ROWS: most rows per thread that stay in registers.
template <int M, bool TIES = false, bool TABLE_IN_LDS = false, int ROWS = kKeepRows>
__device__ void exact_select_block(const SeqCodes& seq_codes,
                                   const int32_t* __restrict__ head_table,
                                   int32_t s_lo, int32_t s_hi, float scale,
                                   const SeqRange& sr, int32_t* __restrict__ out_idx,
                                   float* __restrict__ out_score, unsigned char* tbl, ExactLds& L) {
  constexpr int NT = kExactThreads;
  const int tid = threadIdx.x;
  if (TIES) {   // one to either side for what lies beyond
    s_lo = (int32_t)((uint32_t)s_lo - 1u);
    s_hi = (int32_t)((uint32_t)s_hi + 1u);
  }
  ExactSwizzle<M> sw;
  sw.init(tid & 63);
  __syncthreads();   // tbl may alias LDS the caller was still reading
  if (!TABLE_IN_LDS) {
    load_exact_table<M, NT>(head_table, tbl);
    __syncthreads();
  }

  const int lo = sr.sink_end, hi = sr.win_start;
  uint32_t kth = 0, k_rem = (uint32_t)sr.kk;   // kth: relative
  // Radix digits are taken from key - key(lower bound of any score), so that the histogram bins
  // spread over the occupied range instead of all keys sharing their leading bits.
  // Relative keys are compared in the bits that the histograms look at.  For a table of finite numbers those are all that
  // they have; with an infinite query the entries saturate and their sums wrap, and then this is what makes every level
  // and the emission agree on one order, so that exactly kk winners are written whatever it is worth.
  const uint32_t k_lo = score_key(s_lo), range = score_key(s_hi) - k_lo;
  const uint32_t in_range = range == 0u ? 0u : ~0u >> __clz(range);
  auto key_of = [&](int32_t score) { return (score_key(TIES ? min(max(score, s_lo), s_hi) : score) - k_lo) & in_range; };
  auto relative_key = [&](int j) { return key_of(score_exact_row<M>(row_ptr<M>(seq_codes, j), tbl, sw)); };
  // Up to kKeep rows per thread (16384 candidates: every shape that takes this route for its length)
  // are scored once and their relative keys kept in registers; the select levels and the emission
  // then work on those instead of streaming and scoring the rows again (4 passes at 4096 tokens:
  // 23 us).  Thread t owns rows lo + t + i NT, the order of the streaming loops below.
  constexpr int kKeep = ROWS;
  const bool resident = hi - lo <= kKeep * NT;   // (uniform)
  uint32_t keys[kKeep];
  if (resident && kKeep * M <= 128) {   // all rows are requested before the first is scored
    uint4 w[kKeep][M / 16];
#pragma unroll
    for (int i = 0; i < kKeep; ++i) {
      const uint4* row = (const uint4*)row_ptr<M>(seq_codes, min(lo + tid + i * NT, hi - 1));
#pragma unroll
      for (int qd = 0; qd < M / 16; ++qd) w[i][qd] = row[qd];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < kKeep; ++i) {
      const uint32_t key = key_of(score_exact<M>(w[i], tbl, sw));
      keys[i] = lo + tid + i * NT < hi ? key : 0u;
    }
  } else if (resident) {
#pragma unroll
    for (int i = 0; i < kKeep; ++i) {
      const int j = lo + tid + i * NT;
      keys[i] = j < hi ? relative_key(j) : 0u;
    }
  }
  if (sr.kk < sr.ncand) {
    int remaining = 32 - __clz(range);   // significant bits of a relative key
    uint32_t prefix = 0, mask = 0;
#pragma unroll 1
    while (remaining > 0) {
      const int bits = remaining < 11 ? remaining : 11;
      const int shift = remaining - bits;
      const uint32_t dmask = (1u << bits) - 1u;
      for (int i = tid; i < kHistBins; i += NT) L.hist[i] = 0;
      __syncthreads();
      if (resident) {
#pragma unroll
        for (int i = 0; i < kKeep; ++i) {
          const bool in = lo + tid + i * NT < hi && (keys[i] & mask) == prefix;
          if (TIES) count_shared_bins(L.hist, (keys[i] >> shift) & dmask, in);
          else if (in) atomicAdd(&L.hist[(keys[i] >> shift) & dmask], 1u);
        }
      } else {
        for (int j = lo + tid; j < hi; j += NT) {
          const uint32_t key = relative_key(j);
          if ((key & mask) == prefix) atomicAdd(&L.hist[(key >> shift) & dmask], 1u);
        }
      }
      __syncthreads();
      block_find_rank_desc<NT, kHistBins>([&](int i) { return L.hist[i]; }, k_rem, L.wave_a, L.res);
      const uint32_t bin = L.res[0], above = L.res[1], m_bin = L.hist[bin];
      k_rem -= above;
      prefix |= bin << shift;
      mask |= dmask << shift;
      remaining = shift;
      if (tid == 0) L.small_n = 0;
      __syncthreads();
      // (counting takes about 0.1 us per member, a further level 3 us)
      if (resident && remaining > 0 && m_bin <= (uint32_t)(TIES ? 32 : kSmallList)) {   // (uniform)
        // The bin of the K-th key usually holds a handful of keys: they are listed and each member
        // counts the members above and at its own key -- the member whose range contains k_rem is the
        // K-th key.  (A crowded bin, heavy ties, goes on with the next radix level.)
#pragma unroll
        for (int i = 0; i < kKeep; ++i)
          if (lo + tid + i * NT < hi && (keys[i] & mask) == prefix) L.small_key[atomicAdd(&L.small_n, 1u)] = keys[i];
        __syncthreads();
        if ((uint32_t)tid < m_bin) {
          const uint32_t key = L.small_key[tid];
          uint32_t gt = 0, eq = 0;
          for (uint32_t u = 0; u < m_bin; ++u) {
            const uint32_t ku = L.small_key[u];
            gt += ku > key ? 1u : 0u;
            eq += ku == key ? 1u : 0u;
          }
          if (gt < k_rem && k_rem <= gt + eq) {   // every member at the K-th key writes the same two words
            L.res[0] = key;
            L.res[1] = k_rem - gt;
          }
        }
        __syncthreads();
        prefix = L.res[0];
        k_rem = L.res[1];
        remaining = 0;
        __syncthreads();   // L.res is rewritten by the caller's next use
      }
    }
    kth = prefix;
  }

  // Ordered emission: keys above the K-th, plus the first k_rem positions that equal it.
  uint32_t eq_seen = 0, out_n = 0;
  const bool take_all = sr.kk >= sr.ncand;
  auto emit_round = [&](int base, bool& done) {
    const int j = base + tid;
    uint32_t key = 0, gt = 0, eq = 0;
    if (j < hi) {
      key = relative_key(j);
      gt = take_all ? 1u : (key > kth ? 1u : 0u);
      eq = take_all ? 0u : (key == kth ? 1u : 0u);
    }
    uint32_t tot_eq, tot_sel;
    const uint32_t ex_eq = block_exclusive_scan<NT>(eq, L.wave_a, tot_eq);
    const uint32_t sel = gt | ((eq && (eq_seen + ex_eq < k_rem)) ? 1u : 0u);
    const uint32_t ex_sel = block_exclusive_scan<NT>(sel, L.wave_b, tot_sel);
    if (sel) {
      const uint32_t pos = out_n + ex_sel;
      out_idx[pos] = j;
      if (!TIES && out_score) out_score[pos] = (float)key_score(key + k_lo) * scale;
    }
    eq_seen += tot_eq;
    out_n += tot_sel;
    done = out_n >= (uint32_t)sr.kk;   // (uniform)
  };
  bool done = false;
  if (resident) {
    // All rounds at once: a wave scan of the packed (above, equal) flags per round, one scan over the
    // waves of every round (16 lanes per round), then each thread places its winners -- two barriers
    // instead of four per round.  A winner's slot is the number of keys above the K-th before it plus
    // the number of equal keys before it that still fit (both counts grow with the position).
    constexpr int NW = NT / 64;
    static_assert(kKeep * NW <= NT && NW == 16, "one lane per (round, wave), 16 waves per round");
    const int lane = tid & 63, wave = tid >> 6;
    uint32_t flags = 0;        // bit 2 i: above the K-th key, bit 2 i + 1: equal to it
    uint32_t pre[kKeep];
#pragma unroll
    for (int i = 0; i < kKeep; ++i) {
      uint32_t own = 0;
      if (lo + tid + i * NT < hi) {
        const uint32_t key = keys[i];
        own = take_all ? 1u : (key > kth ? 1u : (key == kth ? 0x10000u : 0u));
      }
      flags |= ((own & 1u) | ((own >> 16) << 1)) << (2 * i);
      const uint32_t v = wave_inclusive_scan(own);
      pre[i] = v - own;
      if (lane == 63) L.round_wave[i][wave] = v;
    }
    __syncthreads();
    if (tid < kKeep * NW) {
      const int i = tid / NW, w = tid % NW;
      const uint32_t own = L.round_wave[i][w];
      uint32_t v = own;
#pragma unroll
      for (int off = 1; off < NW; off <<= 1) {
        const uint32_t n = __shfl_up(v, off, NW);
        if (w >= off) v += n;
      }
      L.round_pre[i][w] = v - own;
      if (w == NW - 1) L.round_tot[i] = v;
    }
    __syncthreads();
    uint32_t gt_base = 0, eq_base = 0;
#pragma unroll
    for (int i = 0; i < kKeep; ++i) {
      const uint32_t f = (flags >> (2 * i)) & 3u;
      if (f) {
        const uint32_t p = pre[i] + L.round_pre[i][wave];
        const uint32_t gt_before = gt_base + (p & 0xffffu), eq_before = eq_base + (p >> 16);
        if ((f & 1u) || eq_before < k_rem) {
          const uint32_t slot = gt_before + min(eq_before, k_rem);
          out_idx[slot] = lo + tid + i * NT;
          if (!TIES && out_score) out_score[slot] = (float)key_score(keys[i] + k_lo) * scale;
        }
      }
      const uint32_t tot = L.round_tot[i];
      gt_base += tot & 0xffffu;
      eq_base += tot >> 16;
    }
  } else {
#pragma unroll 1
    for (int base = lo; base < hi && !done; base += NT) emit_round(base, done);
  }
}

// The same by as many rounds of rows as the sequence needs: rounds that hold none take their time all the same, in the scans
// above all, and where there are few, all are requested at once (4 heads of 4096 candidates in decode_select_head_kernel 16.4
// -> 12.7 us, 32 of 6370 with M = 32 21.9 -> 19.5).  The longest come first in the code: behind the others they take 0.25 us more.
template <int M, bool TABLE_IN_LDS>
__device__ __forceinline__ void exact_select_sized(const SeqCodes& seq_codes, const int32_t* head_table, int32_t s_lo,
                                                   int32_t s_hi, float scale, const SeqRange& sr, int32_t* out_idx,
                                                   float* out_score, unsigned char* tbl, ExactLds& L) {
  if (__builtin_expect(sr.ncand > 8 * kExactThreads, 1))   // (uniform)
    exact_select_block<M, false, TABLE_IN_LDS>(seq_codes, head_table, s_lo, s_hi, scale, sr, out_idx, out_score, tbl, L);
  else if (sr.ncand > 4 * kExactThreads)
    exact_select_block<M, false, TABLE_IN_LDS, 8>(seq_codes, head_table, s_lo, s_hi, scale, sr, out_idx, out_score, tbl, L);
  else
    exact_select_block<M, false, TABLE_IN_LDS, 4>(seq_codes, head_table, s_lo, s_hi, scale, sr, out_idx, out_score, tbl, L);
}

}  // namespace a2ats
