// The top-K of the (up to) four query heads of a group by one workgroup, for sequences whose candidates fit
// its registers (at most 16384): the group route of a2ats_score_topk.
//
// Every row is scored once for the four heads (one 8-byte LDS read per code byte, coarse_score.hpp) and the
// coarse scores stay in registers.  A histogram over them gives, per head, the 32-wide bin of the K-th largest
// coarse score, and since exact = base + (coarse << s) + rem with 0 <= rem < M 2^s
//   - a row at least M units above that bin is a winner: every row with a score as high has a coarse score
//     above the bin, and there are fewer than K of those;
//   - a row at least M units below the bin is not: K rows have coarse scores in the bin or above, hence
//     exact scores above its own;
//   - only the rows in between (the band, 32 + 2 M units wide: some tens of rows) are scored exactly and
//     ranked among themselves, by (score, position).
// Winners are marked in a bitmap over the positions, from which they are written in ascending order.
//
// Where the groups leave CUs idle, two or four workgroups share one: each scores all rows and selects for a part of the
// heads.
//
// What bounds it: one workgroup per CU (the tables and 108 registers a thread), its phases one after the other.
// At 16384 tokens, K 491: table and first rows 1.7 us (5 with all CUs asking at once), scores and histogram 12.3
// (LDS: 16 gathers and four atomics a row), bin 0.8, winners and band 4.6, exact band 3.1, ranks 1.4, output 1.2.
// The exact route, which served these contexts before, scores every row once per head (four times the LDS reads)
// and needs a workgroup per head: 64 sequences of 16384 tokens, 32 heads: 187 us, and 34 us for the tables before
// it, against 99 us for tables and selection in one launch (build_lut.hip); one sequence of 4096 tokens, 4 heads:
// 21 us in two launches against 18.5 in one.
// Counting only rows above a floor taken from a sample, to save atomics, was slower (15.8 us for scores and
// histogram): the branches cost more than the atomics.
//
// Many equal scores overflow the band's list, and such heads are redone, by the exact route between the bounds that the bin
// gives, one after the other in their workgroup.  32 heads, M = 16, tables and selection, the exact route of earlier -> this:
// all rows equal, one sequence of 8228 tokens 45 -> 45 us (186 with all four heads of a group in one workgroup), 16
// sequences of 16384 132 -> 173, 64 of them 508 -> 363; 50 different rows 30 -> 31, 78 -> 104, 277 -> 170; 8 different
// rows 58 -> 55, 66 -> 147, 238 -> 302.
#pragma once
#include <algorithm>
#include <cmath>
#include "common.hpp"
#include "coarse_score.hpp"
#include "exact_select.hpp"
#include "band_select.hpp"

namespace a2ats {

// `old` with lane `lane` (a constant) replaced by the wave-uniform `value`.
__device__ uint32_t write_lane(uint32_t value, uint32_t lane, uint32_t old) __asm("llvm.amdgcn.writelane.i32");

constexpr int kGroupThreads = 1024;
constexpr int kGroupWaves = kGroupThreads / 64;
constexpr int kGroupRows = 16;                               // rows per thread
constexpr int kGroupMaxCand = kGroupThreads * kGroupRows;    // candidates of a sequence, at most
struct GroupLds {
  uint32_t hist[2][kHistBins];   // two heads per word, 16-bit counts (at most 16384 rows)
  uint64_t won[kHeadsPerGroup][kGroupMaxCand / 64];
  uint64_t band[kHeadsPerGroup][kBandCap];
  uint32_t n_band[kHeadsPerGroup];
  uint32_t n_sure[kHeadsPerGroup];
  uint32_t from[kHeadsPerGroup];   // where the band begins
  int32_t bin[kHeadsPerGroup];
  uint32_t wave_tot[kGroupWaves];
};
// Behind the coarse table; a head whose band overflows is redone by the exact route in the same memory.
constexpr size_t kGroupWorkBytes = sizeof(GroupLds) > sizeof(ExactLds) ? sizeof(GroupLds) : sizeof(ExactLds);
constexpr size_t kGroupLdsBytes = kCoarseLdsBytes + (kGroupWorkBytes + 15) / 16 * 16;
static_assert(kExactLdsBytes <= kCoarseLdsBytes, "the exact table of a redone head takes the coarse table's place");

// Workgroups that share a group where CUs would be idle otherwise, a part of its heads each: all score the rows, but what
// follows is done for fewer heads, above all where a head has to be redone.
inline int group_split(long groups, int heads, long others) {   // heads: of a full group; others: workgroups of the launch
  int split = 1;
  while (split < 4 && 2 * split <= heads && groups * split * 2 + others <= 256) split *= 2;
  return split;
}
// The heads (a bit each) of part `part`; n_real: how many the group has.
__device__ __forceinline__ uint32_t group_part(int part, int split, int heads, int n_real) {
  const int per = (heads + split - 1) / split;
  return ((1u << per) - 1u) << (part * per) & ((1u << n_real) - 1u);
}

// Whether a workgroup's bands are expected to be many rows (band_winners), which is a kernel of its own.  A band is as wide for all K, so
// its rows go with the density of scores at the K-th, K sqrt(2 ln(candidates / K)) for scores that are about normal; 36 units of M = 16
// never have as many.  Tables and selection, one form -> the other, M = 32, 47 sequences of 8 groups of four heads, K 3 %: 2654 tokens 72.6 -> 75.9 us, 6500
// 91.2 -> 94.2, 8228 98.7 -> 97.9, 16384 135 -> 124; K 10 %: 2654 81.0 -> 83.6, 4436 95.0 -> 90.6; 20 sequences of 8 groups of four and
// three, K 3 %: 6500 38.8 -> 40.5, 8228 42.2 -> 42.3, 12000 50.6 -> 47.2.
inline bool group_many(int n_sub, long ncand, int top_k, int heads) {   // heads: of a workgroup
  return n_sub == 32 && top_k > 0 && heads * top_k * std::sqrt(2.0 * std::log(std::max(2.0, (double)ncand / top_k))) > 2440.0;
}

// Called by all kGroupThreads threads of a workgroup for the heads `mine` of its group.  dyn_lds: kGroupLdsBytes.  TABLE_IN_LDS: the caller has
// put the group's coarse table at its start (a barrier follows here), otherwise it is copied from `lut`.
template <int M, bool TABLE_IN_LDS, bool MANY>
__device__ __forceinline__ void group_select_body(
    int b, int kv, int g4, int prob, uint32_t mine, const uint8_t* __restrict__ codes, const CodePages& pg,
    const int32_t* __restrict__ lut, const float* __restrict__ lut_scale, const int32_t* __restrict__ seq_lens,
    int32_t* __restrict__ topk_idx, int32_t* __restrict__ topk_count, float* __restrict__ topk_score, int B, int Hq,
    int Hkv, int ctx_len, int64_t ctx_stride, int top_k, int window, int n_sink, unsigned char* dyn_lds) {
  constexpr int NT = kGroupThreads;
  constexpr int U = M == 16 ? 4 : 1;   // rows a thread requests together
  unsigned char* tbl = dyn_lds;
  GroupLds& L = lds_at<GroupLds>(kCoarseLdsBytes);
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int G = Hq / Hkv, head0 = b * Hq + kv * G + g4 * kHeadsPerGroup;
  const SeqRange sr = seq_range(ctx_len, seq_lens, b, window, n_sink, top_k);
  const SeqCodes seq_codes = seq_codes_of<M>(codes, pg, b, kv, Hkv, ctx_stride);
  const LutLayout lay = lut_layout(B, Hq, Hkv, M);

  if (tid < kHeadsPerGroup && ((mine >> tid) & 1u)) topk_count[head0 + tid] = sr.kk;
  for (int r = 0; r < kHeadsPerGroup; ++r)
    if ((mine >> r) & 1u)
      for (int t = sr.kk + tid; t < top_k; t += NT) {
        topk_idx[(size_t)(head0 + r) * top_k + t] = -1;
        if (topk_score) topk_score[(size_t)(head0 + r) * top_k + t] = 0.f;
      }
  if (sr.kk == 0 || mine == 0) return;   // (uniform)

  // Wave w owns chunks w n_i .. w n_i + n_i - 1 of 64 consecutive rows, so the chunks of a wave, and the waves,
  // follow each other in position.
  const int lo = sr.sink_end, hi = sr.win_start;
  const int n_i = (sr.ncand + NT - 1) / NT;   // 1 .. kGroupRows
  const int row0 = lo + wv * n_i * 64 + lane;
  LaneSwizzle<M> sw;
  sw.init(lane);
  auto load_rows = [&](int i0, uint4 (&dst)[U][M / 16]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint8_t* row = row_ptr<M>(seq_codes, min(row0 + (i0 + u) * 64, hi - 1));
#pragma unroll
      for (int qd = 0; qd < M / 16; ++qd) dst[u][qd] = *(const uint4*)(row + ((uint32_t)(qd * 16) ^ sw.row_swz));
    }
  };
  uint4 rows[2][U][M / 16];
  load_rows(0, rows[0]);   // (before the table, so that the latencies overlap)
  if (!TABLE_IN_LDS) load_coarse_table<M, NT>(lut, lay, prob, tbl);
  for (int i = tid; i < 2 * kHistBins; i += NT) (&L.hist[0][0])[i] = 0;
  if (tid < kHeadsPerGroup) {
    L.n_band[tid] = 0;
    L.n_sure[tid] = 0;
  }
  __syncthreads();

  // --- coarse scores of every row, and their histogram
  uint32_t a01[kGroupRows], a23[kGroupRows];
  const bool take_all = sr.kk >= sr.ncand;   // (uniform)
#pragma unroll
  for (int q = 0; q < kGroupRows / U; ++q) {
    const int i0 = q * U;
    if (i0 < n_i) {   // (uniform, as the conditions below)
      if (i0 + U < n_i) load_rows(i0 + U, rows[(q + 1) & 1]);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (i0 + u >= n_i) continue;   // (a chunk past the wave's last is another wave's)
        score_coarse<M>(rows[q & 1][u], sw, a01[i0 + u], a23[i0 + u]);
        if (!take_all && row0 + (i0 + u) * 64 < hi) {
          const uint32_t w01 = a01[i0 + u], w23 = a23[i0 + u];
          if (mine & 1u) atomicAdd(&L.hist[0][(w01 & 0xffffu) >> 5], 1u);
          if (mine & 2u) atomicAdd(&L.hist[0][w01 >> 21], 1u << 16);
          if (mine & 4u) atomicAdd(&L.hist[1][(w23 & 0xffffu) >> 5], 1u);
          if (mine & 8u) atomicAdd(&L.hist[1][w23 >> 21], 1u << 16);
        }
        if ((u & 1) || M == 32) __builtin_amdgcn_sched_barrier(0);   // 32 gathers at a time: bounds live registers
      }
    }
  }
  __syncthreads();
  if (wv < kHeadsPerGroup && ((mine >> wv) & 1u) && !take_all) {
    const int bin = wave_find_bin(L.hist[wv >> 1], 16 * (wv & 1), (uint32_t)sr.kk, lane);
    if (lane == 0) L.bin[wv] = bin;
  }
  __syncthreads();

  // --- winners and band rows.  Lane r 16 + i collects the winners of head r in chunk i.
  // (No coarse score is above 65520: 0xffff keeps the slots of the other heads empty.)
  uint32_t t_lo[kHeadsPerGroup], t_hi[kHeadsPerGroup];
  int kth_bin[kHeadsPerGroup];
#pragma unroll
  for (int r = 0; r < kHeadsPerGroup; ++r) {
    const bool is_mine = (mine >> r) & 1u;
    const int bin = take_all ? 0 : __builtin_amdgcn_readfirstlane(L.bin[r]);   // (of another head: not looked at)
    kth_bin[r] = bin;
    if (is_mine && tid == r) L.from[r] = take_all ? 0u : (uint32_t)max(0, (bin << 5) - M + 1);
    t_lo[r] = !is_mine ? 0xffffu : (take_all ? 0u : (uint32_t)max(0, (bin << 5) - M + 1));
    t_hi[r] = !is_mine ? 0xffffu : (take_all ? 0u : (uint32_t)min(0xffff, (bin << 5) + 32 + M));
  }
  // The low half of a word is compared as 16 bits, the high half as the whole word against the threshold
  // shifted up: no extraction.
  auto reaches = [](uint32_t word, int half, uint32_t t) {
    return __builtin_amdgcn_ballot_w64(half ? word >= (t << 16) : (uint16_t)word >= (uint16_t)t);
  };
  {
    // (two compares, two scalar ands and four lane writes per head and chunk, no branch: a branch on "any
    // band row here" costs a dependent scalar chain each, 7.1 us instead of 4.6 for 16384 rows)
    uint32_t s_lo = 0, s_hi = 0, b_lo = 0, b_hi = 0;
#pragma unroll
    for (int i = 0; i < kGroupRows; ++i) {
      if (i < n_i) {
        const uint64_t valid = __builtin_amdgcn_ballot_w64(row0 + i * 64 < hi);
#pragma unroll
        for (int r = 0; r < kHeadsPerGroup; ++r) {
          const uint64_t sure = reaches(r < 2 ? a01[i] : a23[i], r & 1, t_hi[r]) & valid;
          const uint64_t some = reaches(r < 2 ? a01[i] : a23[i], r & 1, t_lo[r]) & valid;
          s_lo = write_lane((uint32_t)sure, r * kGroupRows + i, s_lo);
          s_hi = write_lane((uint32_t)(sure >> 32), r * kGroupRows + i, s_hi);
          b_lo = write_lane((uint32_t)some, r * kGroupRows + i, b_lo);
          b_hi = write_lane((uint32_t)(some >> 32), r * kGroupRows + i, b_hi);
        }
      }
    }
    const int r = lane / kGroupRows, i = lane % kGroupRows;
    const uint64_t sure = ((uint64_t)s_hi << 32) | s_lo;
    uint64_t band = (((uint64_t)b_hi << 32) | b_lo) & ~sure;
    if (i < n_i) {   // (lanes of chunks past the wave's last hold zeros)
      L.won[r][wv * n_i + i] = sure;
      if (sure) atomicAdd(&L.n_sure[r], (uint32_t)__popcll(sure));
    }
    if (band) {
      uint32_t slot = atomicAdd(&L.n_band[r], (uint32_t)__popcll(band));
      const uint32_t j0 = (uint32_t)(lo + (wv * n_i + i) * 64 - 1);
      for (; band && slot < (uint32_t)kBandCap; ++slot, band &= band - 1)
        L.band[r][slot] = j0 + (uint32_t)__ffsll((unsigned long long)band);
    }
  }
  __syncthreads();

  // --- the band, and the winners in ascending position
  const Band band = {&L.band[0][0], &L.won[0][0], kGroupMaxCand / 64, L.n_band, L.n_sure, L.from, 32u + 2 * M,
                     (int32_t*)tbl, L.hist, L.wave_tot};
  const uint32_t redo = band_winners<M, MANY>(band, mine, head0, seq_codes, lo, sr.kk, lut, lay, [](uint32_t) {});
  write_winners<kGroupMaxCand / 64 / 256>(band, mine & ~redo, head0, lo, sr.ncand, sr.kk, top_k, topk_idx);
  // --- heads with more band rows than the list holds (many equal scores): the exact route.  The K-th coarse score is in the
  // bin, hence the K-th score is at least the bin's lower edge, and its own row's is below the upper edge.
#pragma unroll 1
  for (int r = 0; r < kHeadsPerGroup; ++r)
    if ((redo >> r) & 1u) {
      const size_t bh = (size_t)(head0 + r);
      const int32_t* meta = lut + lay.off_meta + bh * 4;
      const uint32_t bin = (uint32_t)(r == 0 ? kth_bin[0] : (r == 1 ? kth_bin[1] : (r == 2 ? kth_bin[2] : kth_bin[3])));
      const int32_t base = meta[0], shift = meta[1];
      SeqCodes rows = seq_codes;
      SeqRange range = sr;
      // (else the addresses of all rows are formed before the loop, and spilled)
      asm volatile("" : "+s"(rows.base), "+s"(range.sink_end));
      exact_select_block<M, true>(rows, lut + lay.off_exact + bh * (kCentroids * M),
                                  (int32_t)((uint32_t)base + ((bin << 5) << shift)),
                                  (int32_t)((uint32_t)base + (((bin << 5) + 32u + 2u * M) << shift)), 0.f, range,
                                  topk_idx + bh * top_k, nullptr, tbl, *(ExactLds*)(dyn_lds + kCoarseLdsBytes));
    }
  if (topk_score) {
    __syncthreads();
    write_winner_scores<M>(mine, head0, seq_codes, sr.kk, top_k, lut, lay, lut_scale, topk_idx, topk_score);
  }
}

}  // namespace a2ats
