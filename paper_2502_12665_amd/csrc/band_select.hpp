// The end of a selection by coarse scores, for the (up to) four heads of a group by one workgroup of 1024 threads: the band (rows whose coarse score does not tell whether they are winners) is scored exactly and ranked, and
// winners are written from a bitmap over the positions.
#pragma once
#include "common.hpp"
#include "coarse_score.hpp"
#include "exact_select.hpp"

namespace a2ats {

constexpr int kBandCap = 1024;   // band rows per head
// What a selection hands over.  Everything is in LDS.
struct Band {
  uint64_t* row;           // [heads][kBandCap] positions; (exact key, position complemented) afterwards
  uint64_t* won;           // [heads][won_words]: a bit for each candidate, so far of the rows above the band
  int won_words;
  const uint32_t* n;       // [heads] rows of the band, more than kBandCap: not all are in it
  const uint32_t* n_sure;  // [heads] winners above it; fewer than K, and with the band's rows at least K
  const uint32_t* from;    // [heads] coarse score that the band begins at, `width` units wide
  uint32_t width;
  int32_t* table;          // 64 KB
  uint32_t (*hist)[kHistBins];   // two of them
  uint32_t* wave_tot;      // [waves]
};

// The sixteen waves divided among the heads in `heads` (a bit each, at least one of them): the head of this wave, how many
// threads it has, and which of them this one is.  (With four waves a head whatever the heads, one selection per KV head by the list route:
// 160 of 32768 candidates M = 16 46.4 -> 44.5 us, of 65000 68.5 -> 63.5, of 32768 M = 32 73.9 -> 70.2.)
struct HeadShare {
  int head, threads, at;
};
__device__ __forceinline__ HeadShare head_share(uint32_t heads) {
  static_assert(kExactThreads == 16 * 64 && kHeadsPerGroup == 4, "");
  // 16 waves each, 8, 6 + 5 + 5, or 4 (no division: two of them took 0.5 us; the loop below unrolled costs M = 16 1 us of 60, in registers)
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), n = __popc(heads), k = wv * n >> 4;
  auto first = [&](int i) { return n == 3 ? 5 * i + (i > 0 ? 1 : 0) : (16 >> (n >> 1)) * i; };
  const int w0 = first(k), w1 = first(k + 1);
  for (int i = 0; i < k; ++i) heads &= heads - 1;
  return {__ffs((int)heads) - 1, 64 * (w1 - w0), (int)threadIdx.x - 64 * w0};
}

// Exact score of a row from a head's table in global memory.
template <int M>
__device__ __forceinline__ int32_t exact_score_of(const int32_t* __restrict__ t, const uint8_t* __restrict__ row) {
  uint4 w[M / 16];
  int32_t s = 0;
#pragma unroll
  for (int qd = 0; qd < M / 16; ++qd) w[qd] = *(const uint4*)(row + qd * 16);
#pragma unroll
  for (int qd = 0; qd < M / 16; ++qd) {
    const uint32_t d[4] = {w[qd].x, w[qd].y, w[qd].z, w[qd].w};
#pragma unroll
    for (int t4 = 0; t4 < 16; ++t4) s += t[((d[t4 >> 2] >> (8 * (t4 & 3))) & 0xffu) * M + qd * 16 + t4];
  }
  return s;
}

// Of the distinct values, `bits` wide, that the threads of a workgroup of NT hold: one that exactly `need` of them reach.  each(f)
// calls f(in, value) for a thread's own (where `in`), the same every time; there are at least `need`.  In LDS: hist, kHistBins words;
// wave_tot, one a wave; res, two.  By radix: a level takes 11 bits, 1.5 us.
// TAIL: by counting where 64 rows are left, instead of further levels.  (Not in the list route, where it costs registers.)
template <int NT, bool TAIL, typename Each>
__device__ __forceinline__ uint64_t reached_by(uint32_t need, int bits, Each each, uint32_t* hist, uint32_t* wave_tot, uint32_t* res) {
  uint64_t prefix = 0;
#pragma unroll 1
  for (int above = bits; above > 0;) {   // (uniform)
    const int width = min(above, 11), shift = above - width;
    __syncthreads();
    for (int i = threadIdx.x; i < kHistBins; i += NT) hist[i] = 0;
    __syncthreads();
    each([&](bool in, uint64_t value) {
      count_shared_bins(hist, (uint32_t)(value >> shift) & ((1u << width) - 1u), in && value >> above == prefix >> above);
    });
    __syncthreads();
    block_find_rank_desc<NT, kHistBins>([&](int i) { return hist[i]; }, need, wave_tot, res);
    const uint32_t bin = res[0], m = hist[bin];
    need -= res[1];
    prefix |= (uint64_t)bin << shift;
    if (m == need) return prefix;
    above = shift;
    if (!TAIL || m > 64u) continue;
    // a few rows are left: by counting, in one wave
    __syncthreads();
    if (threadIdx.x == 0) wave_tot[0] = 0;
    __syncthreads();
    uint64_t* rows = (uint64_t*)hist;
    each([&](bool in, uint64_t value) {
      if (in && value >> shift == prefix >> shift) rows[atomicAdd(&wave_tot[0], 1u)] = value;
    });
    __syncthreads();
    if (threadIdx.x < m) {
      const uint64_t own = rows[threadIdx.x];
      uint32_t before = 0;
      for (uint32_t u = 0; u < m; ++u) before += rows[u] > own ? 1u : 0u;
      if (before + 1 == need) {
        res[0] = (uint32_t)own;
        res[1] = (uint32_t)(own >> 32);
      }
    }
    __syncthreads();
    return (uint64_t)res[1] << 32 | res[0];
  }
  return prefix;
}

// Marks the K - n_sure best rows of the band in `won`, of the heads in `mine` whose band is complete.  The caller has
// synchronised.  Returns the heads of `mine` whose band is not complete (uniform), for which, if there are any, crowded(heads) is
// called before anything of B but the bitmaps is written.
//
// Few rows (512 of M = 16, 256 of M = 32) read their entries from the exact tables in global memory and are ranked by counting.
// For more the tables come to LDS first, as many as fit 64 KB, which takes 2 us: an entry read from global memory is a cache
// line of its own (4 x 800 rows of M = 32: 75 us against 13).  Then the K-th is found by a histogram of 2048 bins over the
// band's range and, in its bin, by counting, 7 us for those rows instead of 41 by counting alone.  (More than 64 rows in that bin, equal
// scores: four of them at a time against a row that is read, 16 sequences of 32768 tokens whose rows are of 100 kinds 145 -> 106 us.)  MANY false: only the first
// form (the other one's code costs calls that do not use it up to 1 us).
template <int M, bool MANY, typename Crowded>
__device__ __forceinline__ uint32_t band_winners(const Band& B, uint32_t mine, int head0, const SeqCodes& seq_codes, int lo, int kk,
                                                 const int32_t* __restrict__ lut, const LutLayout& lay, Crowded crowded) {
  constexpr int NT = kExactThreads, HP = 64 / M;   // heads whose tables fit
  const int tid = threadIdx.x;
  uint32_t first[kHeadsPerGroup + 1], left = 0;
  first[0] = 0;
#pragma unroll
  for (int r = 0; r < kHeadsPerGroup; ++r) {
    const uint32_t n = (mine >> r) & 1u ? (uint32_t)__builtin_amdgcn_readfirstlane((int)B.n[r]) : 0u;
    left |= n > (uint32_t)kBandCap ? 1u << r : 0u;
    first[r + 1] = first[r] + (n > (uint32_t)kBandCap ? 0u : n);
  }
  if (__builtin_expect(left != 0u, 0)) crowded(left);
  if (first[4] == 0u) return left;
  const bool few = !MANY || first[4] * M <= 8192u;
  auto head_of = [&](uint32_t e) { return (e >= first[1] ? 1 : 0) + (e >= first[2] ? 1 : 0) + (e >= first[3] ? 1 : 0); };
  auto first_of = [&](int r) { return r == 0 ? 0u : (r == 1 ? first[1] : (r == 2 ? first[2] : first[3])); };
  auto place_of = [&](uint32_t e, int r) { return B.row + r * kBandCap + (e - first_of(r)); };
  auto win = [&](int r, uint64_t row) {
    const uint32_t bit = ~(uint32_t)row - (uint32_t)lo;
    atomicOr((uint32_t*)(B.won + (size_t)r * B.won_words) + (bit >> 5), 1u << (bit & 31));
  };
  if (few) {
    for (uint32_t e = tid; e < first[4]; e += NT) {
      const int r = head_of(e);
      uint64_t* at = place_of(e, r);
      const int32_t s = exact_score_of<M>(lut + lay.off_exact + (size_t)(head0 + r) * (kCentroids * M), row_ptr<M>(seq_codes, (int)(uint32_t)*at));
      *at = ((uint64_t)score_key(s) << 32) | ~(uint32_t)*at;   // (of equal scores the lower position is larger)
    }
    __syncthreads();
  }
#pragma unroll
  for (int p = 0; p < kHeadsPerGroup; p += HP) {
    const uint32_t e0 = first[p], e1 = first[p + HP];
    if (few || e0 == e1) continue;
    uint4 w[M / 16];
    uint64_t* at = nullptr;
    int r = p;
    auto load_row = [&](uint32_t e) {
      r = head_of(e);
      at = place_of(e, r);
      const uint8_t* row = row_ptr<M>(seq_codes, (int)(uint32_t)*at);
#pragma unroll
      for (int qd = 0; qd < M / 16; ++qd) w[qd] = *(const uint4*)(row + qd * 16);
    };
    if (e0 + tid < e1) load_row(e0 + tid);   // (the rows and the tables are requested together)
#pragma unroll
    for (int h = p; h < p + HP; ++h) {
      if (first[h] == first[h + 1]) continue;
      const uint4* src = (const uint4*)(lut + lay.off_exact + (size_t)(head0 + h) * (kCentroids * M));
      uint4* dst = (uint4*)B.table + (h - p) * (kCentroids * M / 4);
#pragma unroll
      for (int i = tid; i < kCentroids * M / 4; i += NT) {
        const int c = i / (M / 4);   // (four entries are turned by their centroid, so that a subspace's are not all in one bank)
        dst[c * (M / 4) + ((i + c) & (M / 4 - 1))] = src[i];
      }
    }
    __syncthreads();
    for (uint32_t e = e0 + tid; e < e1; e += NT) {
      if (e != e0 + tid) load_row(e);
      const int32_t* t = B.table + (r - p) * (kCentroids * M);
      int32_t s = 0;
#pragma unroll
      for (int qd = 0; qd < M / 16; ++qd) {
        const uint32_t d[4] = {w[qd].x, w[qd].y, w[qd].z, w[qd].w};
#pragma unroll
        for (int t4 = 0; t4 < 16; ++t4) {
          const uint32_t c = (d[t4 >> 2] >> (8 * (t4 & 3))) & 0xffu;
          s += t[c * M + (((qd * 4 + (t4 >> 2) + c) & (M / 4 - 1)) << 2) + (t4 & 3)];
        }
      }
      *at = ((uint64_t)score_key(s) << 32) | ~(uint32_t)*at;
    }
    __syncthreads();
  }
  // (eight lanes share a row: the lists are short and every step is an LDS round trip)
  if (few) {
    for (uint32_t e = tid >> 3; e < first[4]; e += NT / 8) {
      const int r = head_of(e);
      const uint32_t f = first_of(r), n = (r == 0 ? first[1] : (r == 1 ? first[2] : (r == 2 ? first[3] : first[4]))) - f;
      const uint64_t* row = B.row + r * kBandCap;
      const uint64_t own = row[e - f];
      int32_t before = 0;
#pragma unroll 4
      for (uint32_t u = tid & 7; u < n; u += 8) before += row[u] > own ? 1 : 0;
      before = group8_sum(before);
      if ((tid & 7) == 0 && (uint32_t)before < (uint32_t)kk - B.n_sure[r]) win(r, own);
    }
  } else {
    uint32_t there = 0;
#pragma unroll
    for (int r = 0; r < kHeadsPerGroup; ++r) there |= first[r] != first[r + 1] ? 1u << r : 0u;
    const HeadShare own_head = head_share(there);
    const int mr = own_head.head;
    const uint32_t n = (uint32_t)__builtin_amdgcn_readfirstlane((int)B.n[mr]);
    const uint64_t* row = B.row + mr * kBandCap;
    const int32_t* meta = lut + lay.off_meta + (size_t)(head0 + mr) * 4;
    const uint32_t key0 = score_key((int32_t)((uint32_t)meta[0] + (B.from[mr] << meta[1])));
    const uint32_t range = (B.width + M) << meta[1];   // (a coarse score leaves out less than M units)
    const int shift = max(0, 21 - (int)__clz(range));
    // (the keys of a finite table lie in the range; others in the bins at its ends, which keeps the order)
    auto bin_of = [&](uint32_t key) { return min(key > key0 ? (key - key0) >> shift : 0u, (uint32_t)kHistBins - 1); };
    for (int i = tid; i < kHistBins / 2; i += NT) ((uint4*)B.hist)[i] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    for (uint32_t i = own_head.at; i < n; i += own_head.threads)
      atomicAdd(&B.hist[mr >> 1][bin_of((uint32_t)(row[i] >> 32))], 1u << (16 * (mr & 1)));
    __syncthreads();
    const uint32_t need = (uint32_t)kk - B.n_sure[mr];
    const int bin = wave_find_bin(B.hist[mr >> 1], 16 * (mr & 1), need, tid & 63);
    // (of many rows in that bin, equal scores, four at a time against every row that is read: the reads are what takes the time)
    const bool crowd = bin >= 0 && (B.hist[mr >> 1][bin] >> (16 * (mr & 1)) & 0xffffu) > 64u;
    const uint32_t groups = own_head.threads >> 3;
    if (!crowd) {
      for (uint32_t i = own_head.at >> 3; i < n; i += groups) {
        const uint64_t own = row[i];
        const int b = (int)bin_of((uint32_t)(own >> 32));
        if (b < bin) continue;
        int32_t before = 0;
        if (b == bin) {
#pragma unroll 4
          for (uint32_t u = tid & 7; u < n; u += 8) before += row[u] > own ? 1 : 0;
          before = group8_sum(before);
        }
        if ((tid & 7) == 0 && (uint32_t)before < need) win(mr, own);
      }
    } else {
      constexpr int kRows = 4;
      for (uint32_t i = own_head.at >> 3; i < n; i += kRows * groups) {
        uint64_t own[kRows];
        int32_t before[kRows];
#pragma unroll
        for (int k = 0; k < kRows; ++k) {
          own[k] = row[min(i + k * groups, n - 1)];
          before[k] = 0;
        }
#pragma unroll 2
        for (uint32_t u = tid & 7; u < n; u += 8) {
          const uint64_t other = row[u];
#pragma unroll
          for (int k = 0; k < kRows; ++k) before[k] += other > own[k] ? 1 : 0;
        }
#pragma unroll
        for (int k = 0; k < kRows; ++k) {
          before[k] = group8_sum(before[k]);
          if ((tid & 7) == 0 && i + k * groups < n && (uint32_t)before[k] < need) win(mr, own[k]);
        }
      }
    }
  }
  __syncthreads();
  return left;
}

// Writes the winners of the heads in `mine` in ascending position; ncand: the bits of the bitmap, at most 16384 PER.
template <int PER>
__device__ __forceinline__ void write_winners(const Band& B, uint32_t mine, int head0, int lo, int ncand, int kk, int top_k,
                                              int32_t* __restrict__ topk_idx) {
  if (mine == 0u) return;   // (uniform)
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  // (one word a thread of the four waves of a head's number is as fast as more waves could be)
  const HeadShare own = PER > 1 ? head_share(mine) : HeadShare{wv >> 2, 256, tid & 255};
  auto words_each = [](int words, int threads) {   // their quotient, rounded up, which is 1 to PER
    int n = 1;
#pragma unroll
    for (int w = 1; w < PER; ++w) n += words > w * threads ? 1 : 0;
    return n;
  };
  const int n_words = (mine >> own.head) & 1u ? (ncand + 63) / 64 : 0, per = words_each(n_words, own.threads);
  const int w0 = own.at * per;
  const uint64_t* won = B.won + (size_t)own.head * B.won_words;
  uint64_t word[PER];
  uint32_t n = 0;
#pragma unroll
  for (int w = 0; w < PER; ++w) {
    word[w] = w < per && w0 + w < n_words ? won[w0 + w] : 0ull;
    n += (uint32_t)__popcll(word[w]);
  }
  const uint32_t inc = wave_inclusive_scan(n);
  if (lane == 63) B.wave_tot[wv] = inc;
  __syncthreads();
  uint32_t at = inc - n;
  for (int w = wv - (own.at >> 6); w < wv; ++w) at += B.wave_tot[w];
  int32_t* oi = topk_idx + (size_t)(head0 + own.head) * top_k;
#pragma unroll
  for (int w = 0; w < PER; ++w)
    while (word[w]) {
      if (at < (uint32_t)kk) oi[at] = lo + (w0 + w) * 64 + __ffsll((unsigned long long)word[w]) - 1;
      ++at;
      word[w] &= word[w] - 1;
    }
}

// Scores of the winners in topk_idx, from the exact tables in global memory.  The caller has synchronised.
template <int M>
__device__ __forceinline__ void write_winner_scores(uint32_t mine, int head0, const SeqCodes& seq_codes, int kk, int top_k,
                                                    const int32_t* __restrict__ lut, const LutLayout& lay,
                                                    const float* __restrict__ lut_scale, const int32_t* __restrict__ topk_idx,
                                                    float* __restrict__ topk_score) {
  for (int r = 0; r < kHeadsPerGroup; ++r)
    for (int i = ((mine >> r) & 1u) ? (int)threadIdx.x : kk; i < kk; i += kExactThreads) {
      const int32_t s = exact_score_of<M>(lut + lay.off_exact + (size_t)(head0 + r) * (kCentroids * M),
                                          row_ptr<M>(seq_codes, topk_idx[(size_t)(head0 + r) * top_k + i]));
      topk_score[(size_t)(head0 + r) * top_k + i] = (float)s * lut_scale[head0 + r];
    }
}

}  // namespace a2ats
