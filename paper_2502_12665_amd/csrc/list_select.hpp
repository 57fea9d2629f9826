// The top-K of the (up to) four query heads of a group by one workgroup, for contexts whose scores do not fit its registers:
// the list route of a2ats_score_topk, taken where the groups fill the CUs (list_route).
//
// A sample gives every head a threshold below its K-th coarse score (coarse_score.hpp); one pass over the rows
// scores each against the four heads' coarse table, and a row that reaches a head's threshold goes to that head's list in
// LDS, as its coarse score and position (16 bits each).  A histogram over a list gives the 4-wide bin of the head's K-th
// coarse score, and from there on it is the group route's (group_select.hpp): rows M units above the bin are winners, rows
// M units below it are not, the few between are scored exactly and ranked, and winners are written from a bitmap over the
// positions in ascending order.  The lists hold every row that the bin and the band can need, as long as the band begins
// above the threshold; a head where it does not, or whose list overflows twice, is done by the exact route.
//
// Many equal scores.  A band of more than 1024 rows is ranked from the head's list by a radix select over (score, position); a list
// that overflows tells a higher threshold and is made again by another pass.  A head that overflows that too is done by the exact
// route, one after the other in their workgroup.  Tables and selection, us, by the streaming route of before (whose
// final kernel ranked up to 8192 rows, a workgroup a head) -> with the exact route for all of these -> now, 32 query and 8 KV heads, K 3 %:
// 16 sequences of 32768, M = 16, 1100 equal scores about the K-th of one head in four 67 -> 287 -> 73, 4000 87 -> 256 -> 94, rows of 100 kinds
// 82 -> 144 -> 106, of 20 75 -> 491 -> 112; 32 of 60000 147 -> 509 -> 111, 180 -> 666 -> 409 (8 of 1024 heads by the exact route),
// 194 -> 751 -> 138, 172 -> 872 -> 662 (52 of them); 32 of 32768, M = 32 165 -> 435 -> 126, 206 -> 404 -> 166, 194 -> 451 -> 163, 185 -> 730 -> 186.
//
// Against the streaming route this saves the survivors' way through memory (20 or 36 bytes written and read back by every head),
// the exact scores of 1.4 K rows a head, and the rounds of one workgroup per head: 256 groups of 65536 tokens, M = 32, K 2048
// 192 -> 143 us, tables included, 256 of 32768, M = 16, K 1000 97 -> 67.
// What bounds it (us of those two): tables 16 and 10, sample 13 and 6, the pass 81 and 31 (M = 16: the code matrix at 4.5 TB/s;
// M = 32: LDS reads and the vector ALU, two groups read the same rows), bin 3, winners and band rows 4 and 2, band 16 and 6,
// output 3 and 1.5: phases of one workgroup per CU one after the other.  With eight table reads requested ahead of their sums in
// the pass (score_coarse): of these 143 -> 139 us, 160 groups of 60000, M = 16, K 1500 82.1 -> 79.7.
#pragma once
#include "common.hpp"
#include "coarse_score.hpp"
#include "exact_select.hpp"
#include "band_select.hpp"
#include "group_select.hpp"

namespace a2ats {

constexpr int kListThreads = 1024;
constexpr int kListWaves = kListThreads / 64;
constexpr int kListMaxCand = 65536;   // positions are 16 bits, from the first candidate
constexpr int kListCap = 5632;        // list entries per head
constexpr int kListBin = 2;           // a bin of their histogram is 1 << kListBin coarse units, from the threshold up;
constexpr int kListWide = 5;          // 1 << kListWide, which is the whole range, where the K-th is above those
struct ListLds {
  union {
    uint32_t entry[kHeadsPerGroup][kListCap];   // coarse score in the upper half, position in the lower
    uint32_t sample[2][kHistBins];   // before the pass
    struct {                         // after it
      int32_t table[16384];
      uint32_t hist[2][kHistBins];
    } band;
    ExactLds exact;
  };
  int32_t thr[kHeadsPerGroup];
  uint32_t n[kHeadsPerGroup];
  int32_t bin[kHeadsPerGroup];
  uint32_t n_band[kHeadsPerGroup];
  uint32_t n_sure[kHeadsPerGroup];
  uint32_t from[kHeadsPerGroup], to[kHeadsPerGroup];   // where the band begins, and the first score above it
  uint32_t wave_tot[kListWaves];
};
// In the coarse table's place after the pass.
struct ListEnd {
  uint64_t won[kHeadsPerGroup][kListMaxCand / 64];
  union {
    uint64_t band[kHeadsPerGroup][kBandCap];
    uint32_t hist[2][kHistBins];   // two heads per word, 16-bit counts
  };
};
constexpr size_t kListLdsBytes = kCoarseLdsBytes + (sizeof(ListLds) + 15) / 16 * 16;
static_assert(sizeof(ListEnd) <= kCoarseLdsBytes && kExactLdsBytes <= kCoarseLdsBytes && kListCap < 65536, "");

// Head r's list overflowed: a higher threshold from the entries that are there, which are the first rows of every wave's run.  Those
// of a step of up to 256 rows that no longer fit are missing, so the last 256 are not looked at.
__device__ __forceinline__ void raise_threshold(int r, uint32_t kk, ListLds& L, int lane, int wv) {
  constexpr int NT = kListThreads, kUsed = kListCap - 256, PER = (kUsed + NT - 1) / NT;
  const int tid = threadIdx.x;
  uint32_t e[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) e[k] = L.entry[r][min(tid + k * NT, kUsed - 1)];
  const uint32_t from = (uint32_t)L.thr[r];
  __syncthreads();
  uint32_t* hist = L.entry[r];
  for (int i = tid; i < kHistBins; i += NT) hist[i] = 0;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < PER; ++k) count_shared_bins(hist, min(((e[k] >> 16) - from) >> 5, (uint32_t)kHistBins - 1), tid + k * NT < kUsed);
  __syncthreads();
  if (wv == 0) {
    const float r0 = (float)kk * (float)kUsed / (float)L.n[r];   // (as sample_threshold_body)
    const float x = 0.5f * (kSigma + sqrtf(kSigma * kSigma + 4.f * r0));
    const int bin = wave_find_bin(hist, 0, (uint32_t)ceilf(x * x) + 1, lane, ~0u);
    if (lane == 0) {
      if (bin >= 0) L.thr[r] += max(0, (bin << 5) - 32);
      L.n[r] = 0;
    }
  }
  __syncthreads();
}

// Marks the winners of head r among the rows of its list in a band that does not hold them all, by a radix select over (score,
// position).  The head's list is in registers then, and the table of 16 subspaces at a time in its place; the head's part
// of the band holds the counts.
template <int M>
__device__ __forceinline__ void crowded_band(int r, ListLds& L, ListEnd& E, const SeqCodes& seq_codes, int lo, int kk,
                                             const int32_t* __restrict__ head_table, const int32_t* __restrict__ meta) {
  constexpr int NT = kListThreads, PER = (kListCap + NT - 1) / NT, kPosBits = 16;
  static_assert(kCentroids * 16 + 2 <= kListCap && kListMaxCand <= 1 << kPosBits && sizeof(E.band[0]) >= kHistBins * 4, "");
  const int tid = threadIdx.x;
  const uint32_t n = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.n[r]);
  const uint32_t from = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.from[r]);
  const uint32_t to = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.to[r]);
  uint32_t e[PER];
  int32_t s[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    if (k * NT >= (int)n) continue;   // (uniform, as below)
    const uint32_t i = tid + k * NT;
    e[k] = i < n ? L.entry[r][i] : 0xffffffffu;   // (no coarse score is as high)
    if (e[k] >> 16 < from || e[k] >> 16 >= to) e[k] = 0xffffffffu;
    s[k] = 0;
  }
  int32_t* table = (int32_t*)L.entry[r];
#pragma unroll 1
  for (int qd = 0; qd < M / 16; ++qd) {
    uint4 w[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k)
      if (k * NT < (int)n) w[k] = *(const uint4*)(row_ptr<M>(seq_codes, lo + (e[k] == 0xffffffffu ? 0 : (int)(e[k] & 0xffffu))) + qd * 16);
    __syncthreads();
    for (int i = tid; i < kCentroids * 4; i += NT) {
      const int c = i / 4;   // (four entries are turned by their centroid, see band_select.hpp)
      ((uint4*)table)[c * 4 + ((i + c) & 3)] = ((const uint4*)head_table)[c * (M / 4) + qd * 4 + (i & 3)];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      if (k * NT >= (int)n) continue;
      const uint32_t d[4] = {w[k].x, w[k].y, w[k].z, w[k].w};
#pragma unroll
      for (int t = 0; t < 16; ++t) {
        const uint32_t c = (d[t >> 2] >> (8 * (t & 3))) & 0xffu;
        s[k] += table[c * 16 + ((((t >> 2) + c) & 3) << 2) + (t & 3)];
      }
    }
  }
  const uint32_t key0 = score_key((int32_t)((uint32_t)meta[0] + (from << meta[1])));
  const uint32_t range = (to - from + M) << meta[1];   // (a coarse score leaves out less than M units)
  auto row_of = [&](int k) {
    const uint32_t key = score_key(s[k]);
    return (uint64_t)(key > key0 ? min(key - key0, range) : 0u) << kPosBits | (0xffffu - (e[k] & 0xffffu));
  };
  const uint64_t last = reached_by<NT, false>(
      (uint32_t)kk - L.n_sure[r], kPosBits + 32 - (int)__clz(range),
      [&](auto f) {
#pragma unroll
        for (int k = 0; k < PER; ++k)
          if (k * NT < (int)n) f(e[k] != 0xffffffffu, row_of(k));
      },
      (uint32_t*)E.band[r], L.wave_tot, (uint32_t*)table + kCentroids * 16);
#pragma unroll
  for (int k = 0; k < PER; ++k)
    if (k * NT < (int)n && e[k] != 0xffffffffu && row_of(k) >= last)
      atomicOr((uint32_t*)&E.won[r][0] + ((e[k] & 0xffffu) >> 5), 1u << (e[k] & 31));
}

// Called by all kListThreads threads of a workgroup.  dyn_lds: kListLdsBytes; TABLE_IN_LDS: the caller has put the group's
// coarse table at its start (a barrier follows here), otherwise it is copied from `lut`.  stats (may be null): per head, the
// length of its list, and the route in the upper four bits (as a2ats_score_topk_stats reports them).
template <int M, bool TABLE_IN_LDS>
__device__ __forceinline__ void list_select_body(
    int b, int kv, int g4, int prob, const uint8_t* __restrict__ codes, const CodePages& pg,
    const int32_t* __restrict__ lut, const float* __restrict__ lut_scale, const int32_t* __restrict__ seq_lens,
    int32_t* __restrict__ topk_idx, int32_t* __restrict__ topk_count, float* __restrict__ topk_score,
    uint32_t* __restrict__ stats, int sample_rows, int B, int Hq, int Hkv, int NG, int ctx_len, int64_t ctx_stride, int top_k,
    int window, int n_sink, unsigned char* dyn_lds) {
  constexpr int NT = kListThreads;
  constexpr int U = M == 16 ? 4 : 2, STEP = 64 * U;   // rows a lane requests together; rows of a wave's step
  unsigned char* tbl = dyn_lds;
  ListLds& L = lds_at<ListLds>(kCoarseLdsBytes);
  ListEnd& E = *(ListEnd*)dyn_lds;
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int G = Hq / Hkv, head0 = b * Hq + kv * G + g4 * kHeadsPerGroup;
  const int n_real = min(kHeadsPerGroup, G - g4 * kHeadsPerGroup);
  const uint32_t real = (1u << n_real) - 1u;
  const SeqRange sr = seq_range(ctx_len, seq_lens, b, window, n_sink, top_k);
  const SeqCodes seq_codes = seq_codes_of<M>(codes, pg, b, kv, Hkv, ctx_stride);
  const LutLayout lay = lut_layout(B, Hq, Hkv, M);
  const int lo = sr.sink_end, hi = sr.win_start;

  if (tid < n_real) topk_count[head0 + tid] = sr.kk;
  for (int r = 0; r < n_real; ++r)
    for (int t = sr.kk + tid; t < top_k; t += NT) {
      topk_idx[(size_t)(head0 + r) * top_k + t] = -1;
      if (topk_score) topk_score[(size_t)(head0 + r) * top_k + t] = 0.f;
    }
  if (stats && tid < n_real) stats[head0 + tid] = 0u;
  if (sr.kk == 0) return;   // (uniform)

  // --- thresholds from a sample
  if (tid < kHeadsPerGroup) {
    L.thr[tid] = 0;
    L.n[tid] = 0;
    L.n_band[tid] = 0;
    L.n_sure[tid] = 0;
  }
  if (!TABLE_IN_LDS) load_coarse_table<M, NT>(lut, lay, prob, tbl);
  sample_threshold_body<M, NT, true>(
      prob, 0, codes, pg, lut, seq_lens, [&](int r, int32_t t) { L.thr[r] = max(t, 0); }, B, Hq, Hkv, NG, 1, sample_rows,
      ctx_len, ctx_stride, top_k, window, n_sink, tbl, L.sample);
  __syncthreads();
  uint32_t T[kHeadsPerGroup];
#pragma unroll
  for (int r = 0; r < kHeadsPerGroup; ++r)   // (no coarse score is above 65520: a head that there is not takes no row)
    T[r] = r < n_real ? (uint32_t)__builtin_amdgcn_readfirstlane(L.thr[r]) : 0xffffu;

  // --- one pass over the rows, a run of them for each wave; and another one for lists that overflow
  auto pass = [&](const uint32_t (&T)[kHeadsPerGroup], int lane, SeqCodes seq_codes, int lo, int hi) {
    const int run = (sr.ncand + 64 * kListWaves - 1) / (64 * kListWaves) * 64;
    const int wbegin = lo + wv * run, wend = min(hi, wbegin + run);
    LaneSwizzle<M> sw;
    sw.init(lane);
    uint4 rows_a[U][M / 16], rows_b[U][M / 16];
    // (of codes in pages, the page numbers of a step are requested a step ahead of its rows)
    const bool paged = seq_codes.pages != nullptr;
    int32_t page[U];
    auto load_pages = [&](int base) {
      if (paged)
#pragma unroll
        for (int u = 0; u < U; ++u) page[u] = seq_codes.pages[(uint32_t)min(base + u * 64 + lane, wend - 1) >> seq_codes.shift];
    };
    auto load_rows = [&](int base, uint4 (&dst)[U][M / 16]) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int j = min(base + u * 64 + lane, wend - 1);
        const uint8_t* row = paged ? row_in_page<M>(seq_codes, page[u], j) : seq_codes.base + (size_t)j * M;
#pragma unroll
        for (int qd = 0; qd < M / 16; ++qd) dst[u][qd] = *(const uint4*)(row + ((uint32_t)(qd * 16) ^ sw.row_swz));
      }
      load_pages(base + STEP);
    };
    auto process = [&](int base, const uint4 (&rows)[U][M / 16]) {
      uint32_t a01[U], a23[U];
      uint64_t hit[U][kHeadsPerGroup];
      uint32_t c[kHeadsPerGroup] = {0, 0, 0, 0};
#pragma unroll
      for (int u = 0; u < U; ++u) {
        score_coarse<M, true>(rows[u], sw, a01[u], a23[u]);
        const uint64_t valid = __builtin_amdgcn_ballot_w64(base + u * 64 + lane < wend);
        // The low half of a word is compared as 16 bits, the high half as the whole word against the threshold shifted up.
        hit[u][0] = __builtin_amdgcn_ballot_w64((uint16_t)a01[u] >= (uint16_t)T[0]) & valid;
        hit[u][1] = __builtin_amdgcn_ballot_w64(a01[u] >= (T[1] << 16)) & valid;
        hit[u][2] = __builtin_amdgcn_ballot_w64((uint16_t)a23[u] >= (uint16_t)T[2]) & valid;
        hit[u][3] = __builtin_amdgcn_ballot_w64(a23[u] >= (T[3] << 16)) & valid;
#pragma unroll
        for (int r = 0; r < kHeadsPerGroup; ++r) c[r] += (uint32_t)__popcll(hit[u][r]);
        if ((u & 1) || M == 32) __builtin_amdgcn_sched_barrier(0);   // 32 reads at a time: bounds live registers
      }
      if ((c[0] | c[1] | c[2] | c[3]) == 0u) return;
      // Places in the four lists for the step's rows by one LDS atomic.
      uint32_t at = 0;
#pragma unroll
      for (int r = 0; r < kHeadsPerGroup; ++r) at = write_lane(c[r], r, at);
      if (lane < kHeadsPerGroup) at = atomicAdd(&L.n[lane], at);
      const uint32_t pos = (uint32_t)(base - lo + lane);
#pragma unroll
      for (int r = 0; r < kHeadsPerGroup; ++r) {
        uint32_t slot0 = (uint32_t)__builtin_amdgcn_readlane((int)at, r);
        if (slot0 + c[r] > (uint32_t)kListCap) continue;   // (uniform; the count shows that the list lacks rows)
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const uint64_t h = hit[u][r];
          if (__builtin_amdgcn_inverse_ballot_w64(h)) {
            const uint32_t slot = (uint32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(h >> 32),
                                                                      __builtin_amdgcn_mbcnt_lo((uint32_t)h, slot0));
            const uint32_t a = r < 2 ? a01[u] : a23[u];
            L.entry[r][slot] = ((r & 1) ? a & 0xffff0000u : a << 16) | (pos + u * 64);
          }
          slot0 += (uint32_t)__popcll(h);
        }
      }
    };
    if (wbegin < wend) {
      load_pages(wbegin);
      load_rows(wbegin, rows_a);
#pragma unroll 1
      for (int base = wbegin; base < wend; base += 2 * STEP) {
        load_rows(base + STEP, rows_b);
        process(base, rows_a);
        load_rows(base + 2 * STEP, rows_a);
        process(base + STEP, rows_b);
      }
    }
    __syncthreads();
  };
  pass(T, lane, seq_codes, lo, hi);
  uint32_t over = 0;
#pragma unroll
  for (int r = 0; r < kHeadsPerGroup; ++r)
    over |= (uint32_t)__builtin_amdgcn_readfirstlane((int)L.n[r]) > (uint32_t)kListCap ? 1u << r : 0u;
  if (__builtin_expect(over != 0u, 0)) {   // (uniform)
#pragma unroll 1
    for (int r = 0; r < kHeadsPerGroup; ++r)
      if ((over >> r) & 1u) raise_threshold(r, (uint32_t)sr.kk, L, lane, wv);
    uint32_t higher[kHeadsPerGroup];   // (not in T: the first pass is slower if that changes later)
#pragma unroll
    for (int r = 0; r < kHeadsPerGroup; ++r)
      higher[r] = (over >> r) & 1u ? (uint32_t)__builtin_amdgcn_readfirstlane(L.thr[r]) : 0xffffu;
    // (else what the second pass needs is kept through the first, M = 32 1 us of 140)
    int lane2 = (int)threadIdx.x & 63, lo2 = lo, hi2 = hi;
    SeqCodes codes2 = seq_codes;
    asm volatile("" : "+v"(lane2), "+s"(lo2), "+s"(hi2), "+s"(codes2.base));
    pass(higher, lane2, codes2, lo2, hi2);
  }

  // --- the bin of the K-th coarse score; of a head where it is above all of them, again with wide bins
  const HeadShare own = head_share(real);
  const int mr = own.head, mt = own.at;
  const bool take_all = sr.kk >= sr.ncand;   // (uniform; then the thresholds are zero)
  uint32_t n_list, t_mr, wide = 0;           // wide: heads with wide bins
  int32_t bin_of[kHeadsPerGroup];
  auto bin_log = [&](int r) { return (wide >> r) & 1u ? kListWide : kListBin; };
  auto find_bins = [&]() {
    for (int i = tid; i < (int)(sizeof(ListEnd) / 16); i += NT) ((uint4*)&E)[i] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    n_list = (uint32_t)__builtin_amdgcn_readfirstlane((int)min(L.n[mr], (uint32_t)kListCap));
    t_mr = (uint32_t)__builtin_amdgcn_readfirstlane(L.thr[mr]);
    const int log = bin_log(mr);
    if (!take_all)
      for (uint32_t i = mt; i < n_list; i += own.threads)   // (the last bin holds all that is further up)
        atomicAdd(&E.hist[mr >> 1][min(((L.entry[mr][i] >> 16) - t_mr) >> log, (uint32_t)kHistBins - 1)], 1u << (16 * (mr & 1)));
    __syncthreads();
    if (wv < kHeadsPerGroup) {
      const int bin = take_all ? 0 : wave_find_bin(E.hist[wv >> 1], 16 * (wv & 1), (uint32_t)sr.kk, lane);
      if (lane == 0) L.bin[wv] = bin;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kHeadsPerGroup; ++r) bin_of[r] = __builtin_amdgcn_readfirstlane(L.bin[r]);
  };
  find_bins();
#pragma unroll
  for (int r = 0; r < kHeadsPerGroup; ++r) wide |= r < n_real && bin_of[r] == kHistBins - 1 ? 1u << r : 0u;
  if (__builtin_expect(wide != 0u, 0)) find_bins();
  // A head is done again if its list overflowed, or holds less than K rows, or the band begins below the threshold.
  uint32_t redo = 0;
#pragma unroll
  for (int r = 0; r < kHeadsPerGroup; ++r) {
    const uint32_t n = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.n[r]);
    const int bin = bin_of[r];
    const uint32_t why = r >= n_real ? 0u : (n > (uint32_t)kListCap ? 2u : (bin < 0 ? 1u : ((T[r] != 0u || (over >> r) & 1u) && (bin << bin_log(r)) < M - 1 ? 4u : 0u)));
    redo |= why ? 1u << r : 0u;
    if (stats && tid == r && r < n_real) stats[head0 + r] = n | why << 28;
  }
  // --- winners and band rows (hist is the band's place from here on)
  if (!((redo >> mr) & 1u)) {
    const int bin = mr == 0 ? bin_of[0] : (mr == 1 ? bin_of[1] : (mr == 2 ? bin_of[2] : bin_of[3]));
    const int edge = (int)t_mr + (bin << bin_log(mr));
    const uint32_t t_lo = (uint32_t)max(0, edge - M + 1);
    const uint32_t t_hi = take_all ? 0u : (uint32_t)min(0xffff, edge + (1 << bin_log(mr)) + M);
    if (mt == 0) {
      L.from[mr] = t_lo;
      L.to[mr] = t_hi;
    }
    uint32_t sure = 0;
    for (uint32_t i = mt; i < n_list; i += own.threads) {
      const uint32_t e = L.entry[mr][i], s = e >> 16, j = e & 0xffffu;
      if (s >= t_hi) {
        atomicOr((uint32_t*)&E.won[mr][0] + (j >> 5), 1u << (j & 31));
        ++sure;
      } else if (s >= t_lo) {
        const uint32_t slot = atomicAdd(&L.n_band[mr], 1u);
        if (slot < (uint32_t)kBandCap) E.band[mr][slot] = (uint64_t)((uint32_t)lo + j);
      }
    }
    sure = wave_inclusive_scan(sure);
    if (lane == 63 && sure) atomicAdd(&L.n_sure[mr], sure);
  }
  __syncthreads();

  // --- the band, and the winners in ascending position
  const Band band = {&E.band[0][0], &E.won[0][0], kListMaxCand / 64, L.n_band, L.n_sure, L.from,
                     (1u << (wide ? kListWide : kListBin)) + 2 * M, L.band.table, L.band.hist, L.wave_tot};
  band_winners<M, true>(band, real & ~redo, head0, seq_codes, lo, sr.kk, lut, lay, [&](uint32_t crowded) {
#pragma unroll 1
    for (int r = 0; r < kHeadsPerGroup; ++r)   // (while the lists are there)
      if ((crowded >> r) & 1u)
        crowded_band<M>(r, L, E, seq_codes, lo, sr.kk, lut + lay.off_exact + (size_t)(head0 + r) * (kCentroids * M),
                        lut + lay.off_meta + (size_t)(head0 + r) * 4);
    __syncthreads();
  });
  write_winners<kListMaxCand / 64 / 256>(band, real & ~redo, head0, lo, sr.ncand, sr.kk, top_k, topk_idx);
#pragma unroll 1
  for (int r = 0; r < kHeadsPerGroup; ++r)
    if ((redo >> r) & 1u) {
      const size_t bh = (size_t)(head0 + r);
      const int32_t* meta = lut + lay.off_meta + bh * 4;
      SeqCodes rows = seq_codes;
      SeqRange range = sr;
      // (else the addresses of all rows are formed before the loop, and spilled)
      asm volatile("" : "+s"(rows.base), "+s"(range.sink_end));
      exact_select_block<M>(rows, lut + lay.off_exact + bh * (kCentroids * M), meta[0], meta[2], 0.f, range,
                            topk_idx + bh * top_k, nullptr, tbl, L.exact);
    }
  if (topk_score) {
    __syncthreads();
    write_winner_scores<M>(real, head0, seq_codes, sr.kk, top_k, lut, lay, lut_scale, topk_idx, topk_score);
  }
}

}  // namespace a2ats
