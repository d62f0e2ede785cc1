// kap_compile_plan on the GPU: Alg. 1 of the paper, SelectEvidenceUnderBudget
// through BuildBlockTable, one workgroup per sequence.
//
// Per sequence the workgroup
//   1. checks the CSR bounds, the length and the scores (status codes),
//   2. marks the mandatory prefix / suffix in an LDS bitmap,
//   3. ranks the spans by (prior desc, start asc, index asc): a few by counting
//      for every span how many precede it (1 to 8 threads a span), up to one
//      LDS chunk by buckets of the prior, more by counting chunk by chunk; the
//      inverse permutation goes to LDS (to the workspace with several chunks),
//   4. walks the spans in rank order with one wavefront, 64 at a time: each
//      lane prices its span against the bitmap (its cost in visible tokens),
//      and every round takes all spans, in order, that surely fit,
//   5. compacts the bitmap into the ascending logical-page list (staged in
//      LDS) and maps it through the full block table.
// Page mode keeps one bit per page; token mode (the visibility mask of
// Sec. 3.1 at token resolution) one bit per token, and also emits each view
// page's 16-bit mask of visible tokens.
// Selection uses integer arithmetic only (float priors are only compared), so
// the plan is bit-for-bit deterministic.
#include "kap_internal.h"

namespace kap {
namespace {

constexpr int kRankChunk = 2048;   // ranking keys staged per pass; also the LDS view list
// Spans ranked by counting all pairs; more are ranked by buckets. Up to half
// the threads two or more of them share a span's pairs (4 x 128K, 5.5%, per call:
// 96 spans 11.1 us by pairs, 11.6 by buckets; 112: 11.5, 11.7; 128: 11.6, 11.9),
// above it one counts them all (136: 14.2, 12.5; 160: 15.0, 12.8). Token-granular
// and 64 x 16K plans cross at the same place.
constexpr int kPairsMost = kPlanThreads / 2;
// Most spans in one bucket: a span counts its bucket's spans before it, so
// one of 512 costs about as much as all pairs among 700 spans.
constexpr int kBucketMost = 512;
// Fewest undecided spans worth filtering after a rejection: four batches of
// the walk (at 128, 288 spans took 16.7 us instead of 14.2).
constexpr int kFilterLeast = 256;

// The ranking order without the index, as one unsigned integer: the prior,
// descending (-0 ranks as +0; NaN never gets here), above the start,
// ascending. Span j ranks before span i iff key_j < key_i, or the keys are
// equal and j < i. No span's key is ~0 (the padding key).
__device__ __forceinline__ uint64_t rank_key(float prior, int start) {
  uint32_t u = __float_as_uint(prior == 0.f ? 0.f : prior);
  u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);   // monotone in the float's value
  return ((uint64_t)~u << 32) | (uint32_t)(start ^ 0x80000000);
}
constexpr uint64_t kPadKey = ~0ull;

// Exclusive prefix sum of v over the workgroup (kPlanThreads threads, in
// thread order); *total receives the sum. s_tmp holds kPlanThreads/64 ints.
__device__ __forceinline__ int block_exclusive_scan(int v, int *s_tmp, int *total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int x = wave_scan_add(v);                      // inclusive, within the wavefront
  if (lane == 63) s_tmp[w] = x;
  __syncthreads();
  int before = 0, all = 0;
#pragma unroll
  for (int i = 0; i < kPlanThreads / 64; ++i) {
    before += (i < w) ? s_tmp[i] : 0;
    all += s_tmp[i];
  }
  __syncthreads();
  *total = all;
  return before + x - v;
}

// Bits of bitmap word w (bits 32w .. 32w + 31) that lie in [x, e).
__device__ __forceinline__ uint32_t range_bits(int w, int x, int e) {
  const int lo = min(max(x - 32 * w, 0), 32);
  const int hi = min(max(e - 32 * w, 0), 32);
  return (uint32_t)(((1ull << hi) - 1ull) ^ ((1ull << lo) - 1ull));
}

// Spare words past the last bitmap word: count_clear reads up to 7 of them.
constexpr int kBitmapPadWords = 8;

// Number of clear bits of the bitmap in [x, e), x < e.
// Page bitmap: a span covers one to three words, counted one at a time.
// Token bitmap: a span covers tens of words. The count is the length of the
// range less its set bits, which are summed over the whole words w0 .. w1 (a
// popcount with accumulate per word) and corrected by the set bits of the two
// end words that lie outside [x, e). The words are read eight at a time before
// they are counted, so that their LDS latencies overlap; a batch may read up
// to seven words past w1 (into the spare words at the end) and counts nothing
// there.
template <bool TOK>
__device__ __forceinline__ int count_clear(const uint32_t* bitmap, int x, int e) {
  if constexpr (!TOK) {
    int c = 0;
    for (int w = x >> 5; w <= (e - 1) >> 5; ++w) c += __popc(range_bits(w, x, e) & ~bitmap[w]);
    return c;
  } else {
    constexpr int kW = 8;
    static_assert(kW <= kBitmapPadWords, "batch reads past the spare words");
    const int w0 = x >> 5, w1 = (e - 1) >> 5;
    const uint32_t below = (1u << (x & 31)) - 1u;            // bits of w0 before x
    const uint32_t above = ~((2u << ((e - 1) & 31)) - 1u);   // bits of w1 from e on
    int set = -(int)(__popc(bitmap[w0] & below) + __popc(bitmap[w1] & above));
    for (int w = w0; w <= w1; w += kW) {
      uint32_t v[kW];
#pragma unroll
      for (int k = 0; k < kW; ++k) v[k] = bitmap[w + k];
      const int last = w1 - w;
#pragma unroll
      for (int k = 0; k < kW; ++k) set += __popc(k <= last ? v[k] : 0u);
    }
    return (e - x) - set;
  }
}

template <bool TOK>
__global__ __launch_bounds__(kPlanThreads) void compile_plan_kernel(PlanArgs a) {
  extern __shared__ uint32_t bitmap[];   // page mode: bit per page; token mode: bit per token
  __shared__ int s_flag;
  __shared__ int s_scan[kPlanThreads / 64];
  __shared__ uint32_t s_minmax[kPlanThreads / 64][4];
  __shared__ long long s_used;
  __shared__ int s_taken;
  __shared__ int s_next;
  // ranking keys; after the ranking (one chunk) each span's (length, start);
  // at the end the view list (and its token masks)
  __shared__ __align__(16) union {
    uint64_t key[kRankChunk];
    struct {
      int page[kRankChunk];
      uint32_t mask[kRankChunk];
    } view;
  } s_u;
  uint64_t *const s_key = s_u.key;
  __shared__ uint16_t s_perm[kRankChunk];    // one chunk: rank -> local span index
  // bucket ranking: counts, then first slots, of two buckets a word; the spans
  // by bucket
  __shared__ uint32_t s_cnt[kRankChunk / 2];
  __shared__ uint16_t s_ord[kRankChunk];

  const int b = blockIdx.x;
  const int tid = threadIdx.x;
  const int lane = tid & 63;

  const int lo = a.span_offsets[b];
  const int hi = a.span_offsets[b + 1];

  auto write_fail = [&](int status, bool zero_flags) {
    if (zero_flags && a.span_selected) {
      for (int i = lo + tid; i < hi; i += kPlanThreads) a.span_selected[i] = 0;
    }
    if (tid == 0) {
      a.view_nblk[b] = 0;
      a.view_tokens[b] = 0;
      a.spans_taken[b] = 0;
      a.status[b] = status;
    }
  };

  if (lo < 0 || hi < lo || hi > a.num_spans) {
    write_fail(5 /*KAP_PLAN_BAD_SPANS*/, false);
    return;
  }
  const int L = a.seq_lens[b];
  const int NP = (L >= 1) ? (int)(((long long)L + kPage - 1) / kPage) : 0;
  if (L < 1 || NP > a.fbt_stride) {
    write_fail(4 /*KAP_PLAN_BAD_LENGTH*/, true);
    return;
  }

  // -- scores, and the first chunk of ranking keys -----------------------------
  // Keys are staged in LDS padded to a multiple of four with the padding key,
  // which no span's key equals or exceeds.
  const int n = hi - lo;
  const bool one_chunk = n <= kRankChunk;
  if (tid == 0) s_flag = 0;
  __syncthreads();
  // (one chunk: priors, starts and the lengths that the greedy walk needs are
  // all loaded before the first is used; the lengths are stored to LDS, beside
  // the starts, once the ranking is done)
  constexpr int kSpanRegs = kRankChunk / kPlanThreads;
  int len_r[kSpanRegs];
  if (one_chunk) {
    float pr[kSpanRegs];
    int st[kSpanRegs];
#pragma unroll
    for (int q = 0; q < kSpanRegs; ++q) {
      if (q * kPlanThreads >= n) break;
      const int t = min(tid + q * kPlanThreads, n - 1);
      pr[q] = a.span_prior[lo + t];
      st[q] = a.span_start[lo + t];
      len_r[q] = a.span_len[lo + t];
    }
#pragma unroll
    for (int q = 0; q < kSpanRegs; ++q) {
      if (q * kPlanThreads >= n) break;
      const int t = tid + q * kPlanThreads;
      if (t < n) {
        if (__builtin_isnan(pr[q])) s_flag = 1;
        s_key[t] = rank_key(pr[q], st[q]);
      }
    }
    if (tid < (-n & 3)) s_key[n + tid] = kPadKey;
  } else {
    for (int t = tid; t < n; t += kPlanThreads) {
      const float pr = a.span_prior[lo + t];
      if (__builtin_isnan(pr)) s_flag = 1;
      if (t < kRankChunk) s_key[t] = rank_key(pr, a.span_start[lo + t]);
    }
  }
  __syncthreads();
  if (s_flag) {
    write_fail(2 /*KAP_PLAN_BAD_SCORE*/, true);
    return;
  }
  // -- mandatory prefix / suffix ----------------------------------------------
  const int pre = min(max(a.prefix[b], 0), L);
  const int suf_start = max(0, L - max(a.suffix[b], 1));
  const int W = TOK ? (L + 31) / 32 : (NP + 31) / 32;  // bitmap words
  if constexpr (TOK) {
    // tokens [0, pre) and [suf_start, L); no bit at or past L is ever set
    for (int w = tid; w < W; w += kPlanThreads)
      bitmap[w] = range_bits(w, 0, pre) | range_bits(w, suf_start, L);
  } else {
    for (int w = tid; w < W; w += kPlanThreads) bitmap[w] = 0u;
    __syncthreads();
    const int pre_pages = (pre + kPage - 1) / kPage;     // pages [0, pre_pages)
    const int suf_page0 = suf_start / kPage;             // pages [suf_page0, NP)
    for (int p = tid; p < pre_pages; p += kPlanThreads) atomicOr(&bitmap[p >> 5], 1u << (p & 31));
    for (int p = suf_page0 + tid; p < NP; p += kPlanThreads)
      atomicOr(&bitmap[p >> 5], 1u << (p & 31));
  }

  // -- rank the spans ---------------------------------------------------------
  // rank(i) = number of spans ordered before span i = #{j : key_j < key_i}
  // + #{j < i : key_j = key_i}. Keys are read from LDS in chunks of
  // kRankChunk (a single chunk, staged above, in the common case), four per
  // two broadcast reads. One pass counts the keys below and equal to key_i;
  // only when some span shares its key with another (equal prior and start)
  // does a second pass count the equal keys of lower index. With few spans,
  // TS = 2, 4 or 8 neighbouring threads share span i, thread s counting over
  // keys 4 s, 4 s + 4 TS, ..., and their counts are summed with lane swaps.
  const int TS = n <= kPlanThreads / 8 ? 8 : n <= kPlanThreads / 4 ? 4 : n <= kPlanThreads / 2 ? 2 : 1;
  const int sub = tid & (TS - 1);
  typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));
  // counts over all chunks: below (ties == false) or equal with lower index
  // (ties == true); every thread takes part (chunk staging has barriers)
  auto count = [&](bool act, int i, uint64_t ki, bool ties, int &c_lt, int &c_eq) {
    for (int jb = 0; jb < n; jb += kRankChunk) {
      const int jn = min(kRankChunk, n - jb);
      const int jn4 = (jn + 3) & ~3;
      if (!one_chunk) {
        __syncthreads();
        for (int t = tid; t < jn4; t += kPlanThreads)
          s_key[t] = t < jn ? rank_key(a.span_prior[lo + jb + t], a.span_start[lo + jb + t]) : kPadKey;
        __syncthreads();
      }
      if (act) {
#pragma unroll 2
        for (int t = 4 * sub; t < jn4; t += 4 * TS) {
          const u64x2 k01 = *reinterpret_cast<const u64x2 *>(&s_key[t]);
          const u64x2 k23 = *reinterpret_cast<const u64x2 *>(&s_key[t + 2]);
          if (!ties) {
            c_lt += (k01.x < ki) + (k01.y < ki) + (k23.x < ki) + (k23.y < ki);
            c_eq += (k01.x == ki) + (k01.y == ki) + (k23.x == ki) + (k23.y == ki);
          } else {
            const int j = jb + t;
            c_eq += ((k01.x == ki) & (j < i)) + ((k01.y == ki) & (j + 1 < i)) +
                    ((k23.x == ki) & (j + 2 < i)) + ((k23.y == ki) & (j + 3 < i));
          }
        }
      }
    }
    // the TS threads of span i are lanes l .. l + TS - 1 of one wavefront
    for (int m = 1; m < TS; m <<= 1) {
      c_lt += __shfl_xor(c_lt, m);
      c_eq += __shfl_xor(c_eq, m);
    }
  };
  bool ranked = false;
  if (one_chunk && n > kPairsMost) {
    // Buckets: the high half of the key (the prior), or where it is the same
    // for all the low half, less its minimum and shifted so that 1024 to 2048
    // buckets cover its range -- monotone, so a span's rank is its bucket's
    // first slot plus its rank among the bucket's spans. With more than
    // kBucketMost spans in one bucket (nearly equal priors) all pairs again.
    constexpr int kPer = kRankChunk / kPlanThreads;
    uint64_t ky[kPer];
    uint32_t lo_h = ~0u, hi_h = 0u, lo_l = ~0u, hi_l = 0u;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int i = tid + q * kPlanThreads;
      ky[q] = i < n ? s_key[i] : kPadKey;
      if (i < n) {
        const uint32_t h = (uint32_t)(ky[q] >> 32), l = (uint32_t)ky[q];
        lo_h = min(lo_h, h);
        hi_h = max(hi_h, h);
        lo_l = min(lo_l, l);
        hi_l = max(hi_l, l);
      }
    }
    for (int w = tid; w < kRankChunk / 2; w += kPlanThreads) s_cnt[w] = 0u;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      lo_h = min(lo_h, (uint32_t)__shfl_xor((int)lo_h, o));
      hi_h = max(hi_h, (uint32_t)__shfl_xor((int)hi_h, o));
      lo_l = min(lo_l, (uint32_t)__shfl_xor((int)lo_l, o));
      hi_l = max(hi_l, (uint32_t)__shfl_xor((int)hi_l, o));
    }
    if (lane == 0) {
      uint32_t *m = s_minmax[tid >> 6];
      m[0] = lo_h; m[1] = hi_h; m[2] = lo_l; m[3] = hi_l;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kPlanThreads / 64; ++w) {
      lo_h = min(lo_h, s_minmax[w][0]);
      hi_h = max(hi_h, s_minmax[w][1]);
      lo_l = min(lo_l, s_minmax[w][2]);
      hi_l = max(hi_l, s_minmax[w][3]);
    }
    const bool by_prior = lo_h != hi_h;
    const uint32_t base = by_prior ? lo_h : lo_l, range = by_prior ? hi_h - lo_h : hi_l - lo_l;
    const int shift = range ? max(0, 32 - 11 - __builtin_clz(range)) : 0;
    int bucket[kPer], place[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int i = tid + q * kPlanThreads;
      if (i < n) {
        bucket[q] = (int)(((by_prior ? (uint32_t)(ky[q] >> 32) : (uint32_t)ky[q]) - base) >> shift);
        const int at = 16 * (bucket[q] & 1);
        place[q] = (atomicAdd(&s_cnt[bucket[q] >> 1], 1u << at) >> at) & 0xFFFF;
      }
    }
    __syncthreads();
    // counts -> first slots, 8 buckets a thread
    uint32_t c[4];
    int sum = 0, most = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      c[w] = s_cnt[4 * tid + w];
      sum += (int)(c[w] & 0xFFFF) + (int)(c[w] >> 16);
      most = max(most, max((int)(c[w] & 0xFFFF), (int)(c[w] >> 16)));
    }
    int all = 0;
    int at = block_exclusive_scan(sum, s_scan, &all);
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const int second = at + (int)(c[w] & 0xFFFF);
      s_cnt[4 * tid + w] = (uint32_t)at | ((uint32_t)second << 16);
      at = second + (int)(c[w] >> 16);
    }
    ranked = !__syncthreads_or(most > kBucketMost);
    if (ranked) {
      int b0[kPer];
#pragma unroll
      for (int q = 0; q < kPer; ++q) {
        const int i = tid + q * kPlanThreads;
        if (i < n) {
          b0[q] = (int)(s_cnt[bucket[q] >> 1] >> (16 * (bucket[q] & 1))) & 0xFFFF;
          s_ord[b0[q] + place[q]] = (uint16_t)i;
        }
      }
      __syncthreads();
#pragma unroll
      for (int q = 0; q < kPer; ++q) {
        const int i = tid + q * kPlanThreads;
        if (i < n) {
          const int nx = bucket[q] + 1;
          const int b1 = nx < kRankChunk ? (int)(s_cnt[nx >> 1] >> (16 * (nx & 1))) & 0xFFFF : n;
          int rank = b0[q];
          for (int e = b0[q]; e < b1; ++e) {
            const int j = s_ord[e];
            const uint64_t kj = s_key[j];
            rank += (kj < ky[q]) | ((kj == ky[q]) & (j < i));
          }
          s_perm[rank] = (uint16_t)i;
          if (a.span_selected) a.span_selected[lo + i] = 0;
        }
      }
    }
  }
  for (int ib = 0; ib < n && !ranked; ib += kPlanThreads / TS) {
    const int i = ib + tid / TS;
    const bool act = i < n;
    uint64_t ki = kPadKey;
    if (act) ki = one_chunk ? s_key[i] : rank_key(a.span_prior[lo + i], a.span_start[lo + i]);
    int below = 0, equal = 0;
    count(act, i, ki, false, below, equal);   // equal counts span i itself
    int rank = below;
    if (__syncthreads_or(act && equal > 1)) {
      int unused = 0, tied = 0;
      count(act, i, ki, true, unused, tied);
      rank += tied;
    }
    if (act && sub == 0) {
      if (one_chunk) s_perm[rank] = (uint16_t)i;
      else a.perm[lo + rank] = i;
      if (a.span_selected) a.span_selected[lo + i] = 0;
    }
  }
  __syncthreads();
  if (one_chunk) {
    // (length, start) of every span for the greedy walk, over its key
#pragma unroll
    for (int q = 0; q < kSpanRegs; ++q) {
      if (q * kPlanThreads >= n) break;
      const int t = tid + q * kPlanThreads;
      if (t < n) s_key[t] = ((uint64_t)(uint32_t)len_r[q] << 32) | (uint32_t)(s_key[t] & 0xffffffffu);
    }
  }
  __syncthreads();

  // -- visible tokens of the mandatory part -----------------------------------
  {
    int c = 0;
    for (int w = tid; w < W; w += kPlanThreads) c += __popc(bitmap[w]);
    int total = 0;
    block_exclusive_scan(c, s_scan, &total);
    if (tid == 0) {
      if constexpr (TOK) {
        s_used = total;
      } else {
        // the last page is always selected (suffix >= 1 token)
        const int last_valid = L - kPage * (NP - 1);    // 1..16
        s_used = (long long)kPage * total - (kPage - last_valid);
      }
      s_taken = 0;
    }
  }
  __syncthreads();

  // -- greedy selection in rank order (one wavefront) -------------------------
  // The spans are walked 64 ranks at a time, lane l holding the span of rank
  // r0 + l as a bit range [u0, u1) of the bitmap (pages; tokens in token mode)
  // and its cost, 1 (16 in page mode: every page but the last, which is always
  // selected, holds 16 tokens) per bit not yet set. Taking spans adds to the
  // used tokens at least what it takes off any other span's cost, so
  //  * a span that does not fit now never will: it is rejected (SKIP), or
  //    selection ends there (STOP);
  //  * the running sum of the costs of the spans that fit bounds what taking
  //    them in order uses, so all up to the first sum above the budget are
  //    taken at once, and the bits they newly set are what they cost.
  // A batch then takes a few rounds, each near the end of the budget smaller,
  // instead of one round per taken span (4 x 128K, 500 spans, 40% budget, of
  // which about 190 taken: 101 -> 24 us per call, with the bucket ranking). The budget state is
  // wavefront-uniform.
  // Once a span was rejected little of the budget is left: the four wavefronts
  // then keep, of a long rest of the ranking, only the spans that still fit
  // (2000 spans: 49 -> 30 us; 475 before all three).
  const int T = a.budget[b];
  // bits [u0, u1) of the bitmap span `li` covers; false if it is empty after
  // clipping to [0, L) (such spans are ignored)
  auto bit_range = [&](int st32, int len32, int &u0, int &u1) {
    const long long x64 = st32 > 0 ? st32 : 0;
    long long e64 = (long long)st32 + (long long)len32;
    if (e64 > L) e64 = L;
    const int x = (int)x64, e = (int)(e64 > x64 ? e64 : x64);
    u0 = TOK ? x : x / kPage;
    u1 = TOK ? e : (e + kPage - 1) / kPage;
    return e > x;
  };
  int r0 = 0, ranks = n;                  // ranks [r0, ranks) are undecided
  while (true) {
    if (tid < 64) {
      int used = __builtin_amdgcn_readfirstlane((int)s_used);
      int taken = 0;
      bool stop = false, rejected = false;
      for (; r0 < ranks && !stop && !(rejected && one_chunk && ranks - r0 > kFilterLeast); r0 += 64) {
        int my_i = -1, st32 = 0, len32 = 0;
        if (r0 + lane < ranks) {
          // (two separate paths: merged into one load from a selected address,
          // the LDS and the global read would both become generic loads)
          int li;
          if (one_chunk) {
            li = s_perm[r0 + lane];
          } else {
            li = a.perm[lo + r0 + lane];
            asm volatile("" ::: "memory");
          }
          my_i = lo + li;
          if (one_chunk) {
            const uint64_t v = s_key[li];
            st32 = (int)((uint32_t)v ^ 0x80000000u);
            len32 = (int)(uint32_t)(v >> 32);
          } else {
            st32 = a.span_start[my_i];
            len32 = a.span_len[my_i];
          }
        }
        int u0, u1;
        const bool valid = bit_range(st32, len32, u0, u1);
        const int words = valid ? ((u1 - 1) >> 5) - (u0 >> 5) + 1 : 0;
        int fresh = valid ? count_clear<TOK>(bitmap, u0, u1) : 0;
        bool open = valid;                                // not yet decided
        bool my_taken = false;
        while (true) {
          const int cost = TOK ? fresh : kPage * fresh;
          const bool fits = open && used + cost <= T;
          unsigned long long mf = __ballot(fits);
          if (a.policy == 1 /*KAP_SELECT_STOP*/) {
            // only the spans before the first that does not fit are left
            const unsigned long long mx = __ballot(open && !fits);
            if (mx) {
              mf &= (mx & -mx) - 1;
              stop = mf == 0;
            }
          } else {
            rejected |= __ballot(open && !fits) != 0;
            open = fits;
          }
          if (mf == 0) break;
          // take the fitting spans, in order, up to the first whose sum exceeds
          // the budget
          unsigned long long take = mf;
          if (mf & (mf - 1)) {
            const int upto = used + wave_scan_add((mf >> lane) & 1 ? cost : 0);
            const unsigned long long over = mf & __ballot(upto > T);
            if (over) take = mf & ((over & -over) - 1);
          }
          const bool mine = (take >> lane) & 1;
          taken += __popcll(take);
          my_taken |= mine;
          open &= !mine;
          if ((take & (take - 1)) == 0) {
            // one span: its cost is exact, and what it newly covers of another
            // is what is clear in the overlap
            const int j = __builtin_ctzll(take);
            const int ju0 = __builtin_amdgcn_readlane(u0, j);
            const int ju1 = __builtin_amdgcn_readlane(u1, j);
            used += __builtin_amdgcn_readlane(cost, j);
            const int c0 = max(u0, ju0), c1 = min(u1, ju1);
            if (open && c0 < c1) fresh -= count_clear<TOK>(bitmap, c0, c1);
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            const int jw1 = (ju1 - 1) >> 5;
            for (int w = (ju0 >> 5) + lane; w <= jw1; w += 64)
              atomicOr(&bitmap[w], range_bits(w, ju0, ju1));
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            continue;
          }
          // set their bits, counting those that were clear: short spans a lane
          // each, long ones (up to 64 words at a time) all lanes together
          constexpr int kOwnWords = TOK ? 2 : 4;
          int added = 0;
          if (mine && words <= kOwnWords) {
            for (int w = u0 >> 5; w <= (u1 - 1) >> 5; ++w) {
              const uint32_t m = range_bits(w, u0, u1);
              added += __popc(m & ~atomicOr(&bitmap[w], m));
            }
          }
          unsigned long long wide = __ballot(mine && words > kOwnWords);
          while (wide) {
            const int j = __builtin_ctzll(wide);
            wide &= wide - 1;
            const int ju0 = __builtin_amdgcn_readlane(u0, j);
            const int ju1 = __builtin_amdgcn_readlane(u1, j);
            const int jw1 = (ju1 - 1) >> 5;
            for (int w = (ju0 >> 5) + lane; w <= jw1; w += 64) {
              const uint32_t m = range_bits(w, ju0, ju1);
              added += __popc(m & ~atomicOr(&bitmap[w], m));
            }
          }
          added = lane63(wave_scan_add(added));
          used += TOK ? added : kPage * added;
          __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
          if (open) fresh = count_clear<TOK>(bitmap, u0, u1);
        }
        if (a.span_selected && my_taken) a.span_selected[my_i] = 1;
      }
      if (lane == 0) {
        s_used = used;
        s_taken += taken;
        s_next = stop ? ranks : r0;
      }
    }
    __syncthreads();
    r0 = s_next;
    if (r0 >= ranks) break;
    // thread t keeps, of the ranks r0 + 8 t .. + 7, those that fit
    const int left_to = min(ranks, r0 + 8 * (tid + 1));
    int keep = 0, at = 0;
    unsigned which = 0;
    for (int r = r0 + 8 * tid; r < left_to; ++r) {
      const uint64_t v = s_key[s_perm[r]];
      int u0, u1;
      if (bit_range((int)((uint32_t)v ^ 0x80000000u), (int)(uint32_t)(v >> 32), u0, u1) &&
          s_used + (TOK ? 1 : kPage) * count_clear<TOK>(bitmap, u0, u1) <= T) {
        which |= 1u << (r - r0 - 8 * tid);
        ++keep;
      }
    }
    int kept = 0;
    at = block_exclusive_scan(keep, s_scan, &kept);
    for (; which; which &= which - 1) s_ord[at++] = s_perm[r0 + 8 * tid + __builtin_ctz(which)];
    __syncthreads();
    for (int r = tid; r < kept; r += kPlanThreads) s_perm[r] = s_ord[r];
    r0 = 0;
    ranks = kept;
    __syncthreads();
  }

  // -- compaction: ascending logical pages -> block table ---------------------
  // Token mode: page p is the half p & 1 of token word p >> 1 and is in the
  // view when any of its 16 bits is set; that half is its token mask.
  const int chunk = (W + kPlanThreads - 1) / kPlanThreads;
  const int w0 = min(W, tid * chunk);
  const int w1 = min(W, w0 + chunk);
  int mine = 0;
  for (int w = w0; w < w1; ++w) {
    const uint32_t x = bitmap[w];
    mine += TOK ? ((x & 0xFFFFu) != 0u) + ((x >> 16) != 0u) : __popc(x);
  }
  if (tid == 0) s_flag = 0;
  int nblk = 0;
  const int first = block_exclusive_scan(mine, s_scan, &nblk);
  if (nblk > a.capacity) {
    write_fail(1 /*KAP_PLAN_OVER_CAPACITY*/, true);
    return;
  }
  const int32_t *fbt_row = a.fbt + (size_t)b * a.fbt_stride;
  int32_t *vbt = a.view_bt + (size_t)b * a.capacity;
  int32_t *vlb = a.view_lblk + (size_t)b * a.capacity;
  uint32_t *vmk = TOK ? a.view_mask + (size_t)b * a.capacity : nullptr;
  bool bad = false;
  // kRankChunk entries at a time, the logical pages (and masks) go to LDS at
  // their output index, then every thread maps entries k, k + 256, ... through
  // the full block table, so that the table reads are all in flight at once.
  for (int k0 = 0; k0 < nblk; k0 += kRankChunk) {
    if (k0 > 0) __syncthreads();             // the entries before are read
    int out = first - k0;                    // below 0 or past the chunk: another chunk's
    auto emit = [&](int p, uint32_t mask) {
      if (out >= 0 && out < kRankChunk) {
        s_u.view.page[out] = p;
        if constexpr (TOK) s_u.view.mask[out] = mask;
      }
      ++out;
    };
    if (out < kRankChunk && out + mine > 0) {
      for (int w = w0; w < w1; ++w) {
        const uint32_t x = bitmap[w];
        if constexpr (TOK) {
          if (x & 0xFFFFu) emit(2 * w, x & 0xFFFFu);
          if (x >> 16) emit(2 * w + 1, x >> 16);
        } else {
          uint32_t bits = x;
          while (bits) {
            const int bit = __ffs(bits) - 1;
            bits &= bits - 1u;
            emit(w * 32 + bit, 0u);
          }
        }
      }
    }
    __syncthreads();
    const int cnt = min(kRankChunk, nblk - k0);
    constexpr int kPer = kRankChunk / kPlanThreads;
    int pg[kPer], page[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      if (q * kPlanThreads >= cnt) break;
      const int k = tid + q * kPlanThreads;
      if (k < cnt) {
        pg[q] = s_u.view.page[k];
        page[q] = fbt_row[pg[q]];
      }
    }
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      if (q * kPlanThreads >= cnt) break;
      const int k = tid + q * kPlanThreads;
      if (k < cnt) {
        bad |= (page[q] < 0) || ((int64_t)page[q] >= a.num_pages);
        vlb[k0 + k] = pg[q];
        vbt[k0 + k] = page[q];
        if constexpr (TOK) vmk[k0 + k] = s_u.view.mask[k];
      }
    }
  }
  if (bad) s_flag = 1;
  __syncthreads();
  if (s_flag) {
    write_fail(3 /*KAP_PLAN_BAD_PAGE*/, true);
    return;
  }
  if (tid == 0) {
    a.view_nblk[b] = nblk;
    a.view_tokens[b] = (int)s_used;
    a.spans_taken[b] = s_taken;
    a.status[b] = 0;
  }
}

size_t plan_lds_bytes(int fbt_stride, bool token_mode) {
  // page mode: a bit per page; token mode: a bit per token (16 per page)
  const size_t words = token_mode ? ((size_t)fbt_stride * kPage + 31) / 32
                                  : ((size_t)fbt_stride + 31) / 32;
  return (words + kBitmapPadWords) * sizeof(uint32_t);
}

}  // namespace

hipError_t launch_compile_plan(const PlanArgs &a, hipStream_t s) {
  const bool tok = a.token_mode != 0;
  const size_t lds = plan_lds_bytes(a.fbt_stride, tok);
  if (tok)
    hipLaunchKernelGGL(compile_plan_kernel<true>, dim3(a.batch), dim3(kPlanThreads), lds, s, a);
  else
    hipLaunchKernelGGL(compile_plan_kernel<false>, dim3(a.batch), dim3(kPlanThreads), lds, s, a);
  return hipGetLastError();
}

}  // namespace kap
