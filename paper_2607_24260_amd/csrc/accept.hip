// Target-guided tolerant acceptance of a verify window (Sec. 3.2 of the
// paper, "Full-context verification": a proposed token is accepted when it is
// among the verifier's top candidates; top 3 in the paper).
//
// A grid of (vocabulary chunk, window row) workgroups streams the verifier's
// logits, each counting the tokens of its chunk that rank before the row's
// draft token and taking the chunk's argmax; both are combined per row with
// device-scope vector atomics (integer add, and 64-bit max of (orderable
// value, inverted index), so the largest value and then the lowest index win).
// The workgroup that completes a window sets the accepted count m and the carry
// token argmax(row m), and zeroes the row counters for the next call. Integer
// results: exact.
//
// Bound by HBM (64 x 5 rows of 151936 bf16 logits, 97 MB: 20.6 us per call,
// 22.7 before), as long as a logit costs three and a half vector
// instructions: one to widen it, a compare and a counting
// add, and half a three-way maximum -- the index of the maximum is found
// afterwards, in the 16 bytes that held it. Rows need not be 16-byte
// aligned: the loads are, and the few tokens before and after them go one by
// one (43 x 2 rows of 69433 bf16 logits: 7.5 us, 25 one by one).
#include "kap_internal.h"

#include <algorithm>

namespace kap {
namespace {

constexpr int kThreads = 256;
// Launch shape: about three workgroups per CU (64 x 5 rows of 151936 tokens 20.4
// us; two 23.7, five 22.1) of at least 4096 16-byte loads of a row each (with
// 2048, 14 x 8 rows of 81945 float32 tokens took 11.9 us instead of 10.3: every
// workgroup ends in a chain of atomics). A thread has two to four loads in
// flight (four to eight: 22.2 us).
constexpr int kAcceptPerCU = 3;
constexpr int kAcceptLeast = 4096;
constexpr uint32_t kAcceptArrival = 1u << 20;
constexpr int kAcceptCountMask = (1 << 20) - 1;

// Monotone map of a float to an unsigned key (-0 folded into +0).
__device__ __forceinline__ uint32_t order_key(float x) {
  if (x == 0.f) x = 0.f;
  const uint32_t u = __float_as_uint(x);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

template <int F32>
__device__ __forceinline__ float load1(const void *row, int j) {
  if constexpr (F32) return static_cast<const float *>(row)[j];
  return __uint_as_float((uint32_t)static_cast<const uint16_t *>(row)[j] << 16);
}

// The largest float below x (x not -inf, not NaN): y >= x iff y > below(x).
__device__ __forceinline__ float below(float x) {
  const uint32_t u = __float_as_uint(x);
  return __uint_as_float(x == 0.f ? 0x80000001u : ((u & 0x80000000u) ? u + 1 : u - 1));
}

template <int F32>
__device__ __forceinline__ float value(const kv_u32x4 &r, int e) {
  if constexpr (F32) return __uint_as_float(r[e]);
  return (e & 1) ? bf16_hi(r[e >> 1]) : bf16_lo(r[e >> 1]);
}

// The largest of three (a NaN operand is passed over); as an instruction,
// because the compiler quiets every operand of its own maximum first.
__device__ __forceinline__ float max3(float x, float y, float z) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(x), "v"(y), "v"(z));
  return r;
}

// m and carry of sequence b from its rows' counts and maxima, which become
// zero; one wavefront. Counts of 20 bits if packed (see the row kernel).
__device__ __forceinline__ void finish_window(const AcceptArgs &a, int b, bool packed) {
  const int lane = threadIdx.x & 63, k = a.window - 1;
  int32_t *count = a.row_count + (size_t)b * a.window;
  unsigned long long *best = a.row_best + (size_t)b * a.window;
  bool pass = false;
  unsigned long long mine = 0;
  if (lane < a.window) {
    int c = __hip_atomic_load(count + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (packed) c &= kAcceptCountMask;
    mine = __hip_atomic_load(best + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (lane < k) {
      const int d = a.drafts[(size_t)b * k + lane];
      pass = d >= 0 && d < a.vocab && c < a.top_k;
    }
    __hip_atomic_store(count + lane, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(best + lane, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  const int m = __builtin_ctzll(~__ballot(pass));   // <= k: lane k never passes
  const uint32_t index = 0xFFFFFFFFu - (uint32_t)__shfl((int)(uint32_t)mine, m, 64);
  if (lane == 0) {
    a.accepted[b] = m;
    a.carry[b] = (int)index;
  }
}

// FUSED: arrivals are counted in the upper 12 bits of the row counts, whose
// lower 20 hold the sum of the chunks' counts, each cut to top_k (only whether
// it reaches top_k matters); the last row has no draft and counts the window's
// completed rows there.
template <int F32, bool FUSED>
__global__ __launch_bounds__(kThreads) void accept_rows_kernel(AcceptArgs a) {
  constexpr int kVec = F32 ? 4 : 8;                    // logits of a 16-byte load
  constexpr int kLoads = 2;                            // in flight, and as many being used
  __shared__ int s_cnt[kThreads / 64];
  __shared__ unsigned long long s_best[kThreads / 64];
  const int row = blockIdx.y;                          // b * window + i
  const int b = row / a.window, i = row - b * a.window;
  const char *lrow = static_cast<const char *>(a.logits) + (size_t)row * a.vocab * (F32 ? 4 : 2);
  // the draft of this position (none for the last one, or out of range)
  const int d = i < a.window - 1 ? a.drafts[(size_t)b * (a.window - 1) + i] : -1;
  const bool has_d = d >= 0 && d < a.vocab;
  const float xd = has_d ? load1<F32>(lrow, d) : 0.f;
  // tokens head .. head + kVec * vecs - 1 come in aligned 16-byte loads
  const int head = min(a.vocab, (int)((-reinterpret_cast<uintptr_t>(lrow) & 15) / (F32 ? 4 : 2)));
  const int vecs = (a.vocab - head) / kVec;
  const kv_u32x4 *vrow = reinterpret_cast<const kv_u32x4 *>(lrow + (size_t)head * (F32 ? 4 : 2));
  const int v0 = blockIdx.x * a.chunk_loads;
  const int v1 = min(vecs, v0 + a.chunk_loads);

  // Token j ranks before the draft iff x > xd, or x == xd and j < d: that is
  // x > before for j < d, x > xd for j > d. (-inf has nothing below: such a
  // draft is compared token by token.)
  const bool plain = has_d && xd == -INFINITY;
  const float before = plain ? xd : below(xd);
  int cnt = 0;
  // Each thread visits its tokens in increasing index order, so a strict >
  // keeps the lowest index among equal maxima.
  float bv = -INFINITY;
  int bi = -1, bvec = -1;                              // token, or load, that holds bv
  auto ranks_before = [&](float x, int j) { return (x > xd) | ((x == xd) & (j < d)); };
  auto visit = [&](float x, int j) {
    cnt += ranks_before(x, j);
    if ((bi & bvec) < 0 || x > bv) {
      bv = x;
      bi = j;
      bvec = -1;
    }
  };
  if (blockIdx.x == 0 && (int)threadIdx.x < head) visit(load1<F32>(lrow, threadIdx.x), threadIdx.x);
  auto load = [&](kv_u32x4 r[kLoads], int v) {         // past the end: the last load again
#pragma unroll
    for (int u = 0; u < kLoads; ++u) r[u] = vrow[min(v + u * kThreads, v1 - 1)];
  };
  auto use = [&](const kv_u32x4 r[kLoads], int vb) {
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
      const int v = vb + u * kThreads;
      const int j = head + v * kVec;
      const bool in = v < v1;
      const bool at_d = (unsigned)(d - j) < (unsigned)kVec;
      // +inf counts nothing
      const float t = in && has_d && !plain && !at_d ? (j < d ? before : xd) : INFINITY;
      float x[kVec];
#pragma unroll
      for (int e = 0; e < kVec; ++e) {
        x[e] = value<F32>(r[u], e);
        cnt += x[e] > t;
      }
      float mx = max3(x[0], x[1], x[2]);
      if constexpr (kVec == 8) mx = max3(mx, x[6], max3(x[3], x[4], x[5]));
      mx = max3(mx, x[kVec - 1], x[kVec - 1]);
      if (in && (at_d || plain)) {
#pragma unroll
        for (int e = 0; e < kVec; ++e) cnt += ranks_before(x[e], j + e);
      }
      if (in && ((bi & bvec) < 0 || mx > bv)) {
        bv = mx;
        bvec = v;
        bi = -1;
      }
    }
  };
  if (v0 < v1) {
    constexpr int kStep = kLoads * kThreads;
    kv_u32x4 r0[kLoads], r1[kLoads];
    int v = v0 + threadIdx.x;
    load(r0, v);
    for (int left = v1 - v0; left > 0; left -= 2 * kStep, v += 2 * kStep) {
      load(r1, v + kStep);
      use(r0, v);
      load(r0, v + 2 * kStep);
      use(r1, v + kStep);
    }
  }
  if (blockIdx.x == gridDim.x - 1) {
    const int j = head + vecs * kVec + threadIdx.x;
    if (j < a.vocab) visit(load1<F32>(lrow, j), j);
  }
  if (bvec >= 0) {
    // the first token of the load that has its maximum
    const kv_u32x4 w = vrow[bvec];
    bi = 0;
#pragma unroll
    for (int e = kVec - 1; e >= 0; --e) bi = value<F32>(w, e) == bv ? e : bi;
    bi += head + bvec * kVec;
  }
  if (!has_d) cnt = 0;
  unsigned long long best =
      bi < 0 ? 0ull : ((unsigned long long)order_key(bv) << 32) | (0xFFFFFFFFu - (uint32_t)bi);
  // workgroup reduction, then one atomic each per workgroup
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    cnt += __shfl_xor(cnt, o, 64);
    const unsigned long long y = __shfl_xor(best, o, 64);
    best = y > best ? y : best;
  }
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    s_cnt[w] = cnt;
    s_best[w] = best;
  }
  __syncthreads();
  if (threadIdx.x >= 64) return;
  int c = 0;
  unsigned long long m = 0;
#pragma unroll
  for (int k = 0; k < kThreads / 64; ++k) {
    c += s_cnt[k];
    m = s_best[k] > m ? s_best[k] : m;
  }
  bool last = false;
  if (threadIdx.x == 0) {
    atomicMax(a.row_best + row, m);
    if constexpr (!FUSED) {
      if (c) atomicAdd(a.row_count + row, c);
    } else {
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): the maximum is in before the arrival
      asm volatile("" ::: "memory");
      const uint32_t add = kAcceptArrival + (uint32_t)min(c, a.top_k);
      const uint32_t was = (uint32_t)__hip_atomic_fetch_add(a.row_count + row, (int)add,
                                                            __ATOMIC_RELAXED,
                                                            __HIP_MEMORY_SCOPE_AGENT);
      if (was / kAcceptArrival == gridDim.x - 1)
        last = (__hip_atomic_fetch_add(a.row_count + (size_t)b * a.window + a.window - 1, 1,
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) &
                kAcceptCountMask) == a.window - 1;
    }
  }
  if constexpr (FUSED)
    if (__any(last)) finish_window(a, b, true);
}

__global__ __launch_bounds__(64) void accept_finalize_kernel(AcceptArgs a) {
  finish_window(a, blockIdx.x, false);
}

template <bool FUSED>
void launch_rows(const AcceptArgs &a, dim3 grid, hipStream_t s) {
  if (a.f32)
    hipLaunchKernelGGL((accept_rows_kernel<1, FUSED>), grid, dim3(kThreads), 0, s, a);
  else
    hipLaunchKernelGGL((accept_rows_kernel<0, FUSED>), grid, dim3(kThreads), 0, s, a);
}

}  // namespace

hipError_t launch_accept_top3(const AcceptArgs &a, hipStream_t s) {
  // About kAcceptPerCU workgroups per CU, each of at least kAcceptLeast loads.
  const long long rows = (long long)a.batch * a.window;
  const long long loads = std::max(1ll, (long long)a.vocab * (a.f32 ? 4 : 2) / 16);
  const long long want = std::max(1ll, (long long)kAcceptPerCU * a.cus / rows);
  const long long chunk = std::max<long long>(kAcceptLeast, (loads + want - 1) / want);
  const long long chunks = (loads + chunk - 1) / chunk;
  AcceptArgs c = a;
  c.chunk_loads = (int)chunk;
  const dim3 grid((unsigned)chunks, (unsigned)rows);
  // arrivals and counts fit their bits (a count is at most a chunk's tokens);
  // otherwise the windows are finished by a second launch
  const long long most = std::min<long long>(a.top_k, chunk * 8 + 16);
  if (chunks * most <= kAcceptCountMask && chunks * (long long)kAcceptArrival < (1ll << 32)) {
    launch_rows<true>(c, grid, s);
    return hipGetLastError();
  }
  launch_rows<false>(c, grid, s);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(accept_finalize_kernel, dim3(a.batch), dim3(64), 0, s, a);
  return hipGetLastError();
}

}  // namespace kap
