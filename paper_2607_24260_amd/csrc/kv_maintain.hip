// KV maintenance kernels: the slot-mapped append of new tokens (Sec. 3.1
// slot mappings; Sec. 3.2 KV^{full,+}) and the copy of a selected-KV view
// into a compact workspace of fixed capacity (Alg. 1, AssignCompactSlots and
// BuildBlockTable; Sec. 3.1 "Selected-KV view materialization").
//
// Both move stored bits only (no arithmetic), so their results are exact.
// The compaction streams whole pages: in the library's layout the K tiles of
// all KV heads of one page are one contiguous block (and so are the V
// tiles), copied with 16-byte nontemporal loads and stores.
#include "kap_internal.h"

#include <type_traits>

namespace kap {
namespace {

constexpr int kThreads = 256;

// ---------------------------------------------------------------------------
// append
// ---------------------------------------------------------------------------

// One workgroup per token, element by element (type T, the stored KV type):
// for source arrays that are not 16-byte aligned. K: element (g, d) of the
// token goes to [page][g][d / 8][off][d % 8]; V: to [page][g][d][off].
template <typename T>
__device__ void append_token(const AppendArgs &a, int t, int64_t page, int off) {
  const int Hkv = a.Hkv, D = a.D, C = D / 8;
  const T *kn = static_cast<const T *>(a.k_new) + (size_t)t * Hkv * D;
  const T *vn = static_cast<const T *>(a.v_new) + (size_t)t * Hkv * D;
  T *kp = static_cast<T *>(a.k_pages) + (size_t)page * Hkv * D * kPage;
  T *vp = static_cast<T *>(a.v_pages) + (size_t)page * Hkv * D * kPage;
  for (int e = threadIdx.x; e < Hkv * D; e += blockDim.x) {
    const int g = e / D, d = e - g * D;
    kp[(((size_t)g * C + d / 8) * kPage + off) * 8 + (d & 7)] = kn[e];
    vp[((size_t)g * D + d) * kPage + off] = vn[e];
  }
}

__global__ __launch_bounds__(kThreads) void append_kv_kernel(AppendArgs a) {
  const int t = blockIdx.x;
  const int64_t slot = a.slots[t];
  if (slot < 0) return;                                   // padding
  if (slot >= a.num_pages * kPage) {
    if (threadIdx.x == 0 && a.bad_slots) atomicAdd(a.bad_slots, 1);
    return;
  }
  const int64_t page = slot / kPage;
  const int off = (int)(slot - page * kPage);
  if (a.elem_bytes == 4)
    append_token<uint32_t>(a, t, page, off);
  else if (a.elem_bytes == 2)
    append_token<uint16_t>(a, t, page, off);
  else
    append_token<uint8_t>(a, t, page, off);
}

// Sixteen tokens at a time. A whole page -- 16 consecutive input tokens in the
// 16 slots of one page, as in the middle of a prefill chunk -- is moved by the
// workgroups (blockIdx.x) of the 16 tokens it starts in, wherever in them it
// starts; every other token by the workgroups of its own 16. blockIdx.y names
// the part of the row: parts 2 p move columns 256 p .. of K, parts 2 p + 1 of
// V, a column being 4 bytes of a token (4 / ES dims).
//  * K keeps a token's eight dims of a chunk together: they move as one piece
//    (8 ES bytes), neighbouring lanes neighbouring tokens.
//  * V is transposed. A lane reads its column of the 16 tokens; for a whole
//    page it turns the 16 x 4 bytes around in registers, giving the 64
//    contiguous bytes of its rows, which go out through LDS so that a store
//    instruction covers 1 KB; other tokens are stored as single elements.
// Tokens outside whole pages are also shared out over blockIdx.z: with few of
// them the workgroups are few, and one that moves 16 tokens one after the other
// takes as long (8 KV heads of 128 dims, fp8: 64 tokens in 64 places 3.9 us, one
// workgroup for all 16 tokens 9.9; 64 windows of 5 tokens 4.4, 10.2). Up to
// kAppendWorkgroups in all: more find nothing to do.
// All loads of a whole page are in flight together: at one token per sequence
// latency is all there is, at whole pages HBM: 4 x 2048 bf16 tokens, 8 KV heads
// of 128 dims (67 MB) in 24.9 us per call; one workgroup per token with
// 2-byte stores 16 and 32 bytes apart took 49 us. (Nontemporal loads: 30 us -- new
// tokens come from the caches of the kernels that made them.)
constexpr int kAppendWorkgroups = 1024;
template <int ES>
__device__ __forceinline__ void transpose_column(const uint32_t x[kPage], uint32_t o[kPage]) {
  // o: rows of the column's dims, 4 ES dwords each
  if constexpr (ES == 4) {
#pragma unroll
    for (int i = 0; i < kPage; ++i) o[i] = x[i];
  } else if constexpr (ES == 2) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {          // tokens 2 i, 2 i + 1
      o[i] = __builtin_amdgcn_perm(x[2 * i + 1], x[2 * i], 0x05040100u);
      o[8 + i] = __builtin_amdgcn_perm(x[2 * i + 1], x[2 * i], 0x07060302u);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) {          // tokens 4 i .. 4 i + 3: a 4 x 4 byte transpose
      const uint32_t a01 = __builtin_amdgcn_perm(x[4 * i + 1], x[4 * i], 0x05010400u);
      const uint32_t a23 = __builtin_amdgcn_perm(x[4 * i + 3], x[4 * i + 2], 0x05010400u);
      const uint32_t b01 = __builtin_amdgcn_perm(x[4 * i + 1], x[4 * i], 0x07030602u);
      const uint32_t b23 = __builtin_amdgcn_perm(x[4 * i + 3], x[4 * i + 2], 0x07030602u);
      o[i] = __builtin_amdgcn_perm(a23, a01, 0x05040100u);
      o[4 + i] = __builtin_amdgcn_perm(a23, a01, 0x07060302u);
      o[8 + i] = __builtin_amdgcn_perm(b23, b01, 0x05040100u);
      o[12 + i] = __builtin_amdgcn_perm(b23, b01, 0x07060302u);
    }
  }
}

template <int ES>
__global__ __launch_bounds__(kThreads) void append_runs_kernel(AppendArgs a) {
  typedef uint32_t piece __attribute__((ext_vector_type(ES == 1 ? 2 : 4)));
  constexpr int kPer = ES == 4 ? 2 : 1;        // pieces of a K chunk
  constexpr int kColDims = 4 / ES;
  constexpr int kPartChunks = 32 * kColDims;   // K chunks in 256 columns
  constexpr int kSteps = kPartChunks / 16;     // 16 chunks x 16 tokens at a time
  typedef typename std::conditional<
      ES == 4, uint32_t, typename std::conditional<ES == 2, uint16_t, uint8_t>::type>::type elem;
  __shared__ kv_u32x4 s_rows[kThreads / 64][256];
  const int lane = threadIdx.x & 63;
  const int t0 = blockIdx.x * kPage;
  const int part = blockIdx.y >> 1;
  const bool is_v = blockIdx.y & 1;
  const size_t row = (size_t)a.Hkv * a.D;      // elements of a token
  const int cols = (int)(row / kColDims);

  // Lane l looks at token t0 - 16 + l: is it in the slot after the token before
  // it, on the same page; and does its page's first token start 15 such?
  const int t = t0 - kPage + lane;
  const int64_t slot = t >= 0 && t < a.num_tokens ? a.slots[t] : -1;
  const bool good = slot >= 0 && slot < a.num_pages * kPage;
  const int64_t before = __shfl_up(slot, 1, 64);
  const int off = (int)(slot & (kPage - 1));
  const unsigned long long joined =
      __ballot(lane > 0 && good && before >= 0 && slot == before + 1 && off != 0);
  const int first = lane - off;                // lane of the page's first token
  const bool whole = good && first >= 0 && first + 15 < 64 &&
                     ((joined >> first >> 1) & 0x7FFFu) == 0x7FFFu;
  const bool mine = lane >= kPage && lane < 2 * kPage;
  const unsigned long long starts = __ballot(mine && whole && off == 0);   // at most one
  // of the other tokens, this workgroup's share
  const unsigned single = (unsigned)(__ballot(mine && good && !whole &&
                                              lane % gridDim.z == blockIdx.z) >> kPage);
  if (blockIdx.y == 0 && blockIdx.z == 0 && threadIdx.x < 64 && mine && slot >= 0 && !good &&
      a.bad_slots)
    atomicAdd(a.bad_slots, 1);

  auto slot_at = [&](int l) {                  // slot of lane l (the same l in every lane)
    return ((int64_t)__builtin_amdgcn_readlane((int)(slot >> 32), l) << 32) |
           (uint32_t)__builtin_amdgcn_readlane((int)slot, l);
  };
  auto move_k = [&](int token, bool live, int64_t to) {
    const piece *src = reinterpret_cast<const piece *>(static_cast<const elem *>(a.k_new) +
                                                       (size_t)token * row);
    piece *dst = reinterpret_cast<piece *>(static_cast<elem *>(a.k_pages) +
                                           (size_t)(to / kPage) * row * kPage) +
                 (to & (kPage - 1)) * kPer;
    const int c0 = part * kPartChunks + (threadIdx.x >> 4);
    const int chunks = live ? (int)(row / 8) : 0;
    piece x[kSteps][kPer];
#pragma unroll
    for (int u = 0; u < kSteps; ++u)
#pragma unroll
      for (int h = 0; h < kPer; ++h)
        if (c0 + 16 * u < chunks) x[u][h] = src[(c0 + 16 * u) * kPer + h];
#pragma unroll
    for (int u = 0; u < kSteps; ++u)
#pragma unroll
      for (int h = 0; h < kPer; ++h)
        if (c0 + 16 * u < chunks) dst[(size_t)(c0 + 16 * u) * kPage * kPer + h] = x[u][h];
  };
  const int col = part * kThreads + threadIdx.x;
  auto load_v = [&](int token, unsigned which, uint32_t x[kPage]) {   // tokens token + i, i in which
    const uint32_t *src = reinterpret_cast<const uint32_t *>(static_cast<const elem *>(a.v_new) +
                                                             (size_t)token * row) + col;
#pragma unroll
    for (int i = 0; i < kPage; ++i)
      if (col < cols && ((which >> i) & 1u))
        x[i] = src[(size_t)i * cols];
  };

  if (starts && blockIdx.z == 0) {
    const int f = __builtin_ctzll(starts);     // lane
    const int64_t to = slot_at(f);
    const int token = t0 - kPage + f;
    if (!is_v) {
      move_k(token + (threadIdx.x & 15), true, to + (threadIdx.x & 15));
    } else {
      uint32_t x[kPage] = {}, o[kPage];
      load_v(token, 0xFFFFu, x);
      transpose_column<ES>(x, o);
      // (16-byte units, rotated by column so that the lanes of a write spread
      // over the banks)
      kv_u32x4 *buf = s_rows[threadIdx.x >> 6];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        buf[4 * lane + ((i + (lane >> 1)) & 3)] =
            kv_u32x4{o[4 * i], o[4 * i + 1], o[4 * i + 2], o[4 * i + 3]};
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      const int col0 = part * kThreads + (threadIdx.x & ~63);   // the wavefront's first column
      kv_u32x4 *dst = reinterpret_cast<kv_u32x4 *>(static_cast<elem *>(a.v_pages) +
                                                   (size_t)(to / kPage) * row * kPage +
                                                   (size_t)col0 * kColDims * kPage);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int u = 64 * i + lane, c = u >> 2;
        if (col0 + c < cols) dst[u] = buf[4 * c + (((u & 3) + (c >> 1)) & 3)];
      }
    }
  }
  if (single) {
    if (!is_v) {
      const int i = threadIdx.x & 15;
      const int64_t to = ((int64_t)__shfl((int)(slot >> 32), kPage + i, 64) << 32) |
                         (uint32_t)__shfl((int)slot, kPage + i, 64);
      const bool live = (single >> i) & 1u;
      move_k(live ? t0 + i : t0, live, live ? to : 0);
    } else {
      // element by element, so that a store instruction covers 64 neighbouring
      // rows; more tokens at a time cost the small calls code to fetch
      const elem *src = static_cast<const elem *>(a.v_new) + (size_t)t0 * row;
      const size_t e0 = (size_t)part * kThreads * kColDims + threadIdx.x;
      for (unsigned left = single; left;) {
        constexpr int kBatch = ES == 4 ? 8 : 4;
        int token[kBatch];
        elem x[kBatch][kColDims];
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
          token[i] = left ? __builtin_ctz(left) : -1;
          left &= left - 1;
#pragma unroll
          for (int e = 0; e < kColDims; ++e)
            if (token[i] >= 0 && e0 + e * kThreads < row)
              x[i][e] = src[token[i] * row + e0 + e * kThreads];
        }
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
          if (token[i] < 0) continue;
          const int64_t to = slot_at(kPage + token[i]);
          elem *dst = static_cast<elem *>(a.v_pages) + (size_t)(to / kPage) * row * kPage +
                      (to & (kPage - 1));
#pragma unroll
          for (int e = 0; e < kColDims; ++e)
            if (e0 + e * kThreads < row) dst[(e0 + e * kThreads) * kPage] = x[i][e];
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// compaction: workgroups stride over (sequence, view entry)
// ---------------------------------------------------------------------------

__device__ __forceinline__ void copy_block(const char *src, char *dst, size_t bytes) {
  // bytes is a multiple of 16 (Hkv * D * 16 elements of >= 1 byte, D % 8 == 0)
  const kv_u32x4 *s = reinterpret_cast<const kv_u32x4 *>(src);
  kv_u32x4 *d = reinterpret_cast<kv_u32x4 *>(dst);
  const size_t n = bytes / 16;
  size_t i = threadIdx.x;
  for (; i + 3 * kThreads < n; i += 4 * kThreads) {
    const kv_u32x4 x0 = __builtin_nontemporal_load(s + i);
    const kv_u32x4 x1 = __builtin_nontemporal_load(s + i + kThreads);
    const kv_u32x4 x2 = __builtin_nontemporal_load(s + i + 2 * kThreads);
    const kv_u32x4 x3 = __builtin_nontemporal_load(s + i + 3 * kThreads);
    __builtin_nontemporal_store(x0, d + i);
    __builtin_nontemporal_store(x1, d + i + kThreads);
    __builtin_nontemporal_store(x2, d + i + 2 * kThreads);
    __builtin_nontemporal_store(x3, d + i + 3 * kThreads);
  }
  for (; i < n; i += kThreads) __builtin_nontemporal_store(__builtin_nontemporal_load(s + i), d + i);
}

__global__ __launch_bounds__(kThreads) void compact_view_kernel(CompactArgs a) {
  const size_t page_bytes = (size_t)a.Hkv * a.D * kPage * a.elem_bytes;
  const long long total = (long long)a.batch * a.capacity;
  for (long long idx = blockIdx.x; idx < total; idx += gridDim.x) {
    const int b = (int)(idx / a.capacity);
    const int j = (int)(idx - (long long)b * a.capacity);
    const int nb = min(a.view_num_blocks[b], a.capacity);
    int dst = -1;
    if (j < nb) {
      const int p = a.view_bt[(size_t)b * a.view_stride + j];
      if (p >= 0 && (int64_t)p < a.src_pages) {
        dst = (int)idx;                                   // b * capacity + j
        copy_block(static_cast<const char *>(a.src_k) + (size_t)p * page_bytes,
                   static_cast<char *>(a.dst_k) + (size_t)dst * page_bytes, page_bytes);
        copy_block(static_cast<const char *>(a.src_v) + (size_t)p * page_bytes,
                   static_cast<char *>(a.dst_v) + (size_t)dst * page_bytes, page_bytes);
        if (a.src_scales && threadIdx.x < 2)
          a.dst_scales[2 * (size_t)dst + threadIdx.x] = a.src_scales[2 * (size_t)p + threadIdx.x];
      }
    }
    if (threadIdx.x == 0) a.compact_bt[idx] = dst;
  }
}

}  // namespace

hipError_t launch_append_kv(const AppendArgs &a, hipStream_t s) {
  const auto addr = reinterpret_cast<uintptr_t>(a.k_new) | reinterpret_cast<uintptr_t>(a.v_new);
  if (addr % 16 != 0) {
    hipLaunchKernelGGL(append_kv_kernel, dim3(a.num_tokens), dim3(kThreads), 0, s, a);
    return hipGetLastError();
  }
  const long long cols = (long long)a.Hkv * a.D * a.elem_bytes / 4;
  dim3 grid((a.num_tokens + kPage - 1) / kPage, 2 * (unsigned)((cols + kThreads - 1) / kThreads));
  while (grid.z < kPage && 2ll * grid.x * grid.y * grid.z <= kAppendWorkgroups) grid.z *= 2;
  switch (a.elem_bytes) {
    case 4: hipLaunchKernelGGL(append_runs_kernel<4>, grid, dim3(kThreads), 0, s, a); break;
    case 2: hipLaunchKernelGGL(append_runs_kernel<2>, grid, dim3(kThreads), 0, s, a); break;
    default: hipLaunchKernelGGL(append_runs_kernel<1>, grid, dim3(kThreads), 0, s, a); break;
  }
  return hipGetLastError();
}

hipError_t launch_compact_view(const CompactArgs &a, int grid, hipStream_t s) {
  hipLaunchKernelGGL(compact_view_kernel, dim3(grid), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

}  // namespace kap
