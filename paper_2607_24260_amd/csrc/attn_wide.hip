// Split-KV attention on the matrix cores for every geometry and dtype the
// tuned kernels do not cover: float32, bf16 or fp8 KV, head_dim 64 / 128 / 256,
// any number G of query heads per KV head, decode views and verify windows.
//
// The q_len window tokens times the G heads of a KV head are R = q_len * G
// query rows over the same keys. A workgroup of four wavefronts owns (key
// split, block of NT 16-row tiles, KV head, sequence); each wavefront walks its
// share of the split one step at a time -- 32 keys (two pages) for 16-bit
// operands, 16 keys (one page) for float32 -- holding all NT tiles:
//   S^T[key][row] = K . Q^T       v_mfma_f32_16x16x32_bf16, or
//   O^T[dim][row] += V^T P^T      v_mfma_f32_16x16x4_f32 for float32 KV
// Lane (j = lane / 16, n = lane % 16) loads exactly the operand pieces it
// multiplies (K: dims 32 kb + 8 j .. + 7 of key n; V^T: keys 4 j .. 4 j + 3 of
// dim 16 dt + n), and the S^T accumulators hold row n, keys 4 j .. 4 j + 3,
// which is the layout P^T needs: nothing goes through LDS until the four
// wavefronts combine.
//
// Weights stay float32: with 16-bit V they are split into three bf16 parts by
// truncation (8 + 8 + 8 bits: exact), one product each; float32 KV multiplies
// in float32.
//
// What bounds it: HBM up to two or three row tiles (8 x 16K, 16-bit, 64-dim
// heads, 10 rows: 268 MB in 47 us, 5.7 TB/s); above that the softmax and the
// split of the weights, about 150 vector instructions per tile and step beside
// 32 matrix instructions; for float32 KV above one tile, the float32 matrix
// rate; for a single short sequence, launch, first loads and the merge (about
// 5 + 4 us). One wavefront per query row with vector dot products, which this
// replaces, read KV q_len * G times: 8 x 16K, 64-dim heads, 5-token windows
// 402 -> 47 us; 8 x 32K views of 15%, 8 heads per KV head 190 -> 20.0 us;
// 4K float32, 5-token window 120 -> 17.7 us.
#include "kap_internal.h"

#include <type_traits>

namespace kap {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = 4;

__device__ __forceinline__ f32x4 mfma16(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma32(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ float xor16_max(float x) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_int(x), __float_as_int(x), false, false);
  return max_f(__int_as_float(r[0]), __int_as_float(r[1]));
}
__device__ __forceinline__ float xor32_max(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_int(x), __float_as_int(x), false, false);
  return max_f(__int_as_float(r[0]), __int_as_float(r[1]));
}
__device__ __forceinline__ float xor16_sum(float x) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_int(x), __float_as_int(x), false, false);
  return __int_as_float(r[0]) + __int_as_float(r[1]);
}
__device__ __forceinline__ float xor32_sum(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_int(x), __float_as_int(x), false, false);
  return __int_as_float(r[0]) + __int_as_float(r[1]);
}

// upper halves (bf16 by truncation) of two floats in one dword
__device__ __forceinline__ uint32_t pack_hi(float lo, float hi) {
  return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
}

// x less its truncation to bf16, the lower (HIGH: upper) half of pair: as one
// dot product where two wavefronts share a SIMD and the vector unit is what
// they wait for (R = 256 rows, fp8: 87 vs 93 us), otherwise with mask and
// subtraction, which start earlier.
template <bool DOT, bool HIGH>
__device__ __forceinline__ float rest(uint32_t pair, float x) {
  if constexpr (DOT) return less_bf16<HIGH>(pair, x);
  else return x - __uint_as_float(__float_as_uint(x) & 0xffff0000u);
}

constexpr int elem_bytes(int kv) { return kv == kF32 ? 4 : (kv == kBF16 ? 2 : 1); }
constexpr int pages_per_step(int kv) { return kv == kF32 ? 1 : 2; }

// Raw registers of one page as loaded (fp8 codes are widened at use).
template <int KV, int D> struct PageData;
template <int D> struct PageData<kBF16, D> { u32x4 k[D / 32]; u32x2 v[D / 16]; };
template <int D> struct PageData<kFP8, D> { u32x2 k[D / 32]; u32x4 v[D / 64]; float2 sc; };
template <int D> struct PageData<kF32, D> { u32x4 k[D / 16]; u32x4 v[D / 16]; };

template <int KV, int D>
struct PageRegs : PageData<KV, D> {
  int page;
  uint32_t vis;   // bit t: token t is visible (before the causal limit); 0: nothing is read
};

// Wavefronts per SIMD the compiler leaves room for: two where a wavefront
// fits 256 registers, so that one multiplies while the other computes weights
// (R = 256 rows, fp8, 4 x 16K: 93 vs 117 us); with head_dim 256 or more than
// two row tiles the second one would spill.
constexpr int wide_waves(int D, int nt) { return D == 256 || nt > 2 ? 1 : 2; }

// Steps in flight per wavefront: as many as 64 registers of raw pages hold, up
// to four (128 registers for the 256-dim one-tile kernels, which have a SIMD to
// themselves). With one, each half of the next step's loads is issued as soon
// as this step has used its registers.
constexpr int ring_depth(int kv, int D, int nt) {
  const int fit = (D == 256 && nt == 1 ? 128 : 64) / wide_step_regs(kv, D);
  return fit < 1 ? 1 : (fit > 4 ? 4 : fit);
}

// The K tile of a page (and its fp8 scales), and the V tile. A page with no
// visible token loads through a zero-byte descriptor: zeros, no traffic.
template <int POLICY, int KV, int D>
__device__ __forceinline__ void load_k(PageRegs<KV, D> &r, const AttnArgs &a, int g, int n, int j) {
  constexpr int kTile = kPage * D * elem_bytes(KV);
  const auto kr = tile_rsrc(a.k_pages, ((size_t)r.page * a.Hkv + g) * kTile, r.vis ? kTile : 0);
#pragma unroll
  for (int kb = 0; kb < D / 32; ++kb) {   // chunk 4 kb + j, token n
    if constexpr (KV == kF32) {
      const int off = (4 * kb + j) * 512 + n * 32;
      r.k[2 * kb] = tile_load16<POLICY>(kr, off);
      r.k[2 * kb + 1] = tile_load16<POLICY>(kr, off + 16);
    } else if constexpr (KV == kBF16) {
      r.k[kb] = tile_load16<POLICY>(kr, (4 * kb + j) * 256 + n * 16);
    } else {
      r.k[kb] = tile_load8<POLICY>(kr, (4 * kb + j) * 128 + n * 8);
    }
  }
  if constexpr (KV == kFP8) r.sc = page_scales(a.kv_scales, r.page, r.vis != 0u);
}
template <int POLICY, int KV, int D>
__device__ __forceinline__ void load_v(PageRegs<KV, D> &r, const AttnArgs &a, int g, int n, int j) {
  constexpr int kTile = kPage * D * elem_bytes(KV);
  const auto vr = tile_rsrc(a.v_pages, ((size_t)r.page * a.Hkv + g) * kTile, r.vis ? kTile : 0);
  if constexpr (KV == kFP8) {
    // whole V^T rows 64 c + lane, rearranged at use (16-byte rows read faster
    // than the 4-byte pieces a lane needs)
#pragma unroll
    for (int c = 0; c < D / 64; ++c) r.v[c] = tile_load16<POLICY>(vr, c * 1024 + (16 * j + n) * 16);
  } else {
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt) {   // dim 16 dt + n, keys 4 j .. 4 j + 3
      if constexpr (KV == kF32)
        r.v[dt] = tile_load16<POLICY>(vr, dt * 1024 + n * 64 + j * 16);
      else
        r.v[dt] = tile_load8<POLICY>(vr, dt * 512 + n * 32 + j * 8);
    }
  }
}

// 4 x 4 dword transpose across the four 16-lane rows: row j holds dword w of
// tile 4 c + j and gets dword j of tiles 4 c .. 4 c + 3.
__device__ __forceinline__ void swap_rows16(uint32_t &a, uint32_t &b) {
  const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}
__device__ __forceinline__ void swap_rows32(uint32_t &a, uint32_t &b) {
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}
__device__ __forceinline__ void transpose_rows(u32x4 x, uint32_t out[4]) {
  uint32_t r0 = x[0], r1 = x[1], r2 = x[2], r3 = x[3];
  swap_rows16(r0, r1);
  swap_rows16(r2, r3);
  swap_rows32(r0, r2);
  swap_rows32(r1, r3);
  out[0] = r0;
  out[1] = r1;
  out[2] = r2;
  out[3] = r3;
}

__device__ __forceinline__ u32x4 widen8(u32x2 x) {   // eight fp8 codes -> bf16
  const u32x2 lo = fp8x4_to_bf16x4(x[0]), hi = fp8x4_to_bf16x4(x[1]);
  return u32x4{lo[0], lo[1], hi[0], hi[1]};
}

// Row index (in q / out / lse) of row r = i * G + h of (b, g).
__device__ __forceinline__ size_t wide_row(const AttnArgs &a, int b, int g, int r) {
  const int i = r / a.G;
  return ((size_t)b * a.q_len + i) * a.Hq + g * a.G + (r - i * a.G);
}

// For the second, careful walk over a step's V (see the kernel): the four bf16
// values of v as finite values (others become 0) and the class of every value
// that is not, as 1.0 where it has it.
__device__ __forceinline__ u32x2 v_finite(u32x2 v) {
#pragma unroll
  for (int w = 0; w < 2; ++w) {
    if ((v[w] & 0x7f80u) == 0x7f80u) v[w] &= 0xffff0000u;
    if ((v[w] & 0x7f800000u) == 0x7f800000u) v[w] &= 0xffffu;
  }
  return v;
}
enum VClass { kPosInf, kNegInf, kNan };
__device__ __forceinline__ bool half_is(uint32_t h, int cls) {
  const bool nan = (h & 0x7fffu) > 0x7f80u;
  return cls == kNan ? nan : h == (cls == kPosInf ? 0x7f80u : 0xff80u);
}
__device__ __forceinline__ u32x2 v_class(u32x2 v, int cls) {
#pragma unroll
  for (int w = 0; w < 2; ++w)
    v[w] = (half_is(v[w] & 0xffffu, cls) ? 0x3f80u : 0u) |
           (half_is(v[w] >> 16, cls) ? 0x3f800000u : 0u);
  return v;
}

// LSE merge of ns partials (slots slot0, slot0 + stride, ..., of RS rows each)
// of a row block: rows row0 .. row0 + rows - 1 of (b, g), kBatch splits' loads in
// flight. float32 calls, whose steps are one page, have the most splits to
// merge, and sixteen at a time pay there (4K, 5-token window 17.8 vs 18.6 us);
// elsewhere the registers they take cost more (8 x 16K, 72 bf16 rows 89.8 vs
// 87.5 us).
template <int D, int ITEMS, int kBatch>
__device__ __forceinline__ void merge_wide(const AttnArgs &a, int b, int g, int row0, int rows,
                                           int RS, int slot0, int stride, int ns) {
  constexpr int D4 = D / 4;
  const auto ro = partial_rsrc(a.part_o);
  const auto rl = partial_rsrc(a.part_lse);
  const int n_items = rows * D4;
  for (int e0 = threadIdx.x; e0 < n_items; e0 += ITEMS * 256) {
    int r[ITEMS], d4[ITEMS];
    float M[ITEMS], tot[ITEMS];
    float4 o[ITEMS];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
      const int e = min(e0 + it * 256, n_items - 1);   // the last item again past the end
      r[it] = e / D4;
      d4[it] = (e % D4) * 4;
      M[it] = -INFINITY;
      tot[it] = 0.f;
      o[it] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    for (int s0 = 0; s0 < ns; s0 += kBatch) {
      float ls[ITEMS][kBatch];
      float4 vs[ITEMS][kBatch];
#pragma unroll
      for (int it = 0; it < ITEMS; ++it)
#pragma unroll
        for (int jj = 0; jj < kBatch; ++jj) {
          const size_t pr = (size_t)(slot0 + stride * min(s0 + jj, ns - 1)) * RS + r[it];
          ls[it][jj] = partial_load1(rl, pr * 4);
          vs[it][jj] = partial_load4(ro, (pr * D + d4[it]) * 4);
        }
#pragma unroll
      for (int it = 0; it < ITEMS; ++it) {
        float mc = M[it];
#pragma unroll
        for (int jj = 0; jj < kBatch; ++jj)
          if (s0 + jj < ns) mc = max_f(mc, ls[it][jj]);
        if (mc == -INFINITY) continue;               // every split so far is empty
        const float sc = exp2f(M[it] - mc);          // 0 while M is still -inf
        tot[it] *= sc;
        if (sc != 0.f) {
          o[it].x *= sc; o[it].y *= sc; o[it].z *= sc; o[it].w *= sc;
        } else {
          o[it] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int jj = 0; jj < kBatch; ++jj) {
          if (s0 + jj >= ns) continue;
          const float w = exp2f(ls[it][jj] - mc);
          if (w == 0.f) continue;                    // whatever the split holds
          tot[it] += w;
          o[it].x = fmaf(w, vs[it][jj].x, o[it].x);
          o[it].y = fmaf(w, vs[it][jj].y, o[it].y);
          o[it].z = fmaf(w, vs[it][jj].z, o[it].z);
          o[it].w = fmaf(w, vs[it][jj].w, o[it].w);
        }
        M[it] = mc;
      }
    }
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
      if (e0 + it * 256 >= n_items) continue;
      const size_t row = wide_row(a, b, g, row0 + r[it]);
      float lse = -INFINITY;
      float4 v = o[it];
      if (M[it] != -INFINITY) {
        const float inv = 1.f / tot[it];
        v.x *= inv; v.y *= inv; v.z *= inv; v.w *= inv;
        lse = (M[it] + log2f(tot[it])) * kLn2;
      }
      *reinterpret_cast<float4 *>(a.out + row * D + d4[it]) = v;
      if (d4[it] == 0) a.lse[row] = lse;
    }
  }
}

template <int KV, int D, int NT, bool SHARED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(wide_waves(D, NT))))
void attn_wide_kernel(AttnArgs a) {
  constexpr int PPS = pages_per_step(KV);
  constexpr int KB = D / 32, DT = D / 16;
  // KV read by one workgroup passes through the caches as a stream; where row
  // blocks share it, it is kept
  constexpr int POLICY = SHARED ? 0 : kNonTemporal;
  constexpr int RING = ring_depth(KV, D, NT);
  constexpr int DC = D < 128 ? D : 128;      // dims combined through LDS at a time
  __shared__ float s_acc[kWaves][16][DC + 4];
  __shared__ float s_m[kWaves][16];
  __shared__ float s_l[kWaves][16];
  __shared__ int s_flag;

  // ---- work item: (sequence, KV head, split) and row block ------------------------
  // The row blocks of a work item read the same keys. Workgroups go to the
  // eight XCDs in turn, so blocks eight workgroups apart run side by side on
  // one XCD, and all but the first read KV from its L2.
  const int rb = blockIdx.x >> 3;
  const unsigned item = (blockIdx.z * gridDim.y + blockIdx.y) * 8u + (blockIdx.x & 7);
  WorkItem wi;
  int L;
  auto entries = [&](int bb, int Lb) {   // pages of sequence bb
    const int np = Lb > 0 ? (int)(((long long)Lb + kPage - 1) / kPage) : 0;
    return max(0, min(a.num_blocks ? a.num_blocks[bb] : np, a.max_blocks));
  };
  if (a.ragged) {
    auto load = [&](int bb) {
      const int Lb = a.seq_lens[bb];
      return SeqLoad{(entries(bb, Lb) + PPS - 1) / PPS, Lb};
    };
    int steps_b;
    const SeqLoad first = map_first_loads(a, load);
    if (!ragged_map(a, load, first, (int)item, wi, steps_b, L)) return;
  } else {
    // splits of all (sequence, KV head) pairs in turn: the ones that a short
    // sequence leaves empty are not all on the same XCDs
    const unsigned units = (unsigned)a.batch * (unsigned)a.Hkv;
    const unsigned split_i = item / units, u = item - split_i * units;
    wi.n_split = a.n_split;
    wi.split = (int)split_i;
    wi.b = (int)(u / (unsigned)a.Hkv);
    wi.g = (int)(u - (unsigned)wi.b * a.Hkv);
    wi.slot0 = (int)(u * a.n_split);
    if (wi.split >= a.n_split) return;
    L = a.seq_lens[wi.b];
    if (a.min_chunk > 0) {
      const int steps_b = (entries(wi.b, L) + PPS - 1) / PPS;
      wi.n_split = max(1, min(a.n_split, (steps_b + a.min_chunk - 1) / a.min_chunk));
      if (wi.split >= wi.n_split) return;
    }
  }
  // the same in every lane: keep it in scalar registers
  const int split = __builtin_amdgcn_readfirstlane(wi.split);
  const int g = __builtin_amdgcn_readfirstlane(wi.g);
  const int b = __builtin_amdgcn_readfirstlane(wi.b);
  const int n_split = __builtin_amdgcn_readfirstlane(wi.n_split);
  const int slot0 = __builtin_amdgcn_readfirstlane(wi.slot0);
  const int RB = a.row_blocks;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int n = lane & 15, j = lane >> 4;
  const int R = a.q_len * a.G;
  const int row0 = rb * (16 * NT);
  const int rows = min(R - row0, 16 * NT);   // rows of this block, >= 1
  const int RS = min(R, 16 * NT);            // rows a partial slot holds

  const int np = __builtin_amdgcn_readfirstlane(entries(b, L));
  const int steps = (np + PPS - 1) / PPS;
  const int q0 = (int)(((long long)split * steps) / n_split);
  const int q1 = (int)(((long long)(split + 1) * steps) / n_split);

  // ---- Q^T operand: row n of each tile, dims 32 kb + 8 j .. + 7 -------------------
  // In registers, or (64 of them per lane and more: the kernel would spill) in
  // LDS, where the four wavefronts share it.
  constexpr int QN = KB * (KV == kF32 ? 2 : 1);   // 16-byte pieces of a tile
  constexpr bool kQInLds = NT * QN >= 16;
  __shared__ __attribute__((aligned(16))) u32x4 s_q[kQInLds ? NT * QN : 1][64];
  u32x4 qreg[kQInLds ? 1 : NT * QN];
  int lim[NT];                               // causal: row sees logical positions < lim
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int r = row0 + nt * 16 + n;
    const bool in = r < R;
    const int i = (in ? r : 0) / a.G;
    lim[nt] = in ? (a.causal ? L - a.q_len + i + 1 : L) : 0;
    // rows past the end read row 0; nothing of them is kept
    const size_t q0d = wide_row(a, b, g, in ? r : 0) * D + j * 8;
#pragma unroll
    for (int x = 0; x < QN; ++x) {
      if (kQInLds && x % kWaves != wave) continue;
      u32x4 v;
      if constexpr (KV == kF32)
        v = *reinterpret_cast<const u32x4 *>(static_cast<const float *>(a.q) + q0d +
                                             (x / 2) * 32 + (x % 2) * 4);
      else
        v = *reinterpret_cast<const u32x4 *>(static_cast<const uint16_t *>(a.q) + q0d + x * 32);
      if constexpr (kQInLds) s_q[nt * QN + x][lane] = v;
      else qreg[nt * QN + x] = v;
    }
  }
  if constexpr (kQInLds) __syncthreads();
  auto qop = [&](int nt, int x, int at) {
    if constexpr (kQInLds) return s_q[nt * QN + x][at];
    else return qreg[nt * QN + x];
  };
  // pages below this are visible to every row of the window
  const int first_masked = a.causal ? max(0, L - a.q_len + 1) / kPage : 0x7fffffff;

  float m[NT], l[NT];
  f32x4 acc[NT][DT];
  auto reset = [&] {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      m[nt] = kNoMax;
      l[nt] = 0.f;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) acc[nt][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  };
  reset();

  struct Step { PageRegs<KV, D> p[PPS]; };

  // page id and visible tokens of an entry (see decode: an invalid id, or a
  // block past the sequence, has none)
  // (In scalar registers throughout: a 64-bit comparison runs on the vector unit
  // -- in every step: 2 x 32K 64-dim bf16, one split 188 vs 167 us, and the
  // registers of the 256-dim two-tile kernels ran out --, and of table entries
  // that vector loads read, the compiler does not use that they are uniform: it
  // looped over the lanes around the first page loads, 700 tokens 9.6 vs 9.1 us)
  const uint32_t page_limit = (uint32_t)(a.num_pages < 0x80000000ll ? a.num_pages : 0x80000000ll);
  auto set_page = [&](PageRegs<KV, D> &r, bool live, int page, int lblk, uint32_t mask) {
    const int nvalid = lblk < (L >> 4) ? kPage : (lblk == (L >> 4) ? L & (kPage - 1) : 0);
    const bool ok = live && (uint32_t)page < page_limit;
    r.vis = ok ? (0xFFFFu >> (kPage - nvalid)) & mask : 0u;
    r.page = ok ? page : 0;
  };

  // One step: pages k .. k + PPS - 1 of the sequence's list. next_k / next_v
  // issue the loads of a later step into the registers that are free by then.
  auto process = [&](Step &S, int k, auto careful, auto &&next_k, auto &&next_v) {
    constexpr bool CAREFUL = decltype(careful)::value;
    uint32_t vis[PPS];
    float ksc[PPS], vsc[PPS];
    bool all = true;
#pragma unroll
    for (int x = 0; x < PPS; ++x) {
      vis[x] = S.p[x].vis;
      all = all && vis[x] == 0xFFFFu;
      ksc[x] = a.scale_log2;
      vsc[x] = 1.f;
      if constexpr (KV == kFP8) {
        ksc[x] *= S.p[x].sc.x;
        vsc[x] = S.p[x].sc.y;
      }
    }
    // ---- S^T = K Q^T ---------------------------------------------------------------
    int q_at = lane;   // opaque, or Q would be read once and held in registers after all
    if constexpr (kQInLds) asm volatile("" : "+v"(q_at));
    // (float32: two sums over alternate k-blocks, added at the end -- shorter
    // chains of rounding)
    constexpr int SUMS = KV == kF32 ? 2 : 1;
    f32x4 s[PPS][NT], s_odd[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
      for (int x = 0; x < PPS; ++x) s[x][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
      s_odd[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
#pragma unroll
      for (int x = 0; x < PPS; ++x) {
        if constexpr (KV == kF32) {
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            u32x4 qv[NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) qv[nt] = qop(nt, 2 * kb + e / 4, q_at);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
              f32x4 &sum = kb % SUMS ? s_odd[nt] : s[x][nt];
              sum = mfma32(__uint_as_float(S.p[x].k[2 * kb + e / 4][e % 4]),
                           __uint_as_float(qv[nt][e % 4]), sum);
            }
          }
        } else {
          u32x4 kop;
          if constexpr (KV == kFP8) kop = widen8(S.p[x].k[kb]);
          else kop = S.p[x].k[kb];
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) s[x][nt] = mfma16(kop, qop(nt, kb, q_at), s[x][nt]);
        }
      }
    }
    if constexpr (SUMS == 2)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) s[0][nt] += s_odd[nt];
    // V as it will be multiplied, taken out of the raw registers; values of
    // hidden tokens become zeros, so that zero weights meet zeros
    using VPiece = typename std::conditional<
        KV == kF32, u32x4, typename std::conditional<KV == kBF16, u32x2, uint32_t>::type>::type;
    VPiece v[PPS][DT];
    auto take_v = [&] {
#pragma unroll
      for (int x = 0; x < PPS; ++x) {
        if constexpr (KV == kFP8) {
#pragma unroll
          for (int c = 0; c < D / 64; ++c) transpose_rows(S.p[x].v[c], &v[x][4 * c]);
        } else {
#pragma unroll
          for (int dt = 0; dt < DT; ++dt) v[x][dt] = S.p[x].v[dt];
        }
        if (vis[x] != 0xFFFFu) {
          const uint32_t my = vis[x] >> (4 * j);
          if constexpr (KV == kF32) {
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
              for (int e = 0; e < 4; ++e) v[x][dt][e] = (my >> e) & 1u ? v[x][dt][e] : 0u;
          } else if constexpr (KV == kBF16) {
            const uint32_t m0 = (my & 1u ? 0xffffu : 0u) | (my & 2u ? 0xffff0000u : 0u);
            const uint32_t m1 = (my & 4u ? 0xffffu : 0u) | (my & 8u ? 0xffff0000u : 0u);
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
              v[x][dt][0] &= m0;
              v[x][dt][1] &= m1;
            }
          } else {
            const uint32_t mk = (my & 1u ? 0xffu : 0u) | (my & 2u ? 0xff00u : 0u) |
                                (my & 4u ? 0xff0000u : 0u) | (my & 8u ? 0xff000000u : 0u);
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) v[x][dt] &= mk;
          }
        }
      }
    };
    next_k();

    // ---- online softmax --------------------------------------------------------------
    const bool needs_mask = !all || k + PPS > first_masked;
    // (the page scales are the same in every lane: their signs are scalar)
    int signs = 0;
#pragma unroll
    for (int x = 0; x < PPS; ++x)
      signs |= __builtin_amdgcn_readfirstlane(__float_as_int(ksc[x]));
    const bool scaled = needs_mask || signs < 0;
    float p[NT][4 * PPS];                       // weights x V scale
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      // Logits z * kz: the sums themselves with the pages' scales, or (masked
      // pages, negative scales) the scaled and masked logits with 1. Scaling
      // by kz >= 0 keeps the order, so only the maxima are scaled here, and
      // the weights' exponents below are one fused multiply-add each.
      float z[4 * PPS], kz[PPS];
#pragma unroll
      for (int x = 0; x < PPS; ++x) {
        kz[x] = ksc[x];
#pragma unroll
        for (int e = 0; e < 4; ++e) z[4 * x + e] = s[x][nt][e];
      }
      if (scaled) {
#pragma unroll
        for (int x = 0; x < PPS; ++x) {
          kz[x] = 1.f;
          const int below = a.causal ? lim[nt] - (k + x) * kPage : kPage;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            z[4 * x + e] *= ksc[x];
            if (needs_mask &&
                (!((vis[x] >> (4 * j + e)) & 1u) || 4 * j + e >= below)) z[4 * x + e] = -INFINITY;
          }
        }
      }
      float own = -INFINITY;
#pragma unroll
      for (int x = 0; x < PPS; ++x) {
        float my = z[4 * x];
#pragma unroll
        for (int e = 1; e < 4; ++e) my = max_f(my, z[4 * x + e]);
        own = max_f(own, my * kz[x]);
      }
      if (__any(own > m[nt] + (CAREFUL ? 0.f : kDefer))) {
        float mx = xor16_max(own);
        mx = xor32_max(mx);
        if (mx > m[nt]) {
          const float alpha = exp2_fast(m[nt] - mx);
          l[nt] *= alpha;
#pragma unroll
          for (int dt = 0; dt < DT; ++dt) {
            if (CAREFUL && alpha == 0.f) acc[nt][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
            else acc[nt][dt] *= alpha;
          }
          m[nt] = mx;
        }
      }
      if constexpr (CAREFUL) asm("" : "+v"(m[nt]));   // one register, not a copy for later
      const float mref = m[nt];
      float ps = 0.f;
#pragma unroll
      for (int e = 0; e < 4 * PPS; ++e) {
        p[nt][e] = exp2_fast(fmaf(z[e], kz[e / 4], -mref));
        ps += p[nt][e];
      }
      l[nt] += ps;
      if constexpr (KV == kFP8) {
#pragma unroll
        for (int e = 0; e < 4 * PPS; ++e)
          p[nt][e] = CAREFUL && p[nt][e] == 0.f ? 0.f : p[nt][e] * vsc[e / 4];
      }
    }
    take_v();
    if constexpr (KV == kFP8) next_v();

    // ---- O^T += V^T P^T ----------------------------------------------------------------
    if constexpr (KV == kF32) {
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          if constexpr (!CAREFUL) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              acc[nt][dt] = mfma32(__uint_as_float(v[0][dt][e]), p[nt][e], acc[nt][dt]);
          } else {
            f32x4 kind[3] = {};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float x = __uint_as_float(v[0][dt][e]);
              const bool fin = __builtin_isfinite(x);
              const float one = p[nt][e] != 0.f ? 1.f : 0.f;
              acc[nt][dt] = mfma32(fin ? x : 0.f, p[nt][e], acc[nt][dt]);
              kind[kPosInf] = mfma32(x == INFINITY ? 1.f : 0.f, one, kind[kPosInf]);
              kind[kNegInf] = mfma32(x == -INFINITY ? 1.f : 0.f, one, kind[kNegInf]);
              kind[kNan] = mfma32(x != x ? 1.f : 0.f, one, kind[kNan]);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              if (kind[kPosInf][e] > 0.f) acc[nt][dt][e] += INFINITY;
              if (kind[kNegInf][e] > 0.f) acc[nt][dt][e] -= INFINITY;
              if (kind[kNan][e] > 0.f) acc[nt][dt][e] = __builtin_nanf("");
            }
          }
        }
    } else {
      constexpr bool kDot = wide_waves(D, NT) == 2;
      u32x4 hi[NT], mid[NT], lo[NT], one[CAREFUL ? NT : 1];
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const float p0 = p[nt][2 * w], p1 = p[nt][2 * w + 1];
          hi[nt][w] = pack_hi(p0, p1);
          const float r0 = rest<kDot, false>(hi[nt][w], p0), r1 = rest<kDot, true>(hi[nt][w], p1);
          mid[nt][w] = pack_hi(r0, r1);
          lo[nt][w] = pack_hi(rest<kDot, false>(mid[nt][w], r0), rest<kDot, true>(mid[nt][w], r1));
          if constexpr (CAREFUL)
            one[nt][w] = (p0 != 0.f ? 0x3f80u : 0u) | (p1 != 0.f ? 0x3f800000u : 0u);
        }
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        u32x2 va, vb;
        if constexpr (KV == kFP8) {
          va = fp8x4_to_bf16x4(v[0][dt]);
          vb = fp8x4_to_bf16x4(v[PPS - 1][dt]);
        } else {
          va = v[0][dt];
          vb = v[PPS - 1][dt];
        }
        if constexpr (!CAREFUL) {
          const u32x4 vop = u32x4{va[0], va[1], vb[0], vb[1]};
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) acc[nt][dt] = mfma16(vop, lo[nt], acc[nt][dt]);
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) acc[nt][dt] = mfma16(vop, mid[nt], acc[nt][dt]);
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) acc[nt][dt] = mfma16(vop, hi[nt], acc[nt][dt]);
        } else {
          const u32x2 fa = v_finite(va), fb = v_finite(vb);
          const u32x4 vop = u32x4{fa[0], fa[1], fb[0], fb[1]};
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) {
            acc[nt][dt] = mfma16(vop, lo[nt], acc[nt][dt]);
            acc[nt][dt] = mfma16(vop, mid[nt], acc[nt][dt]);
            acc[nt][dt] = mfma16(vop, hi[nt], acc[nt][dt]);
            f32x4 kind[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
              const u32x2 ca = v_class(va, c), cb = v_class(vb, c);
              kind[c] = mfma16(u32x4{ca[0], ca[1], cb[0], cb[1]}, one[nt],
                               f32x4{0.f, 0.f, 0.f, 0.f});
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              if (kind[kPosInf][e] > 0.f) acc[nt][dt][e] += INFINITY;
              if (kind[kNegInf][e] > 0.f) acc[nt][dt][e] -= INFINITY;
              if (kind[kNan][e] > 0.f) acc[nt][dt][e] = __builtin_nanf("");
            }
          }
        }
      }
    }
    if constexpr (KV != kFP8) next_v();
  };

  // ---- walk: the split's steps, round-robin over the four wavefronts ---------------
  const int qw = q0 + wave;
  const int n_my = qw < q1 ? (q1 - qw + kWaves - 1) / kWaves : 0;
  const int32_t *tbt = a.block_table + (size_t)b * a.bt_stride;
  const int32_t *tlb = a.logical_block ? a.logical_block + (size_t)b * a.bt_stride : nullptr;
  const uint32_t *tmk = a.token_mask ? a.token_mask + (size_t)b * a.bt_stride : nullptr;
  if (n_my > 0) {
    auto kstep = [&](int i) { return PPS * (qw + kWaves * min(i, n_my - 1)); };
    // the entries of step i, read directly (entries past np are not read)
    auto direct = [&](Step &S, int i) {
      const int k = kstep(i);
#pragma unroll
      for (int x = 0; x < PPS; ++x) {
        const int kk = min(k + x, np - 1);
        set_page(S.p[x], i < n_my && k + x < np, __builtin_amdgcn_readfirstlane(tbt[kk]),
                 tlb ? __builtin_amdgcn_readfirstlane(tlb[kk]) : k + x,
                 tmk ? __builtin_amdgcn_readfirstlane(tmk[kk]) : 0xFFFFu);
      }
    };
    auto load_all = [&](Step &S) {
#pragma unroll
      for (int x = 0; x < PPS; ++x) {
        load_k<POLICY>(S.p[x], a, g, n, j);
        load_v<POLICY>(S.p[x], a, g, n, j);
      }
    };
    // ... and a round ahead through the vector memory pipe (lane x & 1: entry
    // k + x; reads past the row's np entries return 0)
    const auto rbt = table_rsrc(tbt, np);
    const auto rlb = table_rsrc(tlb ? tlb : tbt, np);
    const auto rmk = table_rsrc(tmk ? reinterpret_cast<const int32_t *>(tmk) : tbt, np);
    const int voff = opaque_zero() + (lane & 1) * 4;
    struct Ahead { int bt, lb, mk; };
    auto issue = [&](Ahead &h, int i) {
      const int k = kstep(i);
      h.bt = table_ahead(rbt, voff, k);
      if (tlb) h.lb = table_ahead(rlb, voff, k);
      if (tmk) h.mk = table_ahead(rmk, voff, k);
    };
    auto use = [&](Step &S, const Ahead &h, int i) {
      const int k = kstep(i);
#pragma unroll
      for (int x = 0; x < PPS; ++x)
        set_page(S.p[x], i < n_my && k + x < np, lane_value(h.bt, x),
                 tlb ? lane_value(h.lb, x) : k + x,
                 tmk ? (uint32_t)lane_value(h.mk, x) : 0xFFFFu);
    };
    auto none = [] {};
    Step st[RING];
    Ahead ahead[RING] = {};
#pragma unroll
    for (int jr = 0; jr < RING; ++jr) {
      direct(st[jr], jr);
      load_all(st[jr]);
      __builtin_amdgcn_sched_barrier(0);
      issue(ahead[jr], jr + RING);
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (RING == 1) {
      for (int i = 0; i < n_my; ++i) {
        Step nx;   // page ids and visibility of the next step
        use(nx, ahead[0], i + 1);
        process(
            st[0], kstep(i), std::false_type{},
            [&] {
#pragma unroll
              for (int x = 0; x < PPS; ++x) {
                st[0].p[x].page = nx.p[x].page;
                st[0].p[x].vis = nx.p[x].vis;
                load_k<POLICY>(st[0].p[x], a, g, n, j);
              }
            },
            [&] {
#pragma unroll
              for (int x = 0; x < PPS; ++x) load_v<POLICY>(st[0].p[x], a, g, n, j);
              issue(ahead[0], i + 2);
            });
      }
    } else {
      // every round issues its loads unconditionally (past the end through
      // empty descriptors), so the loop waits only for the oldest step
      for (int i = 0; i < n_my; i += RING) {
#pragma unroll
        for (int jr = 0; jr < RING; ++jr) {
          if (i + jr < n_my) process(st[jr], kstep(i + jr), std::false_type{}, none, none);
          use(st[jr], ahead[jr], i + jr + RING);
          load_all(st[jr]);
          issue(ahead[jr], i + jr + 2 * RING);
        }
      }
    }
    // A weight of zero contributes nothing, whatever V holds; a matrix
    // product gives 0 * inf = NaN there (hidden tokens' V is cleared above,
    // but rows of a window see different keys, and a weight or one of its
    // parts can be zero on its own). Rather than test V on the way, a
    // wavefront whose result is not finite (or large, see kLargeSum) walks its
    // share again, with weights of at most 1, keeping infinities and NaNs of V
    // out of the products and adding them by class where the weight is not
    // zero.
    float t = 0.f;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) t = max_abs(t, acc[nt][dt]);
    if (__any(!(t < kLargeSum))) {
      reset();
      for (int i = 0; i < n_my; ++i) {
        direct(st[0], i);
        load_all(st[0]);
        process(st[0], kstep(i), std::true_type{}, none, none);
      }
    }
  }

  // ---- combine the four wavefronts, tile by tile, then write ----------------------
  constexpr int PER = DC / 16;                // dims of one thread
  const auto ro = partial_rsrc(a.part_o);
  const auto rl = partial_rsrc(a.part_lse);
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    float lt = xor16_sum(l[nt]);
    lt = xor32_sum(lt);
#pragma unroll
    for (int c = 0; c < D / DC; ++c) {
      if (nt + c > 0) __syncthreads();        // s_acc, s_m, s_l are read above
#pragma unroll
      for (int dt = 0; dt < DC / 16; ++dt)
        *reinterpret_cast<f32x4 *>(&s_acc[wave][n][dt * 16 + 4 * j]) =
            acc[nt][c * (DC / 16) + dt];
      if (j == 0) {
        // no key seen; a NaN logit, which never moves the reference and must not
        // be dropped as a weight of zero against it; or the reference
        s_m[wave][n] = lt == 0.f ? -INFINITY : (lt != lt ? lt : m[nt]);
        s_l[wave][n] = lt;
      }
      __syncthreads();
      // thread (rn, d0) combines row rn's dims c * DC + d0 .. + PER - 1
      const int rn = threadIdx.x >> 4;
      const int d0 = (threadIdx.x & 15) * PER;
      const int r = nt * 16 + rn;             // row of the block
      if (r < rows) {
        float o[PER];
#pragma unroll
        for (int e = 0; e < PER; ++e) o[e] = 0.f;
        float lse2 = -INFINITY;
        float M = s_m[0][rn];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) M = max_f(M, s_m[w][rn]);
        if (M != -INFINITY) {
          float den = 0.f;
#pragma unroll
          for (int w = 0; w < kWaves; ++w) {
            const float ew = exp2f(s_m[w][rn] - M);
            if (ew == 0.f) continue;          // whatever that wavefront holds
            den = fmaf(ew, s_l[w][rn], den);
#pragma unroll
            for (int e = 0; e < PER; ++e) o[e] = fmaf(ew, s_acc[w][rn][d0 + e], o[e]);
          }
          const float inv = 1.f / den;
#pragma unroll
          for (int e = 0; e < PER; ++e) o[e] *= inv;
          lse2 = M + log2f(den);
        }
        const int d = c * DC + d0;
        const bool first = d == 0;
        if (n_split == 1) {
          const size_t row = wide_row(a, b, g, row0 + r);
#pragma unroll
          for (int e = 0; e < PER; e += 4)
            *reinterpret_cast<float4 *>(a.out + row * D + d + e) =
                make_float4(o[e], o[e + 1], o[e + 2], o[e + 3]);
          if (first) a.lse[row] = lse2 * kLn2;
        } else {
          const size_t pr = (size_t)((slot0 + split) * RB + rb) * RS + r;
#pragma unroll
          for (int e = 0; e < PER; e += 4)
            partial_store4(ro, (pr * D + d + e) * 4,
                           make_float4(o[e], o[e + 1], o[e + 2], o[e + 3]));
          if (first) partial_store1(rl, pr * 4, lse2);
        }
      }
    }
  }

  // ---- the last workgroup merges the splits ------------------------------------------
  // (b, g) has one 64-byte block of 16 counters; row blocks rb, rb + 16, ...
  // share counter rb % 16, and the last arrival over all of them merges them.
  if (n_split > 1) {
    const int c = rb & (kTicketStride - 1);
    const int sharing = (RB - c + kTicketStride - 1) / kTicketStride;
    if (last_arrival_of(a.tickets + ((size_t)b * a.Hkv + g) * kTicketStride + c,
                        n_split * sharing, &s_flag)) {
      for (int x = c; x < RB; x += kTicketStride)
        merge_wide<D, (NT > 1 ? 2 : 1), (KV == kF32 ? 16 : 8)>(
            a, b, g, x * (16 * NT), min(R - x * (16 * NT), 16 * NT), RS, slot0 * RB + x, RB,
            n_split);
    }
  }
}

template <int KV, int D, int NT, bool SHARED>
hipError_t launch(const AttnArgs &a, hipStream_t s) {
  // eight work items per row of workgroups, each with its row blocks (the
  // rows fill y and, past its limit, z)
  const long long items = a.ragged ? a.n_split : (long long)a.batch * a.Hkv * a.n_split;
  const long long groups = (items + 7) / 8;
  const unsigned gy = (unsigned)(groups < 32768 ? groups : 32768);
  const dim3 grid(8 * a.row_blocks, gy, (unsigned)((groups + gy - 1) / gy));
  hipLaunchKernelGGL((attn_wide_kernel<KV, D, NT, SHARED>), grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

template <int KV, int D, int NT>
hipError_t launch_nt(const AttnArgs &a, hipStream_t s) {
  // several row blocks always have more than half of the most tiles each
  constexpr int kMax = wide_max_tiles(KV, D);
  if (a.row_blocks == 1) return launch<KV, D, NT, false>(a, s);
  if constexpr (2 * NT > kMax) return launch<KV, D, NT, true>(a, s);
  return hipErrorInvalidValue;
}

template <int KV, int D>
hipError_t launch_d(const AttnArgs &a, hipStream_t s) {
  constexpr int kMax = wide_max_tiles(KV, D);
  switch (a.row_tiles) {
    case 1: return launch_nt<KV, D, 1>(a, s);
    case 2: if constexpr (kMax >= 2) return launch_nt<KV, D, 2>(a, s); break;
    case 3: if constexpr (kMax >= 3) return launch_nt<KV, D, 3>(a, s); break;
    case 4: if constexpr (kMax >= 4) return launch_nt<KV, D, 4>(a, s); break;
    default: break;
  }
  return hipErrorInvalidValue;
}

template <int KV>
hipError_t launch_kv(const AttnArgs &a, hipStream_t s) {
  switch (a.D) {
    case 64: return launch_d<KV, 64>(a, s);
    case 128: return launch_d<KV, 128>(a, s);
    case 256: return launch_d<KV, 256>(a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_attn_wide(const AttnArgs &a, hipStream_t s) {
  switch (a.kv_type) {
    case kF32: return launch_kv<kF32>(a, s);
    case kBF16: return launch_kv<kBF16>(a, s);
    case kFP8: return launch_kv<kFP8>(a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace kap
