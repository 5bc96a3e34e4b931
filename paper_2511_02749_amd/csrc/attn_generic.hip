// Span attention on fp32 pools for gfx950, any number of query heads per kv head, on fp32
// matrix instructions (v_mfma_f32_16x16x4_f32).  On bf16 pools too, each element widened as it
// is loaded: for plans whose work lists for the split-precision kernel, which is twice as fast
// (attn_split.hip), do not fit the memory they must go to.
//
// One work-group of four waves per (32 rows of a row tile, query head); the planner's row
// tiles hold up to 64 rows, two items.  Every wave holds all 32 rows, as two 16-row blocks
// that share each K and V operand, and takes a quarter of the key pages, so that a short tile
// over a long key list is not one wave's serial chain and no page is read twice.  The four
// partial softmaxes of a row meet in LDS at the end.
//
// Layouts (lane l, r = l % 16, g = l / 16).  A key page has 16 keys.
//   scores  S^T = K Q^T, A = K[16 keys][4 dims] (key r, one dim per g), B = Q^T[4 dims]
//           [16 rows] (row r).  Lane group g stands for dims 16t + 4g .. + 3 in the four
//           steps of t, so K and Q are read 16 bytes at a time.  C: keys 4g .. 4g + 3 of
//           row r.
//   output  O^T = V^T P^T, step j contracts keys 4g + j: B = P^T is the C layout of the
//           scores as it is, A = V^T[16 dims][4 keys] is element j of slots 4g .. 4g + 3
//           of a dim's row, 16 contiguous bytes of the page.  C: dims 4g .. 4g + 3 of
//           each 16-dim block, row r.
//
// Repositioned keys (delta != 0) are read as stored; the query is rotated to its
// position less the key's delta instead, from its raw row and the exact table entry, so
// one fp32 rotation separates it from the caller's value whatever the delta.
//
// K and V go from memory to registers without LDS: 16 bytes per lane and D / 16 loads each
// for a page, all whole 64-byte segments.  A page is D MFMAs of 32 cycles per wave, so the V
// loads, issued before the scores, and the K loads of the next page, issued after them,
// have half a page of matrix work of each of the SIMD's two waves to land in.
//
// Bound: the fp32 matrix rate (256 flop per clock and CU; an MFMA-only loop of this
// instruction reaches 154 TFLOP/s).  8 query over 2 kv heads at head dim 128, prefix 256
// and 8 fragments of about 500 (7.2 GFLOP): 3.5 ms with vector arithmetic, one wave per 64
// rows, keys broadcast from LDS; 141 us with eight waves of 16 rows per 64-row tile; 112 us
// with four; 107 us with both row blocks in every wave; 97 us with one block's softmax
// under the other's MFMAs (74 TFLOP/s).  A timing copy that read one page throughout, and
// one that never rescaled, took the same time to 3%: the rest is item starts and ends and
// the waves of a SIMD reaching their vector phases together.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <type_traits>

#include "../../include/spanq.h"
#include "dev_common.h"
#include "grid.h"
#include "kernels.h"
#include "mfma_common.h"

namespace spanq {

namespace {

using namespace mfma;

constexpr int kGW = 4;  // waves per work-group
constexpr int kRB = 2;                 // 16-row blocks per wave
constexpr int kItemRows = 16 * kRB;    // rows per work-group
constexpr int kItemsPerTile = kGenericBM / kItemRows;

// Four consecutive elements of a caller's row, whose base is only known to be aligned to
// an element.
typedef float row4_t __attribute__((ext_vector_type(4), aligned(4)));
typedef bf16_t row4h_t __attribute__((ext_vector_type(4), aligned(2)));
__device__ __forceinline__ row4_t load_row4(const float* p) { return *reinterpret_cast<const row4_t*>(p); }
__device__ __forceinline__ row4_t load_row4(const bf16_t* p) {
  const row4h_t v = *reinterpret_cast<const row4h_t*>(p);
  return row4_t{to_f32(v[0]), to_f32(v[1]), to_f32(v[2]), to_f32(v[3])};
}
__device__ __forceinline__ void store_row4(float* p, const row4_t& w) { *reinterpret_cast<row4_t*>(p) = w; }
__device__ __forceinline__ void store_row4(bf16_t* p, const row4_t& w) {
  *reinterpret_cast<row4h_t*>(p) = row4h_t{f32_to_bf16(w[0]), f32_to_bf16(w[1]), f32_to_bf16(w[2]), f32_to_bf16(w[3])};
}
// The same of a page (aligned to four elements), and of a partial.
__device__ __forceinline__ f32x4_t load_page4(const float* p) { return *reinterpret_cast<const f32x4_t*>(p); }
__device__ __forceinline__ f32x4_t load_page4(const bf16_t* p) {
  const uint2 v = *reinterpret_cast<const uint2*>(p);
  return f32x4_t{lo_bf16(v.x), hi_bf16(v.x), lo_bf16(v.y), hi_bf16(v.y)};
}
__device__ __forceinline__ void store_part4(float* p, const f32x4_t& w) { *reinterpret_cast<f32x4_t*>(p) = w; }
__device__ __forceinline__ void store_part4(f16_t* p, const f32x4_t& w) {
  *reinterpret_cast<f16x4_t*>(p) =
      f16x4_t{static_cast<f16_t>(w[0]), static_cast<f16_t>(w[1]), static_cast<f16_t>(w[2]), static_cast<f16_t>(w[3])};
}

template <int D>
struct GGeo {
  static constexpr int OROW = D + 4;  // floats per row of a wave's merged O (padded against bank conflicts)
  static constexpr int LDS = kGW * kItemRows * (OROW + 2) * 4;
};

template <typename T, int D>
__global__ __launch_bounds__(64 * kGW) __attribute__((amdgpu_waves_per_eu(2))) void attn_generic_kernel(
    const WorkTile* __restrict__ tiles, const KvPage* __restrict__ kv, const T* __restrict__ q, T* __restrict__ out,
    const T* __restrict__ pool, int64_t layer_off, int hq, int hkv, float scale_log2, const float2* __restrict__ rope,
    bool runs, typename PartOf<T>::type* __restrict__ part_o, float* __restrict__ part_ml) {
  constexpr int H = D / 2;
  constexpr int NT = D / 16;  // 16-dim steps of the scores, 16-dim blocks of the output
  constexpr int OROW = GGeo<D>::OROW;
  extern __shared__ __attribute__((aligned(16))) float smem[];
  float* const sh_o = smem;                       // [wave][row][OROW]
  float* const sh_m = smem + kGW * kItemRows * OROW;  // [wave][row]
  float* const sh_l = sh_m + kGW * kItemRows;

  const int h = blockIdx.x % hq;
  const int part_of_tile = blockIdx.x / hq;
  WorkTile t = tiles[part_of_tile / kItemsPerTile];
  const int row0 = kItemRows * (kItemsPerTile - 1 - part_of_tile % kItemsPerTile);  // longer lists first
  if (row0 >= t.n_rows) return;
  t.q_row0 += row0;
  t.q_pos0 += row0;
  t.n_rows = min(t.n_rows - row0, kItemRows);
  const int kvh = (h * hkv) / hq;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int r = lane & 15, g = lane >> 4;
  const bool two = t.n_rows > 16;  // both row blocks hold rows
  const int last_pos = t.q_pos0 + t.n_rows - 1;
  const int64_t page_elems = 2ll * hkv * kPage * D;
  const T* const kbase = pool + layer_off + static_cast<int64_t>(kvh) * kPage * D + r * D + 4 * g;
  // slots 4g .. 4g + 3 are quad (g & 1) << 1 | g >> 1 of a V row
  const T* const vbase = pool + layer_off + static_cast<int64_t>(hkv + kvh) * kPage * D + r * kPage +
                         4 * (((g & 1) << 1) | (g >> 1));

  f32x4_t o[kRB][NT];
  float qv[kRB][NT][4];
  float m[kRB], l[kRB];  // l: this lane's keys only
#pragma unroll
  for (int x = 0; x < kRB; ++x) {
    m[x] = -INFINITY;
    l[x] = 0.f;
#pragma unroll
    for (int b = 0; b < NT; ++b) o[x][b] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  }
  int q_delta = -1;

  f32x4_t kr[NT], vr[NT];
  auto load_k = [&](int pid) {
    const T* p = kbase + static_cast<int64_t>(pid) * page_elems;
#pragma unroll
    for (int b = 0; b < NT; ++b) kr[b] = load_page4(p + 16 * b);
  };
  auto load_v = [&](int pid) {
    const T* p = vbase + static_cast<int64_t>(pid) * page_elems;
#pragma unroll
    for (int b = 0; b < NT; ++b) vr[b] = load_page4(p + 16 * b * kPage);
  };
  // qv <- R(position - delta) q; positions below the table's start do not occur (a key's
  // stored position is its final one less delta, and no row reads past its own position)
  auto load_q = [&](int x, int delta) {
    const int row = 16 * x + r;
    if (row >= t.n_rows) {
#pragma unroll
      for (int b = 0; b < NT; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) qv[x][b][i] = 0.f;
      return;
    }
    const T* src = q + (static_cast<int64_t>(t.q_row0 + row) * hq + h) * D + 4 * g;
    const float2* tab = rope + static_cast<int64_t>(t.q_pos0 + row - delta) * H + 4 * g;
#pragma unroll
    for (int b = 0; b < NT / 2; ++b) {
      const row4_t y0 = load_row4(src + 16 * b);
      const row4_t y1 = load_row4(src + 16 * b + H);
      const float4 c01 = *reinterpret_cast<const float4*>(tab + 16 * b);
      const float4 c23 = *reinterpret_cast<const float4*>(tab + 16 * b + 2);
      const float cs[4] = {c01.x, c01.z, c23.x, c23.z}, sn[4] = {c01.y, c01.w, c23.y, c23.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float x0 = y0[i], x1 = y1[i];
        qv[x][b][i] = x0 * cs[i] - x1 * sn[i];
        qv[x][b + NT / 2][i] = x1 * cs[i] + x0 * sn[i];
      }
    }
  };
  // The steps of one page for row block x.  raw: K Q^T of the page in kr, two chains.
  auto raw = [&](int x, f32x4_t& s0, f32x4_t& s1) {
    s0 = s1 = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int b = 0; b < NT; b += 2)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(kr[b][i], qv[x][b][i], s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(kr[b + 1][i], qv[x][b + 1][i], s1, 0, 0, 0);
      }
  };
  // top: the scores in base-2 units, masked (partial page, causal), and the row max
  auto top = [&](int x, const KvPage& cur, const f32x4_t& s0, const f32x4_t& s1, float (&s)[4]) -> float {
    const int lim = min(cur.n_valid, t.q_pos0 + 16 * x + r - cur.pos0 + 1) - 4 * g;
#pragma unroll
    for (int j = 0; j < 4; ++j) s[j] = j < lim ? (s0[j] + s1[j]) * scale_log2 : -INFINITY;
    return fmaxf(m[x], row_max4(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]))));
  };
  // weigh: the running max raised (O and l rescaled) if some row needs it, then the weights in s
  auto weigh = [&](int x, float m_new, float (&s)[4]) {
    if (__any(m_new > m[x])) {
      const float corr = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m[x] - m_new);  // m = -inf: 0
      l[x] *= corr;
#pragma unroll
      for (int b = 0; b < NT; ++b)
#pragma unroll
        for (int j = 0; j < 4; ++j) o[x][b][j] *= corr;
      m[x] = m_new;
    }
    const float base = m[x] == -INFINITY ? 0.f : m[x];  // a row with no key so far: every weight 0
#pragma unroll
    for (int j = 0; j < 4; ++j) s[j] = __builtin_amdgcn_exp2f(s[j] - base);
    l[x] += (s[0] + s[1]) + (s[2] + s[3]);
  };
  auto add_v = [&](int x, const float (&p)[4]) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int b = 0; b < NT; ++b)
        o[x][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(vr[b][j], p[j], o[x][b], 0, 0, 0);
  };
  // One matrix instruction, then a few vector ones, over the code since the last fence:
  // the other row block's scores are masked and reduced under the matrix work.
  auto interleave = [&]() {
#pragma unroll
    for (int i = 0; i < 2 * NT; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
    }
  };

  // This wave's pages: wave, wave + kGW, .. of the list, or with `runs` a quarter of it in
  // one run, in either case up to the first that starts past the last row (positions do
  // not decrease along a list).  A step takes the page of pg, whose K is on its way, for
  // row blocks X0 .. X1 - 1.  The planner's tiles start where a page does, or end with the one
  // they start in: every row of a block sees some key of each page that the block takes, so
  // that a page's infinite or NaN values (0 times them is NaN) reach no row before it.
  // Alternate pages keep the waves level on a causal list.  A cross list changes delta from
  // fragment to fragment, and each change costs a wave a trip to memory for its query: in
  // runs a wave meets a few of them, not one with every page (16 rows over 288 keys in
  // four 64-token fragments, head dim 64: 11.0 -> 8.5 us).
  const int n_pages = t.kv_end - t.kv_begin;
  const int run = (n_pages + kGW - 1) / kGW;
  const int stride = runs ? 1 : kGW;
  const int end = runs ? min(t.kv_end, t.kv_begin + (wave + 1) * run) : t.kv_end;
  int pi = t.kv_begin + (runs ? wave * run : wave);
  bool more = pi < end;
  KvPage pg{};
  if (more) {
    pg = kv[pi];
    more = pg.pos0 <= last_pos;
    if (more) load_k(pg.page_id);
  }
  auto step = [&](auto x0, auto x1) __attribute__((always_inline)) {
    constexpr int X0 = decltype(x0)::value, X1 = decltype(x1)::value;
    constexpr bool BOTH = X1 - X0 == 2;
    const KvPage cur = pg;
    pi += stride;
    more = pi < end;
    if (more) pg = kv[pi];
    load_v(cur.page_id);
    if (cur.delta != q_delta) {
      q_delta = cur.delta;
#pragma unroll
      for (int x = X0; x < X1; ++x) load_q(x, q_delta);
    }
    f32x4_t a0, a1, b0, b1;
    float s[4], s2[4], mx;
    raw(X0, a0, a1);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (BOTH) raw(1, b0, b1);
    mx = top(X0, cur, a0, a1, s);
    if constexpr (BOTH) interleave();
    more = more && pg.pos0 <= last_pos;
    // unconditional (the last page again at the end), so that the waits for V need not
    // cover it: behind a branch the compiler would wait for both
    load_k(more ? pg.page_id : cur.page_id);
    weigh(X0, mx, s);
    __builtin_amdgcn_sched_barrier(0);
    add_v(X0, s);
    if constexpr (BOTH) {
      mx = top(1, cur, b0, b1, s2);
      interleave();
      weigh(1, mx, s2);
      add_v(1, s2);
    }
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  if (two) {
    while (more && pg.pos0 <= t.q_pos0 + 15) step(I0{}, I2{});
    while (more) step(I1{}, I2{});  // pages past the first row block
  } else {
    while (more) step(I0{}, I1{});
  }

  // ---- merge the waves' partials of every row through LDS
#pragma unroll
  for (int x = 0; x < kRB; ++x) {
    if (x > 0 && !two) break;
    const float lx = row_sum4(l[x]);
    const int sl = (wave * kRB + x) * 16 + r;
#pragma unroll
    for (int b = 0; b < NT; ++b) *reinterpret_cast<f32x4_t*>(sh_o + sl * OROW + 4 * g + 16 * b) = o[x][b];
    if (g == 0) {
      sh_m[sl] = m[x];
      sh_l[sl] = lx;
    }
  }
  __syncthreads();
  for (int e = threadIdx.x; e < t.n_rows * (D / 4); e += 64 * kGW) {
    const int c = e % (D / 4), x = e / (D / 4);
    float mm = -INFINITY;
#pragma unroll
    for (int k = 0; k < kGW; ++k) mm = fmaxf(mm, sh_m[k * kItemRows + x]);
    const float base = mm == -INFINITY ? 0.f : mm;
    float ll = 0.f;
    f32x4_t a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < kGW; ++k) {
      const int sl = k * kItemRows + x;
      const float f = __builtin_amdgcn_exp2f(sh_m[sl] - base);
      ll += sh_l[sl] * f;
      const f32x4_t v = *reinterpret_cast<const f32x4_t*>(sh_o + sl * OROW + 4 * c);
#pragma unroll
      for (int j = 0; j < 4; ++j) a[j] += v[j] * f;
    }
    const float inv = ll > 0.f ? 1.f / ll : 0.f;
    if (t.part < 0) {
      row4_t w;
#pragma unroll
      for (int j = 0; j < 4; ++j) w[j] = a[j] * inv;
      store_row4(out + (static_cast<int64_t>(t.q_row0 + x) * hq + h) * D + 4 * c, w);
    } else {
      const int64_t slot = (static_cast<int64_t>(t.part) * hq + h) * kGenericBM + row0 + x;
      if constexpr (PartOf<T>::normalized)
#pragma unroll
        for (int j = 0; j < 4; ++j) a[j] *= inv;
      store_part4(part_o + slot * D + 4 * c, a);
      if (c == 0) {
        part_ml[slot * 2] = mm;
        part_ml[slot * 2 + 1] = ll;
      }
    }
  }
}

template <typename T, int D>
hipError_t attn_generic_t(const PoolGeom& g, const WorkTile* tiles, int n, const KvPage* kv, const void* q, void* out,
                          void* part_o, float* part_ml, const float2* rope, bool runs, hipStream_t s) {
  const float scale_log2 = static_cast<float>(1.4426950408889634 / std::sqrt(static_cast<double>(D)));
  constexpr int lds = GGeo<D>::LDS;
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_generic_kernel<T, D>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (attr != hipSuccess) return attr;
  const int64_t items = static_cast<int64_t>(kItemsPerTile) * g.hq;  // of a tile
  return launch_in_slices(n, items * 64 * kGW, hipErrorInvalidValue, [&](int64_t t0, int64_t nt) {
    hipLaunchKernelGGL((attn_generic_kernel<T, D>), dim3(static_cast<unsigned>(nt * items)), dim3(64 * kGW), lds, s,
                       tiles + t0, kv, static_cast<const T*>(q), static_cast<T*>(out), static_cast<const T*>(g.base),
                       g.layer_off, g.hq, g.hkv, scale_log2, rope, runs,
                       static_cast<typename PartOf<T>::type*>(part_o), part_ml);
    return hipGetLastError();
  });
}

}  // namespace

hipError_t launch_attn_generic(const PoolGeom& g, const WorkTile* tiles, int n, const KvPage* kv, const void* q,
                               void* out, void* part_o, float* part_ml, const float2* rope, bool runs, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  auto go = [&](auto d) {
    constexpr int D = decltype(d)::value;
    return g.dtype == SPAN_BF16 ? attn_generic_t<bf16_t, D>(g, tiles, n, kv, q, out, part_o, part_ml, rope, runs, s)
                                : attn_generic_t<float, D>(g, tiles, n, kv, q, out, part_o, part_ml, rope, runs, s);
  };
  return g.d == 128 ? go(std::integral_constant<int, 128>{}) : go(std::integral_constant<int, 64>{});
}

}  // namespace spanq
