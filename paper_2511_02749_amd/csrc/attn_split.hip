// Span attention on bf16 pools for any number of query heads per kv head, for gfx950:
// queries and weights keep fp32 precision, on bf16 matrix instructions.
//
// The pages hold bf16 keys and values, which are matrix operands as they are.  The
// rotated query and the softmax weights are fp32; each is taken as the sum of three
// bf16 numbers (x = hi + mid + lo, each the rounding of what the ones before left: 24
// bits), and every product with K or V is three MFMAs into one fp32 accumulation.  A
// bf16 product is exact in fp32, so the sums are those of an fp32 kernel, at a third of
// the bf16 matrix rate, which is five times the fp32 one.
//
// Work item: (row tile of t tokens, kv head), all query heads of the kv head together.
// Its t x heads rows are numbered token by token and packed into 32-row blocks, one per
// wave, so any head count fills the blocks, and K and V are read once for all heads.  A
// work-group has four waves (128 rows).  With at most 64 rows two waves share a row
// block and each takes one of the two 32-key blocks of a tile; the two partial
// softmaxes meet in LDS at the end.  (More than 128 heads per kv head are cut into
// chunks of 128, each an item of its own.)
//
// Key tiles (four pages, 64 keys) go HBM -> LDS by DMA, two stages, the next tile's DMA
// in flight while this one is used; LDS layouts, the transposed scores S^T = K Q^T and
// the use of P^T as an operand as it stands are those of the other MFMA kernels
// (attn_mfma.hip).  Where a tile's keys are to be repositioned by delta, the query is
// formed again from its raw row at its position less delta, in fp32.
//
// A page that no row of a wave sees is left out, and one that some do not see adds to the others'
// sums only: 0 times an infinite or NaN value of it would be NaN.  (One comparison per page; the
// layer below took 134.5 us with every page of a 32-key block in every row, 132.9 so.)
//
// Two work-groups share a CU (two waves per SIMD, 64 KiB of LDS each at head dim 128),
// so that one's start, softmax and stores run under the other's matrix work.
//
// Bound: the SIMD's issue.  A 32 x 32 block of scores at head dim 128 is 48 MFMAs of 32
// cycles, and about 170 vector instructions with 16 exponentials (about 900 cycles) that
// the two waves of a SIMD, in step, overlap little: 10.3 k cycles per 64-key tile against
// 6.1 k of matrix work.  24 query over 8 kv heads at head dim 128, prefix 200 and 8
// fragments of about 400 (19 GFLOP with a 77-row cross segment): 5.15 ms on one wave per
// row tile with vector arithmetic, 0.26 ms on fp32 MFMAs (the kernel of the fp32 pools),
// 0.133 ms here.  64 rows per work-group, for a shorter last round: 0.148 ms.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "../../include/spanq.h"
#include "dev_common.h"
#include "grid.h"
#include "kernels.h"
#include "mfma_common.h"

namespace spanq {

namespace {

using namespace mfma;

constexpr int kSW = 4;         // waves per work-group
constexpr int kSRows = 32 * kSW;  // packed rows per work item
constexpr int kTerms = 3;      // bf16 terms of an fp32 value

template <int D>
struct SGeo {
  static constexpr int KS = D / 16;           // 16-dim steps of the QK contraction
  static constexpr int DB = D / 32;           // 32-dim blocks of the output
  static constexpr int KBYTES = kBN * D * 2;  // K tile: [64 keys][D]
  static constexpr int VBYTES = D * kBN * 2;  // V tile: [4 pages][D][16 positions]
  static constexpr int STAGE = KBYTES + VBYTES;
  static constexpr int KPW = KBYTES / 1024 / kSW;  // DMA instructions per wave: its page's K, and its V
  static constexpr int VPW = VBYTES / 1024 / kSW;
  static constexpr int MROW = 32 + 1;              // merge: floats per dim of a wave's O (padded)
  static constexpr int MERGE = 2 * (D * MROW + 64) * 4;
  static constexpr int LDS = 2 * STAGE > MERGE ? 2 * STAGE : MERGE;
};

// x0, x1 as sums of three bf16 pairs.  An infinity is its own first term: with INF the
// terms after it are 0, not inf - inf.
template <bool INF>
__device__ __forceinline__ void split3(float x0, float x1, uint32_t (&w)[kTerms]) {
#pragma unroll
  for (int t = 0; t < kTerms; ++t) {
    w[t] = pack_bf16x2(x0, x1);
    const float h0 = lo_bf16(w[t]), h1 = hi_bf16(w[t]);
    x0 = INF && __builtin_isinf(h0) ? 0.f : x0 - h0;
    x1 = INF && __builtin_isinf(h1) ? 0.f : x1 - h1;
  }
}

__device__ __forceinline__ float other_half(float x) {  // the value of lane ^ 32, with x
  const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(s[0]), __uint_as_float(s[1]));
}
__device__ __forceinline__ float both_halves(float x) {
  const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}

template <int D>
__global__ __launch_bounds__(64 * kSW) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_split_kernel(
    const WorkTile* __restrict__ tiles, const TileRec* __restrict__ kt, const bf16_t* __restrict__ q,
    bf16_t* __restrict__ out, const bf16_t* __restrict__ pool, int64_t layer_off, int hq, int hkv, int bm, int chunks,
    float scale_log2, const float2* __restrict__ rope, f16_t* __restrict__ part_o, float* __restrict__ part_ml) {
  using GE = SGeo<D>;
  constexpr int KS = GE::KS, DB = GE::DB, H = D / 2;
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int r = lane & 31, h2 = lane >> 5;
  const int kvh = blockIdx.x % hkv;
  const int rest = blockIdx.x / hkv;
  const int chunk = rest % chunks;
  const WorkTile t = tiles[rest / chunks];
  const int G = hq / hkv;
  const int gc = min(G - chunk * kSRows, kSRows);  // heads of this item
  const int rows = t.n_rows * gc;                  // packed rows: row fr is token fr / gc, head fr % gc
  const bool halves = rows <= 64;  // two waves per row block, a key block each
  const int rb = halves ? (wave & 1) : wave;
  const int kb0 = halves ? wave >> 1 : 0, kb1 = halves ? kb0 + 1 : 2;
  const int fr0 = 32 * rb, fr = fr0 + r;
  const bool row_ok = fr < rows;
  const bool active = fr0 < rows;
  const int tok = fr / gc;
  const int head = kvh * G + chunk * kSRows + (fr - tok * gc);
  const int qpos = t.q_pos0 + tok;
  const int first_pos = t.q_pos0 + fr0 / gc;  // of this wave's rows
  const int last_pos = t.q_pos0 + min(fr0 + 31, rows - 1) / gc;
  const int64_t page_elems = 2ll * hkv * kPage * D;

  // ---- DMA: wave w brings page w of a tile, K then V (per-lane byte offsets in a page)
  constexpr int CPK = D / 8;  // 16-byte chunks per key row
  static_assert(GE::KPW * (64 / CPK) == kPage && GE::VPW * 32 == D, "one page per wave");
  // (recomputed for every tile from an opaque copy of the lane id: no registers to spare)
  auto dk = [&](int ln, int u) {
    const int key = u * (64 / CPK) + ln / CPK;
    return 2u * static_cast<uint32_t>(key * D + 8 * ((ln % CPK) ^ kswz<D>(wave * kPage + key)));
  };
  auto dv = [&](int ln, int u) {
    const int d = 32 * u + (ln >> 1);
    return 2u * static_cast<uint32_t>(hkv * kPage * D + d * kPage + 8 * ((ln & 1) ^ ((d >> 3) & 1)));
  };
  const unsigned char* const pool_b =
      reinterpret_cast<const unsigned char*>(pool + layer_off + static_cast<int64_t>(kvh) * kPage * D);
  auto fetch = [&](int pid, int slot) {
    const unsigned char* pg = pool_b + static_cast<int64_t>(pid) * (page_elems * 2);
    const uint32_t at = lds_byte(lds) + slot * GE::STAGE;
    int ln = lane;
    __asm__ volatile("" : "+v"(ln));
#pragma unroll
    for (int u = 0; u < GE::KPW; ++u) dma16_s(pg, dk(ln, u), at + (wave * GE::KPW + u) * 1024);
#pragma unroll
    for (int u = 0; u < GE::VPW; ++u) dma16_s(pg, dv(ln, u), at + GE::KBYTES + (wave * GE::VPW + u) * 1024);
  };

  bf16x8_t qf[kTerms][KS];  // Q^T operands: rotated, scaled by log2(e)/sqrt(d), in three terms
  f32x16_t o[DB];
  float m = -INFINITY, l = 0.f;  // l: this half-wave's keys
  int q_delta = -1;
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[db][i] = 0.f;

  // qf <- R(position - delta) q.  (No row reads keys past its own position, and a key's
  // stored position, its final one less delta, is at least 0.)
  auto load_q = [&](int delta) {
    if (!row_ok) {
#pragma unroll
      for (int x = 0; x < kTerms; ++x)
#pragma unroll
        for (int s = 0; s < KS; ++s) qf[x][s] = __builtin_bit_cast(bf16x8_t, u32x4_t{0u, 0u, 0u, 0u});
      return;
    }
    // the caller's rows are only known to be aligned to an element
    typedef uint32_t row16 __attribute__((ext_vector_type(4), aligned(2)));
    int tk = tok;
    __asm__ volatile("" : "+v"(tk));
    const bf16_t* src = q + (static_cast<int64_t>(t.q_row0 + tk) * hq + head) * D + 8 * h2;
    const float4* tab =
        reinterpret_cast<const float4*>(rope + static_cast<int64_t>(t.q_pos0 + tk - delta) * H + 8 * h2);
    u32x4_t raw[KS];  // every load first: one trip to memory, not one per frequency block
    float4 cs[KS / 2][4];
#pragma unroll
    for (int s = 0; s < KS; ++s) raw[s] = *reinterpret_cast<const row16*>(src + 16 * s);
#pragma unroll
    for (int s = 0; s < KS / 2; ++s)
#pragma unroll
      for (int e = 0; e < 4; ++e) cs[s][e] = tab[8 * s + e];  // frequencies 16s + 8h2 + 2e, + 1
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < KS / 2; ++s) {
      const u32x4_t a4 = raw[s], b4 = raw[s + KS / 2];
      u32x4_t wa[kTerms], wb[kTerms];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float4 c = cs[s][e];
        const float a0 = lo_bf16(a4[e]), a1 = hi_bf16(a4[e]), b0 = lo_bf16(b4[e]), b1 = hi_bf16(b4[e]);
        uint32_t w[kTerms];
        split3<true>((a0 * c.x - b0 * c.y) * scale_log2, (a1 * c.z - b1 * c.w) * scale_log2, w);
#pragma unroll
        for (int x = 0; x < kTerms; ++x) wa[x][e] = w[x];
        split3<true>((b0 * c.x + a0 * c.y) * scale_log2, (b1 * c.z + a1 * c.w) * scale_log2, w);
#pragma unroll
        for (int x = 0; x < kTerms; ++x) wb[x][e] = w[x];
      }
#pragma unroll
      for (int x = 0; x < kTerms; ++x) {
        qf[x][s] = __builtin_bit_cast(bf16x8_t, wa[x]);
        qf[x][s + KS / 2] = __builtin_bit_cast(bf16x8_t, wb[x]);
      }
    }
  };

  // ---- one 32-key block kb of the tile in `stage`
  auto block = [&](const unsigned char* stage, int kb, int pos0, int nk) {
    const unsigned char* kl = stage + kb * 32 * D * 2;
    // Chunk 2ks + h2 of key row r sits at that chunk ^ kswz(r): one xor with the step's
    // constant.  (From an opaque copy of the lane id, as in fetch.)
    int ln = lane;
    __asm__ volatile("" : "+v"(ln));
    const int lr = ln & 31, lh = ln >> 5;
    const uint32_t krow = 2u * D * lr, kch = 16u * (lh ^ kswz<D>(lr));
    auto kofs = [&](int ks) { return krow + (kch ^ (32u * ks)); };
    const uint32_t vofs = 32u * lr + 16u * (lh ^ ((lr >> 3) & 1));
    f32x16_t sc;
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int i = 0; i < 16; ++i) sc[i] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8_t a = *reinterpret_cast<const bf16x8_t*>(kl + kofs(ks));
#pragma unroll
      for (int x = kTerms - 1; x >= 0; --x) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[x][ks], sc, 0, 0, 0);
    }
    __builtin_amdgcn_s_setprio(0);
    // causal positions and partial or empty pages; element i is key 8(i/4) + 4h2 + i%4
    if (nk < 32 * kb + 32 || pos0 + 32 * kb + 31 > first_pos) {
      const int lim = min(nk, qpos - pos0 + 1) - 32 * kb - 4 * h2;
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (8 * (i >> 2) + (i & 3) >= lim) sc[i] = -INFINITY;
    }
    float mx = sc[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) mx = fmaxf(mx, sc[i]);
    const float m_new = fmaxf(m, other_half(mx));
    if (__any(m_new > m)) {
      const float corr = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m - m_new);  // m = -inf: 0
      l *= corr;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[db][i] *= corr;
      m = m_new;
    }
    const float base = m == -INFINITY ? 0.f : m;  // a row with no key so far: every weight 0
    const bf16x8_t* vl = reinterpret_cast<const bf16x8_t*>(stage + GE::KBYTES + kb * 2 * D * 32 + vofs);
    float ts = 0.f;
#pragma unroll
    for (int half = 0; half < 2; ++half) {  // page 2kb + half: keys 16half .. of the block
      const int key0 = 32 * kb + 16 * half;
      if (key0 >= nk || pos0 + key0 > last_pos) break;  // no row sees it
      u32x4_t pw[kTerms];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float p0 = __builtin_amdgcn_exp2f(sc[8 * half + 2 * e] - base);
        const float p1 = __builtin_amdgcn_exp2f(sc[8 * half + 2 * e + 1] - base);
        ts += p0 + p1;
        uint32_t w[kTerms];
        split3<false>(p0, p1, w);
#pragma unroll
        for (int x = 0; x < kTerms; ++x) pw[x][e] = w[x];
      }
      auto add = [&](int x, int db) {
        o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vl[(half * D * 32 + db * 1024) / 16],
                                                        __builtin_bit_cast(bf16x8_t, pw[x]), o[db], 0, 0, 0);
      };
      if (pos0 + key0 <= first_pos) {
#pragma unroll
        for (int x = kTerms - 1; x >= 0; --x)
#pragma unroll
          for (int db = 0; db < DB; ++db) add(x, db);
      } else {
        // Rows before the page keep their sums as they are: 0 times a value of the page that is
        // infinite or NaN would end up in rows that do not see it.
        const bool sees = qpos >= pos0 + key0;
#pragma unroll
        for (int db = 0; db < DB; ++db) {
          const f32x16_t before = o[db];
#pragma unroll
          for (int x = kTerms - 1; x >= 0; --x) add(x, db);
#pragma unroll
          for (int i = 0; i < 16; ++i) o[db][i] = sees ? o[db][i] : before[i];
          __builtin_amdgcn_sched_barrier(0);  // one block's copy at a time: no registers to spare
        }
      }
    }
    l += ts;
  };

  // ---- the key tiles: wait for this wave's part of tile j, one barrier (every wave's
  // part has landed, and every wave is done with tile j - 1), fetch j + 1, use j
  const TileRec* const rec = kt + (t.kv_begin >> 2);
  const int n_tiles = (t.kv_end - t.kv_begin) >> 2;
  if (n_tiles > 0) {
    fetch(rec[0].page_id[wave], 0);
    if (active) {  // the first query beside the first tile's DMA
      q_delta = rec[0].delta;
      load_q(q_delta);
    }
  }
  for (int j = 0; j < n_tiles; ++j) {
    const int pos0 = rec[j].pos0, nk = rec[j].nk, delta = rec[j].delta;
    const int next_page = j + 1 < n_tiles ? rec[j + 1].page_id[wave] : 0;
    wait_vm_all();
    block_sync();
    if (j + 1 < n_tiles) fetch(next_page, (j + 1) & 1);
    if (active && pos0 <= last_pos) {
      if (delta != q_delta) {
        q_delta = delta;
        load_q(delta);
      }
      const unsigned char* stage = lds + (j & 1) * GE::STAGE;
      for (int kb = kb0; kb < kb1; ++kb)
        if (pos0 + 32 * kb <= last_pos) block(stage, kb, pos0, nk);
    }
  }

  // ---- two waves per row block: the second key group's partial joins the first through LDS
  float lt = both_halves(l);
  if (halves) {
    block_sync();  // every wave is done with the last tile
    float* const mo = reinterpret_cast<float*>(lds) + rb * (D * GE::MROW + 64);  // [dim][row], then m, l
    if (kb0 == 1 && active) {
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) mo[(32 * db + 8 * (i >> 2) + 4 * h2 + (i & 3)) * GE::MROW + r] = o[db][i];
      if (h2 == 0) {
        mo[D * GE::MROW + r] = m;
        mo[D * GE::MROW + 32 + r] = lt;
      }
    }
    __syncthreads();
    if (kb0 == 1 || !active) return;
    const float m2 = mo[D * GE::MROW + r], l2 = mo[D * GE::MROW + 32 + r];
    const float mm = fmaxf(m, m2), base = mm == -INFINITY ? 0.f : mm;
    const float f1 = __builtin_amdgcn_exp2f(m - base), f2 = __builtin_amdgcn_exp2f(m2 - base);
    lt = lt * f1 + l2 * f2;
    m = mm;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i)
        o[db][i] = o[db][i] * f1 + mo[(32 * db + 8 * (i >> 2) + 4 * h2 + (i & 3)) * GE::MROW + r] * f2;
  }
  if (!row_ok) return;
  const float inv = lt > 0.f ? 1.f / lt : 0.f;
  if (t.part < 0) {
    typedef uint16_t out4 __attribute__((ext_vector_type(4), aligned(2)));
    bf16_t* dst = out + (static_cast<int64_t>(t.q_row0 + tok) * hq + head) * D + 4 * h2;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const uint32_t w0 = pack_bf16x2(o[db][4 * g4] * inv, o[db][4 * g4 + 1] * inv);
        const uint32_t w1 = pack_bf16x2(o[db][4 * g4 + 2] * inv, o[db][4 * g4 + 3] * inv);
        *reinterpret_cast<out4*>(dst + 32 * db + 8 * g4) =
            out4{static_cast<uint16_t>(w0), static_cast<uint16_t>(w0 >> 16), static_cast<uint16_t>(w1),
                 static_cast<uint16_t>(w1 >> 16)};
      }
  } else {
    const int64_t slot = (static_cast<int64_t>(t.part) * hq + head) * bm + tok;
    f16_t* po = part_o + slot * D + 4 * h2;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4)
        *reinterpret_cast<f16x4_t*>(po + 32 * db + 8 * g4) =
            f16x4_t{static_cast<f16_t>(o[db][4 * g4] * inv), static_cast<f16_t>(o[db][4 * g4 + 1] * inv),
                    static_cast<f16_t>(o[db][4 * g4 + 2] * inv), static_cast<f16_t>(o[db][4 * g4 + 3] * inv)};
    if (h2 == 0) {
      part_ml[slot * 2] = m;
      part_ml[slot * 2 + 1] = lt;
    }
  }
}

template <int D>
hipError_t launch_t(const PoolGeom& g, const WorkTile* tiles, int n, const TileRec* kt, const void* q, void* out,
                    void* part_o, float* part_ml, const float2* rope, hipStream_t s) {
  const float scale_log2 = static_cast<float>(1.4426950408889634 / std::sqrt(static_cast<double>(D)));
  constexpr int lds = SGeo<D>::LDS;
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_split_kernel<D>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (attr != hipSuccess) return attr;
  const int G = g.hq / g.hkv;
  const int chunks = split_chunks(G);
  const int64_t items = static_cast<int64_t>(g.hkv) * chunks;  // of a tile
  return launch_in_slices(n, items * 64 * kSW, hipErrorInvalidValue, [&](int64_t t0, int64_t nt) {
    hipLaunchKernelGGL((attn_split_kernel<D>), dim3(static_cast<unsigned>(nt * items)), dim3(64 * kSW), lds, s,
                       tiles + t0, kt, static_cast<const bf16_t*>(q), static_cast<bf16_t*>(out),
                       static_cast<const bf16_t*>(g.base), g.layer_off, g.hq, g.hkv, split_bm(G), chunks, scale_log2,
                       rope, static_cast<f16_t*>(part_o), part_ml);
    return hipGetLastError();
  });
}

}  // namespace

int split_bm(int g) { return std::max(1, kSRows / g); }
int split_chunks(int g) { return (g + kSRows - 1) / kSRows; }

hipError_t launch_attn_split(const PoolGeom& g, const WorkTile* tiles, int n, const TileRec* kt, const void* q,
                             void* out, void* part_o, float* part_ml, const float2* rope, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (g.dtype != SPAN_BF16 || (g.d != 64 && g.d != 128)) return hipErrorInvalidValue;
  return g.d == 128 ? launch_t<128>(g, tiles, n, kt, q, out, part_o, part_ml, rope, s)
                    : launch_t<64>(g, tiles, n, kt, q, out, part_o, part_ml, rope, s);
}

}  // namespace spanq
