// MSV-Prune scoring (Sec. 4.1): anchor scores, anchor top-k (Eq. 1),
// K-means on last-layer features (Sec. 4.1.2), anchor max-similarity and the
// per-token multi-layer similarity score of Eq. 3 in its factored form:
//   mean_{j in C} S_ij = sum_l u^l_i . mu^l_C + m_i + mean_{j in C} m_j,
//   u^l_i = F^l_i / |F^l_i|,  mu^l_C = mean_{j in C} u^l_j.
//
// Kernels (all per tile g, enqueued in this order):
//   score_prep     grid (ceil(n/16), G) x 256: a_i (sequential fp32 head sum,
//                  then one IEEE division) and 1/|F^l_i| for every tapped layer.
//   anchor_topk    grid G x 64: one wave finds the n_anchor-th largest score
//                  bit by bit and writes the ascending anchor and non-anchor
//                  lists.
//   anchor_maxsim  m_i = max_p u_i . u_p.  bf16: v_mfma_f32_32x32x16_bf16 on the
//                  raw rows (exact products, fp32 accumulation) scaled by the two
//                  inverse norms: grid (ceil(n/32), G) x 256, a wave per anchor
//                  tile, rows and anchors through an LDS ring (rows32), from 512
//                  128-row blocks on grid (ceil(n/128), G) x 256, anchors staged
//                  in LDS per 64-dimension chunk; fp32: grid (ceil(n/4), G), a
//                  wave-per-row FMA loop.
//   kmeans         grid (NB, G) x 512 per Lloyd pass: rows and centroids in
//                  LDS, distances, then per-block cluster sums in a fixed
//                  order (deterministic).
//   score_final    cluster means of unit rows per tapped layer (same
//                  fixed-order sums), cluster mean of m, and the factored
//                  score of every non-anchor row.
//
// Lane-to-dimension map of the dot products and distances: lane l owns VPL
// dimensions, in chunks of 8: dims {c*512 + 8*l + e : c < VPL/8, e < 8}.
#include <algorithm>
#include <cfloat>
#include <cmath>
#include <mutex>

#include "common.h"
#include "topk.h"

namespace spider {
namespace {

template <typename FT>
struct Feat;
template <>
struct Feat<float> {
  static constexpr spider_dtype dt = SPIDER_F32;
  // 8 consecutive elements -> fp32
  __device__ static inline void load8(const float* p, float* o) {
    const float4 a = *reinterpret_cast<const float4*>(p);
    const float4 b = *reinterpret_cast<const float4*>(p + 4);
    o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w;
    o[4] = b.x; o[5] = b.y; o[6] = b.z; o[7] = b.w;
  }
  __device__ static inline float load1(const float* p) { return *p; }
  // 8 consecutive elements kept raw while in flight
  struct Raw {
    floatx4 a, b;
  };
  __device__ static inline Raw load8_raw(const float* p) {
    return {*reinterpret_cast<const floatx4*>(p), *reinterpret_cast<const floatx4*>(p + 4)};
  }
  __device__ static inline float raw_at(const Raw& v, int e) { return e < 4 ? v.a[e] : v.b[e - 4]; }
  __device__ static inline Raw load8_nt(const float* p) {
    return {__builtin_nontemporal_load(reinterpret_cast<const floatx4*>(p)),
            __builtin_nontemporal_load(reinterpret_cast<const floatx4*>(p + 4))};
  }
  static constexpr int kPrepRowBatch = 2;
};
template <>
struct Feat<uint16_t> {
  static constexpr spider_dtype dt = SPIDER_BF16;
  __device__ static inline void load8(const uint16_t* p, float* o) {
    const uint4 v = *reinterpret_cast<const uint4*>(p);
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      o[2 * i] = __uint_as_float(w[i] << 16);
      o[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
    }
  }
  __device__ static inline float load1(const uint16_t* p) { return bf16_bits_to_f32(*p); }
  typedef u32x4 Raw;
  __device__ static inline Raw load8_raw(const uint16_t* p) { return *reinterpret_cast<const u32x4*>(p); }
  __device__ static inline Raw load8_nt(const uint16_t* p) {
    return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
  }
  __device__ static inline float raw_at(const Raw& v, int e) {
    return __uint_as_float((e & 1) ? (v[e >> 1] & 0xFFFF0000u) : (v[e >> 1] << 16));
  }
  static constexpr int kPrepRowBatch = 4;
};

struct FeatArgs {
  const void* ptr[8];
  int64_t stride_g, stride_row;
  int row0;
};

template <typename FT>
__device__ inline const FT* feat_row(const FeatArgs& fa, int l, int g, int i) {
  return reinterpret_cast<const FT*>(fa.ptr[l]) + (int64_t)g * fa.stride_g +
         (int64_t)(fa.row0 + i) * fa.stride_row;
}

// Load this lane's VPL dims of a row (zeros beyond d).
template <typename FT, int VPL>
__device__ inline void load_slice(const FT* row, int d, int lane, float* x) {
#pragma unroll
  for (int c = 0; c < VPL / 8; ++c) {
    const int base = c * 512 + lane * 8;
    if (base + 8 <= d) {
      Feat<FT>::load8(row + base, x + 8 * c);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) x[8 * c + e] = (base + e < d) ? Feat<FT>::load1(row + base + e) : 0.f;
    }
  }
}

__device__ inline int slice_dim(int v, int lane) { return (v >> 3) * 512 + lane * 8 + (v & 7); }

// ------------------------------------------------------------- score_prep
// Row norms of every tapped layer and the head-mean anchor scores, 16 patches
// per block (the compulsory single read of the features and the CLS rows).
// Each wave owns 4 patches; per tapped layer it issues the 16-byte loads of
// a batch of rows (4 bf16 / 2 fp32 rows, NCH chunks of 512 elements each)
// before reducing any of them.  Small batches keep the kernel at ~58 VGPRs,
// 8 waves per SIMD: more waves in flight moved more bytes than more loads per
// wave (8-row batches at 97 VGPRs ran 35 % slower).  A lane sums its chunks
// in ascending order and the wave sum is a fixed butterfly.  The last 16
// threads own one patch's head mean each, after their rows: all head loads
// are issued (8 at a time) before the sum, which runs over h = 0..H-1 in
// order, then one IEEE division.  Loads are non-temporal when the features
// exceed the last-level cache (kPrepNtBytes): the later passes re-read the
// same rows, from that cache while the tiles fit in it, and from HBM anyway
// once they do not.
constexpr int kPrepRows = 16;
constexpr int64_t kPrepNtBytes = 256ll << 20;  // MI355X Infinity Cache

template <typename FT, int NCH, bool NT>
__global__ void __launch_bounds__(256) score_prep_kernel(
    int n, int H, int d, int n_layers, const float* __restrict__ attn, int64_t as_g,
    int64_t as_h, int col0, FeatArgs fa, float* __restrict__ a_out, float* __restrict__ nu) {
  const int g = blockIdx.y;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int i0 = blockIdx.x * kPrepRows;
  constexpr int RW = kPrepRows / 4;  // rows per wave, in batches of RB
  constexpr int RB = Feat<FT>::kPrepRowBatch;
  const int r0 = i0 + RW * wave;
  for (int l = 0; l < n_layers; ++l) {
#pragma unroll
    for (int rb = 0; rb < RW; rb += RB) {
      typename Feat<FT>::Raw x[RB][NCH];
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        const FT* row = feat_row<FT>(fa, l, g, min(r0 + rb + r, n - 1));
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
          const int e0 = lane * 8 + 512 * c;
          if (e0 < d) x[r][c] = NT ? Feat<FT>::load8_nt(row + e0) : Feat<FT>::load8_raw(row + e0);
        }
      }
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        float ss = 0.f;
#pragma unroll
        for (int c = 0; c < NCH; ++c)
          if (lane * 8 + 512 * c < d) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const float v = Feat<FT>::raw_at(x[r][c], e);
              ss = fmaf(v, v, ss);
            }
          }
        ss = wave_sum(ss);
        const int i = r0 + rb + r;
        if (lane == 0 && i < n) nu[((int64_t)g * n_layers + l) * n + i] = ss > 0.f ? 1.0f / sqrtf(ss) : 0.f;
      }
    }
  }
  const int t = threadIdx.x - (256 - kPrepRows);
  if (attn && t >= 0 && i0 + t < n) {  // null: scores given in a_out
    const int i = i0 + t;
    const float* col = attn + (int64_t)g * as_g + col0 + i;
    float acc = 0.f;
    for (int h0 = 0; h0 < H; h0 += 8) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = h0 + u < H ? col[(int64_t)(h0 + u) * as_h] : 0.f;
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (h0 + u < H) acc = __fadd_rn(acc, v[u]);
    }
    a_out[(int64_t)g * n + i] = __fdiv_rn(acc, (float)H);
  }
}

template <typename FT>
void launch_score_prep(int G, int n, int H, int d, int n_layers, const float* attn, int64_t as_g, int64_t as_h,
                       int col0, const FeatArgs& fa, float* a_out, float* nu, hipStream_t st) {
  const dim3 grid(ceil_div(n, kPrepRows), G);
  const bool nt = (int64_t)G * n * d * (int64_t)sizeof(FT) * n_layers > kPrepNtBytes;
#define SPIDER_PREP(NCH_, NT_) \
  score_prep_kernel<FT, NCH_, NT_><<<grid, 256, 0, st>>>(n, H, d, n_layers, attn, as_g, as_h, col0, fa, a_out, nu)
  if (d <= 512) {
    if (nt) SPIDER_PREP(1, true); else SPIDER_PREP(1, false);
  } else if (d <= 1024) {
    if (nt) SPIDER_PREP(2, true); else SPIDER_PREP(2, false);
  } else {
    if (nt) SPIDER_PREP(4, true); else SPIDER_PREP(4, false);
  }
#undef SPIDER_PREP
}

// ------------------------------------------------------------- anchor_topk
constexpr int kMaxN = 4096;

// One wave per tile: the n_anchor largest scores (ties to the lower index),
// then the ascending anchor and non-anchor lists from ballots.
template <int NV>
__global__ void __launch_bounds__(64) anchor_topk_kernel(int n, int n_anchor, const float* __restrict__ a,
                                                         int32_t* __restrict__ cluster_out, float* __restrict__ s_out,
                                                         int32_t* __restrict__ anc_list,
                                                         int32_t* __restrict__ rest_list, int32_t* __restrict__ conv) {
  const int g = blockIdx.x, lane = threadIdx.x;
  if (lane == 0) conv[g] = 0;
  const int64_t o = (int64_t)g * n;
  const int nv = (n + 63) / 64;
  uint32_t key[NV];
  {
    float x[NV];  // every load first: a load under its own bounds check waits for the one before it
#pragma unroll
    for (int v = 0; v < NV; ++v) x[v] = a[o + min(64 * v + lane, n - 1)];
#pragma unroll
    for (int v = 0; v < NV; ++v) key[v] = 64 * v + lane < n ? float_order_key(x[v]) : 0u;
  }
  const TopK<NV> top = wave_kth_largest<NV>(key, nv, n_anchor);
  int na = 0, ties = 0;  // anchors and ties below register v
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    if (v >= nv) break;
    const int i = 64 * v + lane;
    const uint64_t eq = __ballot(i < n && key[v] == top.t);
    const bool sel = i < n && (key[v] > top.t || (key[v] == top.t && ties + lanes_below(eq) < top.ties));
    const uint64_t m = __ballot(sel);
    const int before = na + lanes_below(m);
    if (sel) {
      anc_list[o + before] = i;
      cluster_out[o + i] = -1;
      s_out[o + i] = INFINITY;
    } else if (i < n) {
      rest_list[o + (i - before)] = i;
      cluster_out[o + i] = 0;
    }
    ties += __popcll(eq);
    na += __popcll(m);
  }
}

// ------------------------------------------------------------- anchor_maxsim
// m_i = max_p u_i . u_p over the anchors p of the tile (bf16 features):
// one block per 128 rows, one 32-row tile per wave (B operand: lane % 32 owns
// a row and its output), the anchors in tiles of 32 (A operand), up to 8 tiles
// per pass over the rows.  The anchors go through LDS one 64-dimension chunk
// at a time (double buffered; 16-byte chunk q of anchor a at slot
// q ^ ((a >> 1) & 7), so a 16-lane read of 16 anchors hits distinct banks)
// and serve all four waves; each wave reads its own rows once, the next
// chunk's loads in flight while the current chunk's MFMAs run.  A lane
// covers k in [k0 + 32 hi, k0 + 32 hi + 32) as 4 chunks of 8 for both
// operands (v_mfma_f32_32x32x16_bf16, exact products, fp32 accumulation in
// chunk order), then acc * nu_row * nu_anchor, maxed.
// Accumulator register r of an anchor tile: anchor p0 + 8 (r / 4) + 4 hi + r % 4
// against the lane's row.  The anchors' inverse norms are loaded all at once (a
// load under its own bounds check waits for the one before it: 16 times two
// dependent loads per tile).
__device__ __forceinline__ float max_over_anchors(const floatx16& acc, int p0, int hi, int n_anchor,
                                                  const int32_t* anc, const float* nu_g, float nu_r, float best) {
  int at[16];
  float nu[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) at[r] = anc[min(p0 + 8 * (r >> 2) + 4 * hi + (r & 3), n_anchor - 1)];
#pragma unroll
  for (int r = 0; r < 16; ++r) nu[r] = nu_g[at[r]];
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const float v = acc[r] * nu_r * nu[r];
    best = p0 + 8 * (r >> 2) + 4 * hi + (r & 3) < n_anchor ? fmaxf(best, v) : best;
  }
  return best;
}

constexpr int kMaxAnchorTiles = 8;
// Up to two 128-row blocks per CU the 32-row kernel is faster (64 tiles of 576,
// 320 such blocks: 69 against 80 us); from there on the anchors it reads once
// per 32 rows instead of once per 128 cost more (256 tiles: 243 against 218 us).
constexpr int kMaxsimBlocks = 512;

__global__ void __launch_bounds__(256) anchor_maxsim_bf16_kernel(
    int n, int d, int n_anchor, FeatArgs fa, int last, const float* __restrict__ nu_last,
    int64_t nu_stride_g, const int32_t* __restrict__ anc_list, float* __restrict__ mvec) {
  __shared__ __attribute__((aligned(16))) uint8_t abuf[2][kMaxAnchorTiles * 32 * 128];
  const int g = blockIdx.y;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, hi = lane >> 5, lo = lane & 31;
  const int my_row = blockIdx.x * 128 + 32 * wave + lo;
  const bool row_ok = my_row < n;
  const uint16_t* rowp = feat_row<uint16_t>(fa, last, g, row_ok ? my_row : 0);
  const float* nu_g = nu_last + (int64_t)g * nu_stride_g;
  const int32_t* anc = anc_list + (int64_t)g * n;
  const float nu_r = row_ok ? nu_g[my_row] : 0.f;
  float best = -INFINITY;
  const int n_at = (n_anchor + 31) / 32;
  const int nkc = (d + 63) / 64;
  // staging: thread (anchor a = tid / 8 + 32 j of the pass, chunk q = tid % 8)
  const int sq = tid & 7, sa0 = tid >> 3;
  for (int t0 = 0; t0 < n_at; t0 += kMaxAnchorTiles) {
    const int nt = min(kMaxAnchorTiles, n_at - t0);
    const uint16_t* sp[kMaxAnchorTiles];
#pragma unroll
    for (int j = 0; j < kMaxAnchorTiles; ++j) {
      const int p = 32 * (t0 + j) + sa0;
      sp[j] = (j < nt && p < n_anchor) ? feat_row<uint16_t>(fa, last, g, anc[p]) : nullptr;
    }
    u32x4 ast[kMaxAnchorTiles], bv[4], bn[4];
    auto load_anchors = [&](int k0) {
      const int kk = k0 + 8 * sq;
#pragma unroll
      for (int j = 0; j < kMaxAnchorTiles; ++j)
        ast[j] = (sp[j] && kk + 8 <= d) ? *reinterpret_cast<const u32x4*>(sp[j] + kk) : u32x4{0, 0, 0, 0};
    };
    auto store_anchors = [&](int buf) {
#pragma unroll
      for (int j = 0; j < kMaxAnchorTiles; ++j)
        if (j < nt) {
          const int a = sa0 + 32 * j;
          *reinterpret_cast<u32x4*>(&abuf[buf][a * 128 + 16 * (sq ^ ((a >> 1) & 7))]) = ast[j];
        }
    };
    auto load_rows = [&](int k0, u32x4* dst) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int kk = k0 + 32 * hi + 8 * c;
        dst[c] = (row_ok && kk + 8 <= d) ? *reinterpret_cast<const u32x4*>(rowp + kk) : u32x4{0, 0, 0, 0};
      }
    };
    floatx16 acc[kMaxAnchorTiles];
#pragma unroll
    for (int j = 0; j < kMaxAnchorTiles; ++j) acc[j] = floatx16{};
    load_anchors(0);
    load_rows(0, bv);
    store_anchors(0);
    __syncthreads();
    for (int kc = 0; kc < nkc; ++kc) {
      const bool more = kc + 1 < nkc;
      if (more) {
        load_anchors(64 * (kc + 1));
        load_rows(64 * (kc + 1), bn);
      }
      const uint8_t* ab = abuf[kc & 1];
#pragma unroll
      for (int j = 0; j < kMaxAnchorTiles; ++j)
        if (j < nt) {
          const int a = 32 * j + lo;
          bf16x8 av[4];
#pragma unroll
          for (int c = 0; c < 4; ++c)
            av[c] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(ab + a * 128 + 16 * ((4 * hi + c) ^ ((a >> 1) & 7))));
#pragma unroll
          for (int c = 0; c < 4; ++c)
            acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[c], __builtin_bit_cast(bf16x8, bv[c]), acc[j], 0, 0, 0);
        }
      if (more) store_anchors((kc + 1) & 1);  // that buffer was last read before the previous barrier
      __syncthreads();
#pragma unroll
      for (int c = 0; c < 4; ++c) bv[c] = bn[c];
    }
    // acc[j][r]: anchor 32 (t0 + j) + 8 (r / 4) + 4 hi + r % 4, data row my_row
#pragma unroll
    for (int j = 0; j < kMaxAnchorTiles; ++j)
      if (j < nt) best = max_over_anchors(acc[j], 32 * (t0 + j), hi, n_anchor, anc, nu_g, nu_r, best);
  }
  best = fmaxf(best, __shfl_xor(best, 32, 64));
  if (hi == 0 && row_ok) mvec[(int64_t)g * n + my_row] = n_anchor > 0 ? best : 0.f;
}

// The same similarities where 128-row blocks would leave most CUs idle: a block
// per 32 rows, a wave per anchor tile (4 tiles per pass over the rows).  Rows
// and anchors of a 64-dimension chunk go to LDS by DMA into a ring of four
// stages, three chunks ahead (row r's 16-byte chunk c at slot c ^ ((r >> 1) & 7)
// as in the kernel above).  Same MFMAs in the same order, and a maximum does
// not depend on its order: the same bits.  Bounded by the latency of the
// chunks; one tile of 576 x 1024 with 89 anchors: 5 blocks took 31 us, 18 take
// 11 us; 20 tiles with 201 anchors 49 -> 26 us.
__global__ void __launch_bounds__(256) anchor_maxsim_bf16_rows32_kernel(
    int n, int d, int n_anchor, FeatArgs fa, int last, const float* __restrict__ nu_last,
    int64_t nu_stride_g, const int32_t* __restrict__ anc_list, float* __restrict__ mvec) {
  constexpr int STAGES = 4, LEAD = STAGES - 1, STAGE = 5 * 4096, PER_IT = 5;  // rows, then 4 anchor tiles
  __shared__ __attribute__((aligned(1024))) uint8_t ring[STAGES * STAGE];
  const int g = blockIdx.y;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, hi = lane >> 5,
            lo = lane & 31;
  const int i0 = blockIdx.x * 32, my_row = i0 + lo;
  const uint32_t lds = lds_offset(ring);
  const float* nu_g = nu_last + (int64_t)g * nu_stride_g;
  const int32_t* anc = anc_list + (int64_t)g * n;
  const float nu_r = my_row < n ? nu_g[my_row] : 0.f;
  const int n_at = (n_anchor + 31) / 32, nkc = (d + 63) / 64;
  // DMA: lane l fills slot l % 8 of row 8 q + l / 8 of a 32-row tile; this wave
  // brings rows 8 wave .. of the row tile and its own anchor tile
  const int dr = lane >> 3, dc = lane & 7;
  const int r_row = 8 * wave + dr, r_ch = 8 * (dc ^ ((r_row >> 1) & 7));
  const uint16_t* rp = feat_row<uint16_t>(fa, last, g, min(i0 + r_row, n - 1));
  float best = -INFINITY;
  for (int t0 = 0; t0 < n_at; t0 += 4) {
    const int t = min(t0 + wave, n_at - 1);  // a repeated tile changes no maximum
    const uint16_t* ap[4];
    int a_ch[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = 8 * q + dr;
      ap[q] = feat_row<uint16_t>(fa, last, g, anc[min(32 * t + r, n_anchor - 1)]);
      a_ch[q] = 8 * (dc ^ ((r >> 1) & 7));
    }
    auto issue = [&](int kc, auto S) {
      const uint32_t st = lds + decltype(S)::value * STAGE;
      // past the last dimension: any element of the row (its products are dropped below)
      auto at = [&](int ch) { return 64 * kc + ch < d ? 64 * kc + ch : 0; };
      dma16(rp + at(r_ch), st + wave * 1024);
#pragma unroll
      for (int q = 0; q < 4; ++q) dma16(ap[q] + at(a_ch[q]), st + 4096 * (1 + wave) + q * 1024);
    };
    floatx16 acc{};
    __syncthreads();  // the pass before is done with the ring
    static_for<0, LEAD>([&](auto P) { issue(min((int)P.value, nkc - 1), P); });
    dma_wait_barrier<(LEAD - 1) * PER_IT>();
    for (int k0 = 0; k0 < nkc; k0 += STAGES) {
      static_for<0, STAGES>([&](auto P) {
        const int kc = k0 + P.value;
        if (kc < nkc) {
          issue(min(kc + LEAD, nkc - 1), std::integral_constant<int, (P.value + LEAD) % STAGES>{});
          const uint8_t* st = ring + P.value * STAGE;
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const int at = lo * 128 + 16 * ((4 * hi + c) ^ ((lo >> 1) & 7));
            u32x4 bv = *reinterpret_cast<const u32x4*>(st + at);
            u32x4 av = *reinterpret_cast<const u32x4*>(st + 4096 * (1 + wave) + at);
            if (64 * kc + 32 * hi + 8 * c >= d) av = bv = u32x4{0, 0, 0, 0};
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av),
                                                          __builtin_bit_cast(bf16x8, bv), acc, 0, 0, 0);
          }
          dma_wait_barrier<(LEAD - 1) * PER_IT>();
        }
      });
    }
    dma_wait_all();
    best = max_over_anchors(acc, 32 * t, hi, n_anchor, anc, nu_g, nu_r, best);
  }
  best = fmaxf(best, __shfl_xor(best, 32, 64));
  __syncthreads();
  float* wbest = reinterpret_cast<float*>(ring);  // [4][32]
  if (hi == 0) wbest[32 * wave + lo] = best;
  __syncthreads();
  if (wave == 0 && hi == 0 && my_row < n)
    mvec[(int64_t)g * n + my_row] =
        n_anchor > 0 ? fmaxf(fmaxf(wbest[lo], wbest[32 + lo]), fmaxf(wbest[64 + lo], wbest[96 + lo])) : 0.f;
}

// fp32 features: one wave per data row, loop over anchors.
__global__ void __launch_bounds__(256) anchor_maxsim_f32_kernel(
    int n, int d, int n_anchor, FeatArgs fa, int last, const float* __restrict__ nu_last,
    int64_t nu_stride_g, const int32_t* __restrict__ anc_list, float* __restrict__ mvec) {
  const int g = blockIdx.y;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int i = blockIdx.x * 4 + wave;
  if (i >= n) return;
  const float* row = feat_row<float>(fa, last, g, i);
  const float* nu_g = nu_last + (int64_t)g * nu_stride_g;
  float best = -INFINITY;
  for (int q = 0; q < n_anchor; ++q) {
    const int p = anc_list[(int64_t)g * n + q];
    const float* pr = feat_row<float>(fa, last, g, p);
    float dot = 0.f;
    for (int c = lane; c < d; c += 64) dot = fmaf(row[c], pr[c], dot);
    dot = wave_sum(dot);
    best = fmaxf(best, dot * nu_g[i] * nu_g[p]);
  }
  if (lane == 0) mvec[(int64_t)g * n + i] = n_anchor > 0 ? best : 0.f;
}

// ------------------------------------------------------------- clustering
// Lloyd iterations.  Each tile's m non-anchor rows are split into NB
// contiguous row ranges, one 512-thread block per range and pass.  The host
// enqueues max_iter passes; the passes after the first that changes no
// assignment return at once.
//
// A pass (kmeans_pass_kernel): the block's rows go to LDS by DMA (at most
// kRowLdsBytes at a time), the centroids into LDS beside them; each wave takes
// 4 rows at a time against 4 centroids, whose 16 sums over the dimensions are
// reduced together (reduce_4x4); then every thread owns 2 or 4 dimensions and
// adds the rows from LDS to their clusters.  Sums run in a fixed order, the
// same whatever the number of tiles: row j of the block's range belongs to
// lane group j % 4, each group adds its rows in ascending order, and the groups
// are added ((0 + 1) + 2) + 3.
//
// Centroids of pass p > 0: the NB blocks' partial sums added in block order,
// divided by the count; an empty cluster keeps its centroid.  Up to
// kSelfUpdateBlocks blocks every block forms them itself from the partial sums
// (which alternate between two buffers), more blocks read what
// kmeans_update_kernel wrote between the passes: reading NB * K * d floats per
// block costs less than a launch only while few blocks do it (20 tiles, 320
// blocks: 94 us against 113; 64 tiles alike; 256 tiles: 484 against 416).
//
// What bounds it: latency.  One tile of 576 x 1024 bf16 patches has 16 blocks
// and ten passes of which 3 or 4 work; 19 launches (pass and update) took
// 180 us, ten take 62 us (20 tiles: 171 -> 82 us).
constexpr int kClusterThreads = 512;
constexpr int kRowLdsBytes = 64 << 10;
constexpr int kMaxRowsPerBlock = 128;
constexpr int kSelfUpdateBlocks = 512;

struct ClusterWs {
  float* cent;      // [G][K][d]
  float* psum;      // [G][NB][K][d] (kmeans; two such buffers with self-update) / [G][NB][L][K][d] (means)
  int32_t* pcnt;    // [G][NB][K]       rows per cluster; kmeans: bit 16 of the first = an assignment changed
  float* pm;        // [G][NB][K]       partial sums of m (kmeans with self-update: the second pcnt)
  int32_t* conv;    // [G]
  int32_t* assign;  // [G][n]  assignment of non-anchor row j (index into U)
  float* mu;        // [G][L][K][d] (kmeans with self-update: the second cent)
  float* mbar;      // [G][K]
  int NB, RB;       // blocks per tile, rows per block
  int nb_used;
  int64_t psum2;    // elements from the first to the second partial-sum buffer
};
constexpr int kChangedBit = 1 << 16;

// Rows staged at a time: a multiple of 4 (at least 8: a row has at most 8 KB).
__host__ __device__ inline int chunk_rows(int rb, int row_bytes) {
  const int fit = kRowLdsBytes / row_bytes / 4 * 4, need = (rb + 3) / 4 * 4;
  return fit < need ? fit : need;
}

// LDS bytes of the staged rows (the DMA writes whole KBs).
__host__ __device__ inline int chunk_bytes(int rb, int row_bytes) {
  const int ch = chunk_rows(rb, row_bytes), rows = ch < rb ? ch : rb;
  return (rows * row_bytes + 1023) / 1024 * 1024;
}

// Rows sidx[0..nr) of layer l into LDS at byte offset `lds`, packed at d elements.
template <typename FT>
__device__ __forceinline__ void stage_rows(const FeatArgs& fa, int l, int g, int d, const int* sidx, int nr,
                                           uint32_t lds) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  constexpr int E = 16 / (int)sizeof(FT);
  const int per_row = d / E, total = nr * per_row;  // 16-byte pieces
  for (int base = wave * 64; base < total; base += kClusterThreads) {
    const int p = min(base + lane, total - 1);
    const int r = p / per_row, c = p - r * per_row;
    dma16(reinterpret_cast<const uint16_t*>(feat_row<FT>(fa, l, g, sidx[r]) + c * E), lds + base * 16);
  }
}

// 16 values v[4 r + k] per lane summed over the wave: lane row rho (16 lanes)
// ends with the sums of r = rho, for k = 0..3 in v[0..3].  The butterfly of
// wave_sum (same pairs in the same order, so the same bits), halving the number
// of values at its first two steps instead of repeating them for each.
__device__ __forceinline__ void reduce_4x4(float (&v)[16]) {
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[i]), __float_as_uint(v[i + 8]), false, false);
    v[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[i]), __float_as_uint(v[i + 4]), false, false);
    v[i] = row16_sum(__uint_as_float(r[0]) + __uint_as_float(r[1]));
  }
}

// Dimensions per thread of the row sums (512 threads).
template <int NCH>
constexpr int kDims = NCH <= 2 ? 2 : 4;

// Adds the nr staged rows to acc[row % 4][cluster][this thread's dimensions]
// (first dimension DP * threadIdx.x); sc: the rows' scales, null for 1.
template <typename FT, int KM, int DP>
__device__ __forceinline__ void add_rows(float (&acc)[4][KM][DP], const uint8_t* rows, int d, int nr, const int* lab,
                                         const float* sc) {
  const int dim = DP * threadIdx.x;
  if (dim >= d) return;
  for (int q = 0; q < nr; q += 4) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      if (q + v >= nr) break;
      const FT* src = reinterpret_cast<const FT*>(rows) + (q + v) * d + dim;
      float x[DP];
#pragma unroll
      for (int e = 0; e < DP; ++e) x[e] = Feat<FT>::load1(src + e);
      const int k = __builtin_amdgcn_readfirstlane(lab[q + v]);
      const float w = sc ? sc[q + v] : 1.0f;
#pragma unroll
      for (int c = 0; c < KM; ++c)
#pragma unroll
        for (int e = 0; e < DP; ++e) {
          const float t = fmaf(x[e], w, acc[v][c][e]);
          acc[v][c][e] = k == c ? t : acc[v][c][e];
        }
    }
  }
}

template <int KM, int DP>
__device__ __forceinline__ void store_sums(const float (&acc)[4][KM][DP], int K, int d, float* out) {
  const int dim = DP * threadIdx.x;
  if (dim >= d) return;
#pragma unroll
  for (int k = 0; k < KM; ++k) {
    if (k >= K) break;
#pragma unroll
    for (int e = 0; e < DP; ++e)
      out[k * d + dim + e] = ((acc[0][k][e] + acc[1][k][e]) + acc[2][k][e]) + acc[3][k][e];
  }
}

template <typename FT, int NCH, int KM>
__global__ void __launch_bounds__(kClusterThreads) kmeans_pass_kernel(int n, int d, int n_anchor, int K, int pass,
                                                                      int self, FeatArgs fa, int last,
                                                                      const int32_t* __restrict__ rest_list,
                                                                      ClusterWs cw, int32_t* __restrict__ cluster_out) {
  extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];  // staged rows, then centroids [K][d]
  __shared__ int lab[kMaxRowsPerBlock], old[kMaxRowsPerBlock], sidx[kMaxRowsPerBlock];
  __shared__ int scnt[8];
  __shared__ int chg;
  const int g = blockIdx.y, b = blockIdx.x;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int m = n - n_anchor;
  const int j0 = b * cw.RB, j1 = min(m, j0 + cw.RB), nr = j1 - j0;
  const int64_t slot = (int64_t)g * cw.NB + b;
  // buffers of this pass and of the one before (the same without self-update)
  const bool odd = self && (pass & 1);
  int32_t* cnt_cur = odd ? reinterpret_cast<int32_t*>(cw.pm) : cw.pcnt;
  const int32_t* cnt_prev = self && !odd ? reinterpret_cast<const int32_t*>(cw.pm) : cw.pcnt;
  float* cent_cur = (odd ? cw.mu : cw.cent) + (int64_t)g * K * d;
  const float* cent_prev = (self && !odd ? cw.mu : cw.cent) + (int64_t)g * K * d;
  float* sum_cur = cw.psum + (odd ? cw.psum2 : 0) + slot * K * d;
  const float* sum_prev = cw.psum + (self && !odd ? cw.psum2 : 0) + (int64_t)g * cw.NB * K * d;
  const int32_t* U = rest_list + (int64_t)g * n;
  int32_t* asg = cw.assign + (int64_t)g * n;
  // nothing below waits for the convergence flags but the exit itself: the
  // loads of a pass form one chain of two (indices, rows), not of four
  const int u_j = U[j0 + min(tid, nr - 1)];
  const int a_j = pass > 0 ? asg[j0 + min(tid, nr - 1)] : -1;
  if (self && pass > 0) {
    const int32_t* cp = cnt_prev + ((int64_t)g * cw.NB + min(lane, cw.nb_used - 1)) * K;
    const int c = cp[0], ck = cp[min(wave, K - 1)];
    // converged: the pass before changed nothing (NB <= 64 blocks, one lane each)
    if (!__ballot(c & kChangedBit)) {
      if (tid == 0) cnt_cur[slot * K] = 0;  // for the next pass, which reads this buffer
      return;
    }
    // rows of cluster `wave` over all blocks
    const int rows_k = wave_sum_int(lane < cw.nb_used ? (ck & 0xFFFF) : 0);
    if (lane == 0 && wave < K) scnt[wave] = rows_k;
  } else if (!self && cw.conv[g]) {
    return;
  }
  if (tid < nr) {  // nr <= kMaxRowsPerBlock
    sidx[tid] = u_j;
    old[tid] = a_j;
  }
  if (tid == 0) chg = 0;
  __syncthreads();
  const int row_bytes = d * (int)sizeof(FT);
  const int CH = chunk_rows(cw.RB, row_bytes);
  const uint32_t lds = lds_offset(smem);
  stage_rows<FT>(fa, last, g, d, sidx, min(CH, nr), lds);
  float* cs = reinterpret_cast<float*>(smem + chunk_bytes(cw.RB, row_bytes));
  if (pass == 0) {
    // centroids at rows floor(k*m/K) of the non-anchor list
    for (int t = tid * 8; t < K * d; t += kClusterThreads * 8) {
      const int k = t / d, c = t - k * d;
      float x[8];
      Feat<FT>::load8(feat_row<FT>(fa, last, g, U[(int)(((int64_t)k * m) / K)]) + c, x);
#pragma unroll
      for (int e = 0; e < 8; ++e) cs[t + e] = x[e];
      if (b == 0) {
#pragma unroll
        for (int e = 0; e < 8; ++e) cent_cur[t + e] = x[e];
      }
    }
  } else if (self) {
    for (int t = tid * 4; t < K * d; t += kClusterThreads * 4) {
      const int c = scnt[t / d];
      float4 v;
      if (c > 0) {
        float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int b0 = 0; b0 < cw.nb_used; b0 += 8) {
          float4 x[8];
#pragma unroll
          for (int u = 0; u < 8; ++u)
            if (b0 + u < cw.nb_used) x[u] = *reinterpret_cast<const float4*>(sum_prev + (int64_t)(b0 + u) * K * d + t);
#pragma unroll
          for (int u = 0; u < 8; ++u)
            if (b0 + u < cw.nb_used) {
              s.x += x[u].x;
              s.y += x[u].y;
              s.z += x[u].z;
              s.w += x[u].w;
            }
        }
        const float fc = (float)c;
        v = make_float4(__fdiv_rn(s.x, fc), __fdiv_rn(s.y, fc), __fdiv_rn(s.z, fc), __fdiv_rn(s.w, fc));
      } else {
        v = *reinterpret_cast<const float4*>(cent_prev + t);
      }
      *reinterpret_cast<float4*>(cs + t) = v;
      if (b == 0) *reinterpret_cast<float4*>(cent_cur + t) = v;
    }
  } else {
    for (int t = tid * 4; t < K * d; t += kClusterThreads * 4)
      *reinterpret_cast<float4*>(cs + t) = *reinterpret_cast<const float4*>(cent_prev + t);
  }
  constexpr int DP = kDims<NCH>;
  float acc[4][KM][DP];
#pragma unroll
  for (int v = 0; v < 4; ++v)
#pragma unroll
    for (int k = 0; k < KM; ++k)
#pragma unroll
      for (int e = 0; e < DP; ++e) acc[v][k][e] = 0.f;
  for (int c0 = 0; c0 < nr; c0 += CH) {
    const int cn = min(CH, nr - c0);
    if (c0 > 0) {
      __syncthreads();  // the chunk before is summed
      stage_rows<FT>(fa, last, g, d, sidx + c0, cn, lds);
    }
    dma_wait_all();
    __syncthreads();
    const FT* rows = reinterpret_cast<const FT*>(smem);
    for (int r0 = wave; r0 < cn; r0 += 32) {  // rows r0, r0 + 8, r0 + 16, r0 + 24
      float bd = 0.f;
      int best = 0;
#pragma unroll
      for (int kb = 0; kb < KM; kb += 4) {
        if (kb >= K) break;
        float s[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) s[q] = 0.f;
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
          const int base = c * 512 + lane * 8;
          if (base < d) {
            float x[4][8];
#pragma unroll
            for (int r = 0; r < 4; ++r) Feat<FT>::load8(rows + min(r0 + 8 * r, cn - 1) * d + base, x[r]);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              if (kb + k >= K) break;
              float cc[8];
              Feat<float>::load8(cs + (kb + k) * d + base, cc);
#pragma unroll
              for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                  const float t = x[r][e] - cc[e];
                  s[4 * r + k] = fmaf(t, t, s[4 * r + k]);
                }
            }
          }
        }
        reduce_4x4(s);
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (kb + k < K && (kb + k == 0 || s[k] < bd)) {
            bd = s[k];
            best = kb + k;
          }
      }
      const int r = r0 + 8 * (lane >> 4);
      if ((lane & 15) == 0 && r < cn) {
        lab[c0 + r] = best;
        if (old[c0 + r] != best) chg = 1;
        asg[j0 + c0 + r] = best;
        cluster_out[(int64_t)g * n + sidx[c0 + r]] = best;
      }
    }
    __syncthreads();
    add_rows<FT, KM, DP>(acc, smem, d, cn, lab + c0, nullptr);
  }
  store_sums<KM, DP>(acc, K, d, sum_cur);
  if (wave == 0) {
    for (int k = 0; k < K; ++k) {
      int c = 0;
      for (int q = 0; q < nr; q += 64) c += __popcll(__ballot(q + lane < nr && lab[min(q + lane, nr - 1)] == k));
      if (lane == 0) cnt_cur[slot * K + k] = c | (k == 0 && chg ? kChangedBit : 0);
    }
  }
}

// grid (ceil(K*d/256), G): new centroids = fixed-order sums of the partials.
__global__ void __launch_bounds__(256) kmeans_update_kernel(int d, int K, ClusterWs cw) {
  const int g = blockIdx.y;
  if (cw.conv[g]) return;
  int any = 0;
  for (int b = 0; b < cw.nb_used; ++b) any |= cw.pcnt[((int64_t)g * cw.NB + b) * K] & kChangedBit;
  if (!any) {
    if (blockIdx.x == 0 && threadIdx.x == 0) cw.conv[g] = 1;
    return;
  }
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t >= K * d) return;
  const int k = t / d;
  float s = 0.f;
  int c = 0;
  for (int b = 0; b < cw.nb_used; ++b) {
    const int64_t slot = (int64_t)g * cw.NB + b;
    s += cw.psum[slot * K * d + t];
    c += cw.pcnt[slot * K + k] & 0xFFFF;
  }
  if (c > 0) cw.cent[(int64_t)g * K * d + t] = __fdiv_rn(s, (float)c);
}

// Partial per-cluster sums of unit rows, a tapped layer per blockIdx.z, and of
// m.  The rows are staged and summed as in a K-means pass.
template <typename FT, int NCH, int KM>
__global__ void __launch_bounds__(kClusterThreads) cluster_sum_kernel(int n, int d, int n_anchor, int K, int n_layers,
                                                                      FeatArgs fa, const float* __restrict__ nu,
                                                                      const int32_t* __restrict__ rest_list,
                                                                      const float* __restrict__ mvec, ClusterWs cw) {
  extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];  // staged rows
  __shared__ int lab[kMaxRowsPerBlock], sidx[kMaxRowsPerBlock];
  __shared__ float sc[kMaxRowsPerBlock], sm_m[kMaxRowsPerBlock];
  const int g = blockIdx.y, b = blockIdx.x, l = blockIdx.z;
  const int tid = threadIdx.x;
  const int m = n - n_anchor;
  const int j0 = b * cw.RB, j1 = min(m, j0 + cw.RB), nr = j1 - j0;
  const int32_t* U = rest_list + (int64_t)g * n;
  const float* nul = nu + ((int64_t)g * n_layers + l) * n;
  for (int j = tid; j < nr; j += kClusterThreads) {
    const int i = U[j0 + j];
    sidx[j] = i;
    lab[j] = cw.assign[(int64_t)g * n + j0 + j];
    sc[j] = nul[i];
    sm_m[j] = mvec[(int64_t)g * n + i];
  }
  __syncthreads();
  constexpr int DP = kDims<NCH>;
  float acc[4][KM][DP];
#pragma unroll
  for (int v = 0; v < 4; ++v)
#pragma unroll
    for (int k = 0; k < KM; ++k)
#pragma unroll
      for (int e = 0; e < DP; ++e) acc[v][k][e] = 0.f;
  const int CH = chunk_rows(cw.RB, d * (int)sizeof(FT));
  const uint32_t lds = lds_offset(smem);
  const int64_t slot = (int64_t)g * cw.NB + b;
  for (int c0 = 0; c0 < nr; c0 += CH) {
    const int cn = min(CH, nr - c0);
    if (c0 > 0) __syncthreads();
    stage_rows<FT>(fa, l, g, d, sidx + c0, cn, lds);
    if (c0 == 0 && l == 0 && tid < K) {  // while the rows arrive
      int c = 0;
      float sm = 0.f;
      for (int j = 0; j < nr; ++j) {
        const bool mine = lab[j] == tid;
        const float t = sm + sm_m[j];
        c += mine;
        sm = mine ? t : sm;
      }
      cw.pcnt[slot * K + tid] = c;
      cw.pm[slot * K + tid] = sm;
    }
    dma_wait_all();
    __syncthreads();
    add_rows<FT, KM, DP>(acc, smem, d, cn, lab + c0, sc + c0);
  }
  store_sums<KM, DP>(acc, K, d, cw.psum + (slot * n_layers + l) * K * d);
}

// grid (ceil(L*K*d/256), G): mu = fixed-order sums / counts; mbar likewise.
__global__ void __launch_bounds__(256) cluster_mean_kernel(int d, int K, int n_layers, ClusterWs cw) {
  const int g = blockIdx.y;
  const int t = blockIdx.x * 256 + threadIdx.x;
  const int per = K * d;
  if (t < n_layers * per) {
    const int l = t / per, r = t - l * per, k = r / d;
    float s = 0.f;
    int c = 0;
    for (int b0 = 0; b0 < cw.nb_used; b0 += 8) {
      float x[8];
      int y[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int64_t slot = (int64_t)g * cw.NB + min(b0 + u, cw.nb_used - 1);
        x[u] = cw.psum[(slot * n_layers + l) * per + r];
        y[u] = cw.pcnt[slot * K + k];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (b0 + u < cw.nb_used) {
          s += x[u];
          c += y[u];
        }
    }
    cw.mu[((int64_t)g * n_layers + l) * per + r] = c ? __fdiv_rn(s, (float)c) : 0.f;
  }
  if (blockIdx.x == 0 && threadIdx.x < K) {
    const int k = threadIdx.x;
    float s = 0.f;
    int c = 0;
    for (int b = 0; b < cw.nb_used; ++b) {
      const int64_t slot = (int64_t)g * cw.NB + b;
      s += cw.pm[slot * K + k];
      c += cw.pcnt[slot * K + k];
    }
    cw.mbar[(int64_t)g * K + k] = c ? __fdiv_rn(s, (float)c) : 0.f;
  }
}

// One wave per non-anchor row (fallback where the cluster means do not fit in LDS): s = sum_l nu_l * (F^l_i . mu^l_c) + m_i + mbar_c.
template <typename FT, int VPL>
__global__ void __launch_bounds__(256) score_rows_wave_kernel(int n, int d, int n_anchor, int K,
                                                              int n_layers, FeatArgs fa,
                                                         const float* __restrict__ nu,
                                                         const int32_t* __restrict__ rest_list,
                                                         const float* __restrict__ mvec, ClusterWs cw,
                                                         float* __restrict__ s_out,
                                                         float* __restrict__ m_out) {
  const int g = blockIdx.y;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int m = n - n_anchor;
  if (m_out && blockIdx.x == 0)
    for (int i = threadIdx.x; i < n; i += blockDim.x) m_out[(int64_t)g * n + i] = mvec[(int64_t)g * n + i];
  const int j = blockIdx.x * 4 + wave;
  if (j >= m) return;
  const int i = rest_list[(int64_t)g * n + j];
  const int k = cw.assign[(int64_t)g * n + j];
  float s = 0.f;
  for (int l = 0; l < n_layers; ++l) {
    float x[VPL];
    load_slice<FT, VPL>(feat_row<FT>(fa, l, g, i), d, lane, x);
    const float* mu = cw.mu + (((int64_t)g * n_layers + l) * K + k) * d;
    float dot = 0.f;
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
      const int dim = slice_dim(v, lane);
      if (dim < d) dot = fmaf(x[v], mu[dim], dot);
    }
    dot = wave_sum(dot);
    s += dot * nu[((int64_t)g * n_layers + l) * n + i];
  }
  if (lane == 0) s_out[(int64_t)g * n + i] = s + mvec[(int64_t)g * n + i] + cw.mbar[(int64_t)g * K + k];
}

// The same scores, 64 or 16 rows per block, a quarter per wave in batches of RB rows
// whose feature loads (two tapped layers at a time) are all issued before
// any is used; the tile's cluster means mu[l][k] (n_layers * K * d floats, at
// most kMuLdsFloats) are staged in LDS once per block.  Per row and layer a
// lane adds its dimensions in ascending order, then the wave sum, then
// s += dot * nu_l in layer order: the arithmetic of score_rows_wave_kernel in
// the same order, so the same bits.
constexpr int kScoreRowsPerBlock = 64;
constexpr int kMuLdsFloats = 8192;

template <typename FT, int VPL>
__global__ void __launch_bounds__(256) score_rows_kernel(int n, int d, int n_anchor, int K, int n_layers,
                                                         FeatArgs fa, const float* __restrict__ nu,
                                                         const int32_t* __restrict__ rest_list,
                                                         const float* __restrict__ mvec, ClusterWs cw,
                                                         float* __restrict__ s_out, float* __restrict__ m_out,
                                                         int rows_per_wave) {
  __shared__ __attribute__((aligned(16))) float smu[kMuLdsFloats];
  const int g = blockIdx.y;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int m = n - n_anchor;
  if (m_out && blockIdx.x == 0)
    for (int i = threadIdx.x; i < n; i += blockDim.x) m_out[(int64_t)g * n + i] = mvec[(int64_t)g * n + i];
  if (m <= 0) return;
  const int lkd = n_layers * K * d;  // a multiple of 8 (d is)
  const float* mug = cw.mu + (int64_t)g * lkd;
  for (int t = threadIdx.x * 4; t < lkd; t += 1024)
    *reinterpret_cast<float4*>(smu + t) = *reinterpret_cast<const float4*>(mug + t);
  __syncthreads();
  constexpr int RB = Feat<FT>::kPrepRowBatch;
  constexpr int NCH = VPL / 8;
  const int32_t* U = rest_list + (int64_t)g * n;
  const int32_t* asg = cw.assign + (int64_t)g * n;
  const int jw = (blockIdx.x * 4 + wave) * rows_per_wave;
  for (int jb = 0; jb < rows_per_wave; jb += RB) {
    if (jw + jb >= m) break;
    int ii[RB], kc[RB];
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      const int j = min(jw + jb + r, m - 1);
      ii[r] = U[j];
      kc[r] = asg[j];
    }
    float sacc[RB];
#pragma unroll
    for (int r = 0; r < RB; ++r) sacc[r] = 0.f;
    for (int l0 = 0; l0 < n_layers; l0 += 2) {
      const bool two = l0 + 1 < n_layers;
      typename Feat<FT>::Raw x[2][RB][NCH];
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int r = 0; r < RB; ++r) {
          const FT* row = feat_row<FT>(fa, q == 0 || !two ? l0 : l0 + 1, g, ii[r]);
#pragma unroll
          for (int c = 0; c < NCH; ++c) {
            const int e0 = lane * 8 + 512 * c;
            if (e0 < d && (q == 0 || two)) x[q][r][c] = Feat<FT>::load8_raw(row + e0);
          }
        }
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        if (q == 1 && !two) break;
        const int l = l0 + q;
#pragma unroll
        for (int r = 0; r < RB; ++r) {
          const float* mu = smu + (l * K + kc[r]) * d;
          float dot = 0.f;
#pragma unroll
          for (int c = 0; c < NCH; ++c) {
            const int e0 = lane * 8 + 512 * c;
            if (e0 < d) {
              const float4 m0 = *reinterpret_cast<const float4*>(mu + e0);
              const float4 m1 = *reinterpret_cast<const float4*>(mu + e0 + 4);
              const float mv[8] = {m0.x, m0.y, m0.z, m0.w, m1.x, m1.y, m1.z, m1.w};
#pragma unroll
              for (int e = 0; e < 8; ++e) dot = fmaf(Feat<FT>::raw_at(x[q][r][c], e), mv[e], dot);
            }
          }
          dot = wave_sum(dot);
          sacc[r] += dot * nu[((int64_t)g * n_layers + l) * n + ii[r]];
        }
      }
    }
    if (lane == 0)
#pragma unroll
      for (int r = 0; r < RB; ++r)
        if (jw + jb + r < m)
          s_out[(int64_t)g * n + ii[r]] = sacc[r] + mvec[(int64_t)g * n + ii[r]] + cw.mbar[(int64_t)g * K + kc[r]];
  }
}

struct ScoreWs {
  float* nu;
  int32_t* anc;
  int32_t* rest;
  float* mvec;
  ClusterWs cw;
};

// Blocks per tile: about 32 rows each (at most 16 per tile, never more than
// kMaxRowsPerBlock rows per block).  It depends on n only, so a tile gets the
// same partial-sum order, hence the same bits, whatever the batch size G.
int blocks_per_tile(int G, int n) {
  (void)G;
  const int need = (n + kMaxRowsPerBlock - 1) / kMaxRowsPerBlock;
  const int want = std::min(16, (n + 31) / 32);
  return std::max(need, std::max(1, want));
}

size_t score_ws_layout(int G, int n, int d, int n_layers, int K, ScoreWs* w, char* base) {
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off = align_up(off + bytes, 256);
    return base ? base + o : nullptr;
  };
  const int NB = blocks_per_tile(G, n);
  const int L1 = std::max(1, n_layers);
  char* p_nu = take((size_t)G * n_layers * n * 4);
  char* p_anc = take((size_t)G * n * 4);
  char* p_rest = take((size_t)G * n * 4);
  char* p_mvec = take((size_t)G * n * 4);
  char* p_cent = take((size_t)G * K * d * 4);
  char* p_psum = take((size_t)G * NB * L1 * K * d * 4);
  char* p_pcnt = take((size_t)G * NB * K * 4);
  char* p_pm = take((size_t)G * NB * K * 4);
  char* p_conv = take((size_t)G * 4);
  char* p_asg = take((size_t)G * n * 4);
  char* p_mu = take((size_t)G * L1 * K * d * 4);
  char* p_mbar = take((size_t)G * K * 4);
  if (w) {
    w->nu = reinterpret_cast<float*>(p_nu);
    w->anc = reinterpret_cast<int32_t*>(p_anc);
    w->rest = reinterpret_cast<int32_t*>(p_rest);
    w->mvec = reinterpret_cast<float*>(p_mvec);
    w->cw.cent = reinterpret_cast<float*>(p_cent);
    w->cw.psum = reinterpret_cast<float*>(p_psum);
    w->cw.pcnt = reinterpret_cast<int32_t*>(p_pcnt);
    w->cw.pm = reinterpret_cast<float*>(p_pm);
    w->cw.conv = reinterpret_cast<int32_t*>(p_conv);
    w->cw.assign = reinterpret_cast<int32_t*>(p_asg);
    w->cw.mu = reinterpret_cast<float*>(p_mu);
    w->cw.mbar = reinterpret_cast<float*>(p_mbar);
    w->cw.NB = NB;
  }
  return off;
}

// NCH = chunks of 512 dimensions of a row (1, 2, 4); KM = 4 or 8 clusters.
template <typename FT, int NCH, int KM>
hipError_t launch_cluster_kernels(int G, int n, int d, int n_anchor, int K, int max_iter,
                                  int n_layers, const FeatArgs& fa, ScoreWs ws,
                                  int32_t* cluster_out, float* s_out, float* m_out, hipStream_t st) {
  const int m = n - n_anchor;
  const int NB = ws.cw.NB;
  ws.cw.RB = m > 0 ? (m + NB - 1) / NB : 1;
  const int nb_used = m > 0 ? (m + ws.cw.RB - 1) / ws.cw.RB : 0;
  ws.cw.nb_used = nb_used;
  ws.cw.psum2 = (int64_t)G * NB * K * d;
  // NB >= ceil(n / kMaxRowsPerBlock) guarantees these; checked before any launch
  if (ws.cw.RB > kMaxRowsPerBlock || nb_used > NB || NB > 64) return hipErrorInvalidValue;
  const size_t rows_lds = chunk_bytes(ws.cw.RB, d * (int)sizeof(FT));
  if (m > 0) {
    ProfScope ps(KC_KMEANS, st);
    // the second partial-sum buffer is the second layer's part of psum
    const bool self = n_layers >= 2 && G * nb_used <= kSelfUpdateBlocks;
    for (int it = 0; it < max_iter; ++it) {
      kmeans_pass_kernel<FT, NCH, KM><<<dim3(nb_used, G), kClusterThreads, rows_lds + (size_t)K * d * 4, st>>>(
          n, d, n_anchor, K, it, self, fa, n_layers - 1, ws.rest, ws.cw, cluster_out);
      hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
      if (!self && it + 1 < max_iter) {
        kmeans_update_kernel<<<dim3(ceil_div(K * d, 256), G), 256, 0, st>>>(d, K, ws.cw);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
      }
    }
  }
  {
    ProfScope ps(KC_SCORE_FINAL, st);
    if (m > 0) {
      cluster_sum_kernel<FT, NCH, KM><<<dim3(nb_used, G, n_layers), kClusterThreads, rows_lds, st>>>(
          n, d, n_anchor, K, n_layers, fa, ws.nu, ws.rest, ws.mvec, ws.cw);
      hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
      cluster_mean_kernel<<<dim3(ceil_div(n_layers * K * d, 256), G), 256, 0, st>>>(d, K, n_layers, ws.cw);
      e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    constexpr int VPL = 8 * NCH;
    if ((int64_t)n_layers * K * d <= kMuLdsFloats) {
      // 16 rows per block while 64 would leave most CUs without one
      const int rpb = (int64_t)ceil_div(std::max(m, 1), kScoreRowsPerBlock) * G >= 256 ? kScoreRowsPerBlock : 16;
      score_rows_kernel<FT, VPL><<<dim3(std::max(1, ceil_div(m, rpb)), G), 256, 0, st>>>(
          n, d, n_anchor, K, n_layers, fa, ws.nu, ws.rest, ws.mvec, ws.cw, s_out, m_out, rpb / 4);
    } else
      score_rows_wave_kernel<FT, VPL><<<dim3(std::max(1, ceil_div(m, 4)), G), 256, 0, st>>>(
          n, d, n_anchor, K, n_layers, fa, ws.nu, ws.rest, ws.mvec, ws.cw, s_out, m_out);
    return hipGetLastError();
  }
}

template <typename FT>
hipError_t dispatch_cluster(int G, int n, int d, int n_anchor, int K, int max_iter, int n_layers,
                            const FeatArgs& fa, const ScoreWs& ws, int32_t* cl, float* s,
                            float* mo, hipStream_t st) {
#define SPIDER_CLUSTER(NCH_, KM_) \
  launch_cluster_kernels<FT, NCH_, KM_>(G, n, d, n_anchor, K, max_iter, n_layers, fa, ws, cl, s, mo, st)
  if (d <= 512) return K <= 4 ? SPIDER_CLUSTER(1, 4) : SPIDER_CLUSTER(1, 8);
  if (d <= 1024) return K <= 4 ? SPIDER_CLUSTER(2, 4) : SPIDER_CLUSTER(2, 8);
  return SPIDER_CLUSTER(4, 4);  // K <= 4 past 1024 dimensions
#undef SPIDER_CLUSTER
}

}  // namespace
}  // namespace spider

using namespace spider;

extern "C" size_t spider_score_workspace_size(int G, int n, int d_v, int n_layers, int K) {
  if (G <= 0 || n <= 0 || d_v <= 0 || n_layers <= 0 || K <= 0) return 0;
  return score_ws_layout(G, n, d_v, n_layers, K, nullptr, nullptr);
}

extern "C" spider_status spider_score(int G, int n, int H, int d_v, int n_layers,
                                      const float* cls_attn, int64_t attn_stride_g,
                                      int64_t attn_stride_h, int attn_col0,
                                      const void* const* feats, spider_dtype feat_dtype,
                                      int64_t feat_stride_g, int64_t feat_stride_row, int feat_row0,
                                      int n_anchor, int K, int kmeans_max_iter, float* a_out,
                                      int32_t* cluster_out, float* s_out, float* m_out,
                                      void* workspace, size_t workspace_bytes,
                                      spider_stream stream) {
  clear_error();
  SPIDER_REQUIRE(G >= 1 && n >= 1 && d_v >= 1 && n_layers >= 1, SPIDER_ERR_INVALID_ARG,
                 "spider_score: G, n, d_v and n_layers must be >= 1");
  // cls_attn == NULL with H == 0: a_out already holds the anchor scores (input)
  const bool given_a = cls_attn == nullptr;
  SPIDER_REQUIRE(given_a ? H == 0 : H >= 1, SPIDER_ERR_INVALID_ARG,
                 "spider_score: H must be >= 1 with CLS attention, 0 with given anchor scores");
  SPIDER_REQUIRE(n <= kMaxN, SPIDER_ERR_UNSUPPORTED, "spider_score: n = %d exceeds 4096", n);
  SPIDER_REQUIRE(d_v <= 2048, SPIDER_ERR_UNSUPPORTED, "spider_score: d_v = %d exceeds 2048", d_v);
  SPIDER_REQUIRE(n_layers <= 8, SPIDER_ERR_UNSUPPORTED, "spider_score: at most 8 tapped layers");
  SPIDER_REQUIRE(K >= 1 && K <= 8, SPIDER_ERR_UNSUPPORTED, "spider_score: K must be in [1, 8]");
  SPIDER_REQUIRE(!(d_v > 1024 && K > 4), SPIDER_ERR_UNSUPPORTED,
                 "spider_score: K > 4 needs d_v <= 1024");
  SPIDER_REQUIRE(n_anchor >= 0 && n_anchor <= n, SPIDER_ERR_SHAPE,
                 "spider_score: n_anchor = %d outside [0, n = %d]", n_anchor, n);
  SPIDER_REQUIRE(kmeans_max_iter >= 1, SPIDER_ERR_INVALID_ARG,
                 "spider_score: kmeans_max_iter must be >= 1");
  SPIDER_REQUIRE(feats && a_out && cluster_out && s_out, SPIDER_ERR_INVALID_ARG,
                 "spider_score: null pointer argument");
  SPIDER_REQUIRE(feat_dtype == SPIDER_F32 || feat_dtype == SPIDER_BF16, SPIDER_ERR_INVALID_ARG,
                 "spider_score: bad feature dtype");
  SPIDER_REQUIRE(given_a || (attn_col0 >= 0 && attn_stride_h >= attn_col0 + n &&
                              attn_stride_g >= (int64_t)H * attn_stride_h),
                 SPIDER_ERR_SHAPE, "spider_score: attention strides do not cover [H, col0 + n]");
  SPIDER_REQUIRE(feat_row0 >= 0, SPIDER_ERR_SHAPE, "spider_score: feat_row0 must be >= 0");
  SPIDER_REQUIRE(feat_stride_row >= d_v && feat_stride_g >= (int64_t)(feat_row0 + n) * feat_stride_row,
                 SPIDER_ERR_SHAPE, "spider_score: feature strides do not cover [row0 + n, d_v]");
  SPIDER_REQUIRE(feat_stride_row % 8 == 0 && feat_stride_g % 8 == 0 && d_v % 8 == 0,
                 SPIDER_ERR_UNSUPPORTED,
                 "spider_score: d_v and the feature strides must be multiples of 8 elements");
  for (int l = 0; l < n_layers; ++l) {
    SPIDER_REQUIRE(feats[l] != nullptr, SPIDER_ERR_INVALID_ARG, "spider_score: feats[%d] is null", l);
    SPIDER_REQUIRE(((uintptr_t)feats[l] % 16) == 0, SPIDER_ERR_UNSUPPORTED,
                   "spider_score: feats[%d] must be 16-byte aligned", l);
  }
  const size_t need = score_ws_layout(G, n, d_v, n_layers, K, nullptr, nullptr);
  SPIDER_REQUIRE(workspace && workspace_bytes >= need, SPIDER_ERR_WORKSPACE,
                 "spider_score: workspace of %zu bytes needed, %zu given", need, workspace_bytes);
  SPIDER_REQUIRE(((uintptr_t)workspace % 256) == 0, SPIDER_ERR_WORKSPACE,
                 "spider_score: workspace must be 256-byte aligned");

  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  ScoreWs ws;
  score_ws_layout(G, n, d_v, n_layers, K, &ws, reinterpret_cast<char*>(workspace));
  FeatArgs fa;
  for (int l = 0; l < 8; ++l) fa.ptr[l] = l < n_layers ? feats[l] : nullptr;
  fa.stride_g = feat_stride_g;
  fa.stride_row = feat_stride_row;
  fa.row0 = feat_row0;
  const int last = n_layers - 1;

  {
    ProfScope ps(KC_SCORE_PREP, st);
    if (feat_dtype == SPIDER_BF16)
      launch_score_prep<uint16_t>(G, n, H, d_v, n_layers, cls_attn, attn_stride_g, attn_stride_h, attn_col0, fa,
                                  a_out, ws.nu, st);
    else
      launch_score_prep<float>(G, n, H, d_v, n_layers, cls_attn, attn_stride_g, attn_stride_h, attn_col0, fa,
                               a_out, ws.nu, st);
    SPIDER_LAUNCHED("score_prep");
  }
  {
    ProfScope ps(KC_ANCHOR_TOPK, st);
    if (n <= 1024)
      anchor_topk_kernel<16><<<G, 64, 0, st>>>(n, n_anchor, a_out, cluster_out, s_out, ws.anc, ws.rest, ws.cw.conv);
    else
      anchor_topk_kernel<kMaxN / 64><<<G, 64, 0, st>>>(n, n_anchor, a_out, cluster_out, s_out, ws.anc, ws.rest,
                                                       ws.cw.conv);
    SPIDER_LAUNCHED("anchor_topk");
  }
  {
    ProfScope ps(KC_MAXSIM, st);
    const float* nu_last = ws.nu + (size_t)last * n;
    const int64_t nu_stride = (int64_t)n_layers * n;
    if (feat_dtype == SPIDER_BF16 && ceil_div(n, 128) * G < kMaxsimBlocks)
      anchor_maxsim_bf16_rows32_kernel<<<dim3(ceil_div(n, 32), G), 256, 0, st>>>(
          n, d_v, n_anchor, fa, last, nu_last, nu_stride, ws.anc, ws.mvec);
    else if (feat_dtype == SPIDER_BF16)
      anchor_maxsim_bf16_kernel<<<dim3(ceil_div(n, 128), G), 256, 0, st>>>(
          n, d_v, n_anchor, fa, last, nu_last, nu_stride, ws.anc, ws.mvec);
    else
      anchor_maxsim_f32_kernel<<<dim3(ceil_div(n, 4), G), 256, 0, st>>>(
          n, d_v, n_anchor, fa, last, nu_last, nu_stride, ws.anc, ws.mvec);
    SPIDER_LAUNCHED("anchor_maxsim");
  }
  hipError_t e = feat_dtype == SPIDER_BF16
                     ? dispatch_cluster<uint16_t>(G, n, d_v, n_anchor, K, kmeans_max_iter, n_layers,
                                                  fa, ws, cluster_out, s_out, m_out, st)
                     : dispatch_cluster<float>(G, n, d_v, n_anchor, K, kmeans_max_iter, n_layers, fa,
                                               ws, cluster_out, s_out, m_out, st);
  SPIDER_REQUIRE(e == hipSuccess, SPIDER_ERR_HIP, "spider_score: cluster kernels failed: %s",
                 hipGetErrorString(e));
  return SPIDER_OK;
}

// ------------------------------------------------------------------ no-allocation variant
// Scratch of spider_score_noalloc: a file-scope device array, so the call needs
// no device allocation (for callers that cannot allocate, e.g. under graph
// capture or in a serving loop).  Every GPU the library runs on holds its own
// copy until the process ends.  Host code never uses the array's name as an
// address: the device address is looked up once per device with
// hipGetSymbolAddress and kept in g_scratch_ptr.
static __device__ __align__(256) uint8_t scratch[SPIDER_SCORE_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of this device's copy of the scratch array (looked up on the
// first call made with that device current).
spider_status scratch_of_current_device(void** out) {
  int dev = -1;
  SPIDER_HIP(hipGetDevice(&dev));
  SPIDER_REQUIRE(dev >= 0 && dev < kMaxDevices, SPIDER_ERR_UNSUPPORTED,
                 "spider_score_noalloc: device %d beyond the %d the library tracks", dev, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    SPIDER_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    SPIDER_REQUIRE(p != nullptr && ((uintptr_t)p % 256) == 0, SPIDER_ERR_HIP,
                   "spider_score_noalloc: scratch address of device %d is not usable", dev);
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return SPIDER_OK;
}
}  // namespace

extern "C" spider_status spider_score_noalloc(int G, int n, int H, int d_v, int n_layers,
                                              const float* cls_attn, int64_t attn_stride_g,
                                              int64_t attn_stride_h, int attn_col0,
                                              const void* const* feats, spider_dtype feat_dtype,
                                              int64_t feat_stride_g, int64_t feat_stride_row,
                                              int feat_row0, int n_anchor, int K, int kmeans_max_iter,
                                              float* a_out, int32_t* cluster_out, float* s_out,
                                              float* m_out, spider_stream stream) {
  clear_error();
  SPIDER_REQUIRE(G >= 1 && n >= 1 && d_v >= 1 && n_layers >= 1 && K >= 1, SPIDER_ERR_INVALID_ARG,
                 "spider_score_noalloc: G, n, d_v, n_layers and K must be >= 1");
  const size_t need = score_ws_layout(G, n, d_v, n_layers, K, nullptr, nullptr);
  SPIDER_REQUIRE(need <= (size_t)SPIDER_SCORE_SCRATCH_BYTES, SPIDER_ERR_WORKSPACE,
                 "spider_score_noalloc: these sizes need %zu bytes of scratch, the static scratch "
                 "holds %zu (use spider_score with a workspace)",
                 need, (size_t)SPIDER_SCORE_SCRATCH_BYTES);
  void* ws = nullptr;
  const spider_status st = scratch_of_current_device(&ws);
  if (st != SPIDER_OK) return st;
  // the kernels write every scratch element they read: stale contents from an
  // earlier call on this device need no clearing
  return spider_score(G, n, H, d_v, n_layers, cls_attn, attn_stride_g, attn_stride_h, attn_col0, feats,
                      feat_dtype, feat_stride_g, feat_stride_row, feat_row0, n_anchor, K, kmeans_max_iter,
                      a_out, cluster_out, s_out, m_out, ws, SPIDER_SCORE_SCRATCH_BYTES, stream);
}
