// Complementary-token selection and decoder-input assembly (Sec. 4.1.2,
// Eq. 2; Sec. 4.1 spatial-order union; Sec. 5 AnyRes per-tile budgets).
//
// select_kernel   grid G x 512, a wave per cluster.  Per tile: cluster sizes
//                 (ballots), quotas N_k computed exactly in integers (a lane
//                 per cluster), each wave marks its cluster's N_k smallest
//                 scores (ties to the lower index) beside the anchors, and the
//                 first wave writes the kept indices ascending.  A block-wide
//                 sort of the keys took 22 us for 576 patches (a barrier per
//                 stage), this takes 12 us.
// assemble_kernel grid (ceil(cap/8), G + B) x 256.  Blocks y < G copy the
//                 kept rows of tile y (when src is given), blocks y >= G copy the text rows of
//                 sample y - G; every block derives its destination row from
//                 the tile counts (a short serial prefix over at most G
//                 values), block (0,0) writes cu_seqlens.  16-byte copies.
#include "common.h"
#include "topk.h"

namespace spider {
namespace {

constexpr int kMaxN = 4096;
constexpr int kMaxK = 8;

// round(p / q) with halves to even; p >= 0, q > 0.
__device__ inline long long rne_div(long long p, long long q) {
  long long t = p / q, r = p - t * q;
  if (2 * r > q || (2 * r == q && (t & 1))) ++t;
  return t;
}

template <int NV>
__global__ void __launch_bounds__(64 * kMaxK) select_kernel(int n, const int32_t* __restrict__ cluster,
                                                            const float* __restrict__ s, int n_cmp, int K,
                                                            int quota_mode, int32_t* __restrict__ idx_out,
                                                            int32_t* __restrict__ count_out, int cap) {
  __shared__ uint8_t keep[64 * NV];
  __shared__ int size[kMaxK];
  const int g = blockIdx.x;
  const int k = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;  // wave k: cluster k
  const int32_t* cl = cluster + (int64_t)g * n;
  const float* sg = s + (int64_t)g * n;
  const int nv = (n + 63) / 64;
  // smallest scores first: the complement of the order key (0 for indices outside the cluster)
  uint32_t key[NV];
  uint64_t mine = 0;  // bit v: index 64 v + lane is in cluster k
  int cnt = 0;
  int cv[NV];
  float x[NV];  // every load first: a load under its own bounds check waits for the one before it
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    cv[v] = cl[min(64 * v + lane, n - 1)];
    x[v] = sg[min(64 * v + lane, n - 1)];
  }
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int i = 64 * v + lane;
    const int c = i < n ? cv[v] : -2;
    const bool in = c == k && k < K;
    key[v] = in ? ~float_order_key(x[v]) : 0u;
    mine |= (uint64_t)in << v;
    cnt += __popcll(__ballot(in));
    if (k == 0 && i < n) keep[i] = c < 0 || c >= K;  // anchors
  }
  if (lane == 0) size[k] = cnt;
  __syncthreads();
  // quotas: lane j of every wave works out cluster j's
  int quota = 0;
  {
    const int sz = lane < K ? size[lane] : 0;
    int D = 0;
    for (int j = 0; j < K; ++j) D += size[j];
    if (n_cmp > 0 && D > 0) {
      if (quota_mode == 0) {
        long long q = sz == 0 ? 0 : rne_div((long long)n_cmp * sz, D);
        if (sz > 0 && q < 1) q = 1;
        quota = (int)(q > sz ? sz : q);
      } else {
        // the largest remainders (ties to the lower cluster) take one more each
        const int budget = n_cmp < D ? n_cmp : D;
        quota = budget * sz / D;
        const int rem = budget * sz % D;
        int used = 0, rank = 0;
        for (int j = 0; j < K; ++j) {
          const int rj = __shfl(rem, j, 64);
          used += __shfl(quota, j, 64);
          rank += rj > rem || (rj == rem && j < lane);
        }
        if (lane < K && rank < budget - used) ++quota;
        if (quota > sz) quota = sz;
      }
    }
  }
  quota = k < K ? __shfl(quota, k, 64) : 0;
  if (quota > 0) {
    const TopK<NV> top = wave_kth_largest<NV>(key, nv, quota);
    int ties = 0;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      if (v >= nv) break;
      const bool in = (mine >> v) & 1;
      const uint64_t eq = __ballot(in && key[v] == top.t);
      if (in && (key[v] > top.t || (key[v] == top.t && ties + lanes_below(eq) < top.ties))) keep[64 * v + lane] = 1;
      ties += __popcll(eq);
    }
  }
  __syncthreads();
  if (k != 0) return;
  // ascending kept indices
  int32_t* out = idx_out + (int64_t)g * cap;
  int run = 0;
  for (int v = 0; v < nv; ++v) {
    const int i = 64 * v + lane;
    const bool on = i < n && keep[i];
    const uint64_t m = __ballot(on);
    const int at = run + lanes_below(m);
    if (on && at < cap) out[at] = i;
    run += __popcll(m);
  }
  const int total = run < cap ? run : cap;
  for (int t = total + lane; t < cap; t += 64) out[t] = -1;
  if (lane == 0) count_out[g] = total;
}

// Destination row of the first kept row of tile g, and of the text rows of
// sample b (g = b*tps + tps), in the packed layout.
__device__ inline int64_t packed_row(const int32_t* count, int g_end, int tps, int n_text) {
  int64_t r = 0;
  for (int t = 0; t < g_end; ++t) r += count[t];
  return r + (int64_t)(g_end / tps) * n_text;
}

__global__ void __launch_bounds__(256) assemble_kernel(
    int G, int tps, int cap, const int32_t* __restrict__ idx, const int32_t* __restrict__ count,
    const uint8_t* __restrict__ src, int64_t src_stride_g_bytes, int row_bytes,
    const uint8_t* __restrict__ text, int n_text, uint8_t* __restrict__ x,
    int32_t* __restrict__ cu_seqlens) {
  const int y = blockIdx.y;
  const int B = G / tps;
  if (blockIdx.x == 0 && y == 0 && threadIdx.x <= B)
    cu_seqlens[threadIdx.x] = (int32_t)packed_row(count, threadIdx.x * tps, tps, n_text);
  const int chunks = row_bytes / 16;
  if (y < G) {
    if (!src) return;
    const int cnt = count[y];
    const int64_t base = packed_row(count, y, tps, n_text);
    for (int r = blockIdx.x * 8; r < min(cnt, blockIdx.x * 8 + 8); ++r) {
      const int i = idx[(int64_t)y * cap + r];
      const uint4* sp = reinterpret_cast<const uint4*>(src + y * src_stride_g_bytes + (int64_t)i * row_bytes);
      uint4* dp = reinterpret_cast<uint4*>(x + (base + r) * row_bytes);
      for (int c = threadIdx.x; c < chunks; c += blockDim.x) dp[c] = sp[c];
    }
  } else {
    const int b = y - G;
    const int64_t base = packed_row(count, (b + 1) * tps, tps, n_text) - n_text;
    for (int r = blockIdx.x * 8; r < min(n_text, blockIdx.x * 8 + 8); ++r) {
      const uint4* sp = reinterpret_cast<const uint4*>(text + ((int64_t)b * n_text + r) * row_bytes);
      uint4* dp = reinterpret_cast<uint4*>(x + (base + r) * row_bytes);
      for (int c = threadIdx.x; c < chunks; c += blockDim.x) dp[c] = sp[c];
    }
  }
}

}  // namespace
}  // namespace spider

using namespace spider;

extern "C" spider_status spider_select(int G, int n, const int32_t* cluster, const float* s,
                                       int n_anchor, int n_cmp, int K, int quota_mode,
                                       int32_t* idx_out, int32_t* count_out, int cap,
                                       int tiles_per_sample, const void* src, int64_t src_stride_g,
                                       int d_model, spider_dtype act_dtype, const void* text,
                                       int n_text, void* x_out, int32_t* cu_seqlens_out,
                                       spider_stream stream) {
  clear_error();
  SPIDER_REQUIRE(G >= 1 && n >= 1, SPIDER_ERR_INVALID_ARG, "spider_select: G and n must be >= 1");
  SPIDER_REQUIRE(n <= kMaxN, SPIDER_ERR_UNSUPPORTED, "spider_select: n = %d exceeds 4096", n);
  SPIDER_REQUIRE(K >= 1 && K <= kMaxK, SPIDER_ERR_UNSUPPORTED, "spider_select: K must be in [1, 8]");
  SPIDER_REQUIRE(quota_mode == 0 || quota_mode == 1, SPIDER_ERR_INVALID_ARG,
                 "spider_select: quota_mode must be 0 (literal) or 1 (exact)");
  SPIDER_REQUIRE(n_anchor >= 0 && n_anchor <= n && n_cmp >= 0, SPIDER_ERR_SHAPE,
                 "spider_select: need 0 <= n_anchor <= n and n_cmp >= 0");
  SPIDER_REQUIRE(cluster && s && idx_out && count_out, SPIDER_ERR_INVALID_ARG,
                 "spider_select: null pointer argument");
  const long long need_cap = std::min<long long>(n, (long long)n_anchor + n_cmp + K);
  SPIDER_REQUIRE(cap >= need_cap, SPIDER_ERR_SHAPE,
                 "spider_select: cap = %d is below min(n, n_anchor + n_cmp + K) = %lld", cap, need_cap);
  SPIDER_REQUIRE(tiles_per_sample >= 1 && G % tiles_per_sample == 0, SPIDER_ERR_SHAPE,
                 "spider_select: tiles_per_sample must divide G");
  // assembly: with src, kept rows and text rows; with x_out but no src, the
  // text rows and boundaries only (the kept rows come from spider_project_kept)
  const bool assemble = src != nullptr || x_out != nullptr;
  size_t esz = 0;
  if (assemble) {
    SPIDER_REQUIRE(act_dtype == SPIDER_F32 || act_dtype == SPIDER_BF16, SPIDER_ERR_INVALID_ARG,
                   "spider_select: bad activation dtype");
    esz = act_dtype == SPIDER_BF16 ? 2 : 4;
    SPIDER_REQUIRE(d_model >= 8 && d_model % 8 == 0, SPIDER_ERR_UNSUPPORTED,
                   "spider_select: d_model must be a positive multiple of 8");
    SPIDER_REQUIRE(!src || (src_stride_g >= (int64_t)n * d_model && src_stride_g % 8 == 0), SPIDER_ERR_SHAPE,
                   "spider_select: src_stride_g must be >= n*d_model and a multiple of 8");
    SPIDER_REQUIRE(x_out && cu_seqlens_out, SPIDER_ERR_INVALID_ARG,
                   "spider_select: assembly needs x_out and cu_seqlens_out");
    SPIDER_REQUIRE(n_text >= 0 && (n_text == 0 || text), SPIDER_ERR_INVALID_ARG,
                   "spider_select: n_text > 0 needs text rows");
    SPIDER_REQUIRE(((uintptr_t)src % 16) == 0 && ((uintptr_t)x_out % 16) == 0 &&
                       (!text || ((uintptr_t)text % 16) == 0),
                   SPIDER_ERR_UNSUPPORTED, "spider_select: src, text and x_out must be 16-byte aligned");
    SPIDER_REQUIRE(G / tiles_per_sample <= 255, SPIDER_ERR_UNSUPPORTED,
                   "spider_select: at most 255 samples per call");
  }
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  {
    ProfScope ps(KC_SELECT, st);
    if (n <= 1024)
      select_kernel<16><<<G, 64 * kMaxK, 0, st>>>(n, cluster, s, n_cmp, K, quota_mode, idx_out, count_out, cap);
    else
      select_kernel<kMaxN / 64><<<G, 64 * kMaxK, 0, st>>>(n, cluster, s, n_cmp, K, quota_mode, idx_out, count_out,
                                                          cap);
    SPIDER_LAUNCHED("select");
  }
  if (assemble) {
    ProfScope ps(KC_ASSEMBLE, st);
    const int B = G / tiles_per_sample;
    const int rows_per_y = std::max(cap, n_text);
    dim3 grid(std::max(1, ceil_div(rows_per_y, 8)), G + B);
    assemble_kernel<<<grid, 256, 0, st>>>(
        G, tiles_per_sample, cap, idx_out, count_out, reinterpret_cast<const uint8_t*>(src),
        src_stride_g * (int64_t)esz, (int)(d_model * esz), reinterpret_cast<const uint8_t*>(text),
        n_text, reinterpret_cast<uint8_t*>(x_out), cu_seqlens_out);
    SPIDER_LAUNCHED("assemble");
  }
  return SPIDER_OK;
}
