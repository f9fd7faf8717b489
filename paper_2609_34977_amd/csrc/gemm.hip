// Decoder GEMMs: out = A[rows] x W^T with W in nn.Linear layout [N, K].
//
// Up to 4 rows (decoding) gemv_kernel streams the weights against the few
// activation rows.  Up to 256 rows (the pruned-prefill regime: a few hundred
// rows against multi-MB weight matrices) gemm_stream_kernel streams every
// weight element from HBM once through an LDS ring into the MFMAs.  More rows
// use gemm_tile_kernel (256-column tiles of 128-256 rows).  Shapes neither of
// the last two takes (N not a multiple of their column tiles, unaligned
// outputs) use gemm_bf16_kernel: 256 threads = 4 waves, block tile BM x BN x
// 32 with v_mfma_f32_16x16x32_bf16 (fp32 accumulation), a wave owning a
// (BM/WGM) x (BN/WGN) sub-tile; a ring of PF register stages of 16-byte
// global loads in flight, double-buffered LDS (row pitch 40 bf16: the
// 16 rows x 16 bytes of a fragment read hit distinct banks), one barrier per
// k-tile.  The kernels may gather A rows through a row list and take a
// grouped launch: up to three problems sharing K (Q over the query rows, K and
// V over all rows) in one grid.  Logical tiles are ordered (group, n-tile,
// k-split, m-tile) and the hardware block id is remapped so consecutive
// logical tiles run on the same XCD (blocks are dispatched round-robin over
// the 8 XCDs) and share its L2.  Epilogues: fp32 split-K partials (summed by
// the consumer kernel in fixed order: deterministic without atomics), the
// fused SwiGLU silu(A Wg^T) * (A Wu^T) rounded to bf16 (dual weights, no split),
// or, unsplit, Q, K and V with their RoPE, scaling and rounding (gemm_qkv_fused).
//
// fp32 path (gemm_f32_kernel): 16x16 or 32x32 FMA tiles through LDS with the same
// group/gather/split/epilogue semantics (used by fp32 workloads).
#include <algorithm>
#include <type_traits>

#include "kernels.h"

namespace spider {
namespace {

constexpr int kNumXcd = 8;

__device__ inline int xcd_remap(int b, int total) {
  const int q = total / kNumXcd, r = total % kNumXcd;
  const int xcd = b % kNumXcd, idx = b / kNumXcd;
  return xcd < r ? xcd * (q + 1) + idx : r * (q + 1) + (xcd - r) * q + idx;
}

template <typename T>
__device__ __forceinline__ T sel3(int gi, T x0, T x1, T x2) {
  return gi == 0 ? x0 : (gi == 1 ? x1 : x2);
}

struct TileCoord {
  int gi, m0, n0, s;
};

__device__ inline TileCoord decode_tile(const GemmArgs& a, int t, int BM, int BN) {
  int gi = 0;
  if (a.ngroups > 1 && t >= a.g[1].tile_begin) gi = 1;
  if (a.ngroups > 2 && t >= a.g[2].tile_begin) gi = 2;
  const int tb = sel3(gi, a.g[0].tile_begin, a.g[1].tile_begin, a.g[2].tile_begin);
  const int tm = sel3(gi, a.g[0].tiles_m, a.g[1].tiles_m, a.g[2].tiles_m);
  int local = t - tb;
  const int m_tile = local % tm;
  local /= tm;
  const int s = local % a.split;
  const int n_tile = local / a.split;
  return {gi, m_tile * BM, n_tile * BN, s};
}

// silu(g) = g / (1 + e^-g) with the hardware reciprocal (1 ulp): the result is
// rounded to bf16 or summed in fp32 afterwards, far coarser than that.
__device__ inline float silu(float g) { return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)); }

// Fields of group gi, read with constant offsets from the kernel arguments
// (a dynamic index into the argument array would be materialised in scratch).
struct GroupView {
  const void* A;
  const int32_t* rows;
  int M;
  const void* W;
  const void* W2;
  void* out;
  int N;
  int64_t ldo, sstride;
};

__device__ __forceinline__ GroupView group_view(const GemmArgs& a, int gi) {
  GroupView v;
  v.A = sel3(gi, a.g[0].A, a.g[1].A, a.g[2].A);
  v.rows = sel3(gi, a.g[0].a_rows, a.g[1].a_rows, a.g[2].a_rows);
  v.M = sel3(gi, a.g[0].M, a.g[1].M, a.g[2].M);
  const int32_t* md = sel3(gi, a.g[0].m_dev, a.g[1].m_dev, a.g[2].m_dev);
  if (md) v.M = min(v.M, *md);
  v.W = sel3(gi, a.g[0].W, a.g[1].W, a.g[2].W);
  v.W2 = sel3(gi, a.g[0].W2, a.g[1].W2, a.g[2].W2);
  v.out = sel3(gi, a.g[0].out, a.g[1].out, a.g[2].out);
  v.N = sel3(gi, a.g[0].N, a.g[1].N, a.g[2].N);
  v.ldo = sel3(gi, a.g[0].ldo, a.g[1].ldo, a.g[2].ldo);
  v.sstride = sel3(gi, a.g[0].split_stride, a.g[1].split_stride, a.g[2].split_stride);
  return v;
}

template <int BM, int BN, int WGM, int WGN, int PF, bool DUAL>
__global__ void __launch_bounds__(256) gemm_bf16_kernel(GemmArgs a) {
  constexpr int BK = 32, PITCH = BK + 8;
  constexpr int BROWS = DUAL ? 2 * BN : BN;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int TM = WTM / 16, TN = WTN / 16;
  constexpr int A_CH = BM * (BK / 8) / 256;
  constexpr int B_CH = BROWS * (BK / 8) / 256;
  static_assert(WGM * WGN == 4, "4 waves");
  static_assert(TM >= 1 && TN >= 1 && WTM % 16 == 0 && WTN % 16 == 0, "wave tile");
  static_assert(A_CH >= 1 && B_CH >= 1 && A_CH * 256 == BM * 4 && B_CH * 256 == BROWS * 4, "chunks");
  __shared__ __attribute__((aligned(16))) uint16_t sA[2][BM * PITCH];
  __shared__ __attribute__((aligned(16))) uint16_t sB[2][BROWS * PITCH];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, lg = lane >> 4;
  const int wm = wave / WGN, wn = wave % WGN;
  const TileCoord tc = decode_tile(a, xcd_remap(blockIdx.x, a.total_tiles), BM, BN);
  const GroupView G = group_view(a, tc.gi);
  const int M = G.M;
  if (tc.m0 >= M) return;  // a device row count below the launch's bound
  const int kbeg = tc.s * a.k_per_split;
  const int kend = min(a.K, kbeg + a.k_per_split);
  const int nt = kend > kbeg ? (kend - kbeg) / BK : 0;

  // per-thread global sources and LDS slots of its chunks (fixed across k)
  const uint16_t* pa[A_CH];
  int ca[A_CH];
#pragma unroll
  for (int c = 0; c < A_CH; ++c) {
    const int lin = c * 256 + tid;
    const int row = lin >> 2, col = (lin & 3) * 8;
    const int gm = tc.m0 + row;
    ca[c] = row * PITCH + col;
    pa[c] = nullptr;
    if (gm < M) {
      const int src = G.rows ? G.rows[gm] : gm;
      pa[c] = reinterpret_cast<const uint16_t*>(G.A) + (int64_t)src * a.lda + kbeg + col;
    }
  }
  const uint16_t* pb[B_CH];
  int cb[B_CH];
#pragma unroll
  for (int c = 0; c < B_CH; ++c) {
    const int lin = c * 256 + tid;
    const int row = lin >> 2, col = (lin & 3) * 8;
    cb[c] = row * PITCH + col;
    const bool second = DUAL && row >= BN;
    const uint16_t* W = reinterpret_cast<const uint16_t*>(second ? G.W2 : G.W);
    pb[c] = W + (int64_t)(tc.n0 + (second ? row - BN : row)) * a.K + kbeg + col;
  }

  floatx4 acc[TM][TN];
  floatx4 acc2[DUAL ? TM : 1][DUAL ? TN : 1];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      acc[i][j] = floatx4{};
      if constexpr (DUAL) acc2[i][j] = floatx4{};
    }

  u32x4 ra[PF][A_CH], rb[PF][B_CH];
  auto load = [&](int t, u32x4 (&xa)[A_CH], u32x4 (&xb)[B_CH]) {
    const int ko = t * BK;
#pragma unroll
    for (int c = 0; c < A_CH; ++c)
      xa[c] = pa[c] ? *reinterpret_cast<const u32x4*>(pa[c] + ko) : u32x4{0, 0, 0, 0};
#pragma unroll
    for (int c = 0; c < B_CH; ++c) xb[c] = *reinterpret_cast<const u32x4*>(pb[c] + ko);
  };
  auto store = [&](int buf, const u32x4 (&xa)[A_CH], const u32x4 (&xb)[B_CH]) {
#pragma unroll
    for (int c = 0; c < A_CH; ++c) *reinterpret_cast<u32x4*>(&sA[buf][ca[c]]) = xa[c];
#pragma unroll
    for (int c = 0; c < B_CH; ++c) *reinterpret_cast<u32x4*>(&sB[buf][cb[c]]) = xb[c];
  };
  auto compute = [&](int buf) {
    const uint16_t* A = sA[buf];
    const uint16_t* B = sB[buf];
    bf16x8 af[TM], bfr[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
      af[i] = __builtin_bit_cast(
          bf16x8, *reinterpret_cast<const u32x4*>(&A[(wm * WTM + i * 16 + l16) * PITCH + lg * 8]));
#pragma unroll
    for (int j = 0; j < TN; ++j)
      bfr[j] = __builtin_bit_cast(
          bf16x8, *reinterpret_cast<const u32x4*>(&B[(wn * WTN + j * 16 + l16) * PITCH + lg * 8]));
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
    if constexpr (DUAL) {
#pragma unroll
      for (int j = 0; j < TN; ++j)
        bfr[j] = __builtin_bit_cast(
            bf16x8,
            *reinterpret_cast<const u32x4*>(&B[(BN + wn * WTN + j * 16 + l16) * PITCH + lg * 8]));
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc2[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bfr[j], acc2[i][j], 0, 0, 0);
    }
  };

  // prologue: tiles 0..PF-1 in flight (tile t lives in register set t % PF),
  // tile 0 in LDS buffer 0
  static_for<0, PF>([&](auto P) {
    if (P.value < nt) load(P.value, ra[P.value], rb[P.value]);
  });
  if (nt > 0) {
    store(0, ra[0], rb[0]);
    if (PF < nt) load(PF, ra[0], rb[0]);
  }
  __syncthreads();
  for (int i0 = 0; i0 < nt; i0 += PF) {
    static_for<0, PF>([&](auto J) {
      constexpr int nx = (J.value + 1) % PF;
      const int i = i0 + J.value;
      if (i < nt) {
        compute(i & 1);
        if (i + 1 < nt) {
          store((i + 1) & 1, ra[nx], rb[nx]);
          if (i + 1 + PF < nt) load(i + 1 + PF, ra[nx], rb[nx]);
        }
        __syncthreads();
      }
    });
  }

  // epilogue: 16x16 D layout, n = lane%16 (weight row), m = 4*(lane/16) + r
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = tc.n0 + wn * WTN + j * 16 + l16;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = tc.m0 + wm * WTM + i * 16 + 4 * lg + r;
        if (m < M) {
          if constexpr (DUAL) {
            const float v = silu(acc[i][j][r]) * acc2[i][j][r];
            reinterpret_cast<uint16_t*>(G.out)[(int64_t)m * G.ldo + n] = f32_to_bf16_bits(v);
          } else {
            reinterpret_cast<float*>(G.out)[tc.s * G.sstride + (int64_t)m * G.ldo + n] =
                acc[i][j][r];
          }
        }
      }
    }
}

// ------------------------------------------------------------------ weight streaming
// gemm_stream_kernel: up to 32*MT (<= 256) rows, the pruned-prefill regime.
// A block takes all rows against 32*NW weight rows: 32*NW output columns, or
// (SwiGLU) 16*NW columns whose gate and up rows alternate in groups of 16, so
// that one 32-row weight tile holds both.
//
// Both operands go global -> LDS with global_load_lds (no register round
// trip) into a ring of STAGES stages; a stage holds BM activation rows and the
// block's weight rows, 64 k each.  Every row is 128 B = eight 16-B chunks;
// chunk c of row r sits in slot c ^ swz(r), so the DMA writes (1 KB per
// instruction, 8 rows of 8 lanes: a whole cache line per 8 lanes) and the MMA
// fragment reads (32 rows, one chunk) are both free of bank conflicts.  Each
// k-block is four v_mfma_f32_32x32x16_bf16 steps; step q takes chunk
// 4*(lane/32) + q on both operands (a consistent permutation of k leaves every
// dot product unchanged).
//
// 4 waves, one per SIMD: wave (wh, mh) takes row tiles [MH mh, MH mh + MH) and, for
// even NW, half wh of the weight tiles.  Three weight tiles do not halve: there
// wave (wh, mh) multiplies k-steps 2 wh and 2 wh + 1 of every k-block with all
// three, and the two k halves are added through LDS at the end.  The weight
// fragment is the MMA's A operand: a lane ends with one activation row and runs
// of four consecutive weight rows.
//
// Pipeline: at iteration kb the block multiplies k-block kb, issues the DMA of
// k-block kb+LEAD, waits until k-block kb+1 has landed and passes one barrier.
// Every iteration issues the same loads (the tail re-reads the last k-block
// into a slot never consumed), so the wait is an exact count of outstanding
// loads; ring slots are compile-time (k-block kb lives in slot kb % STAGES).
// Rows past M read row M-1, weight rows past N read row N-1 (never stored).
//
// What bounds it: the two DMA streams, which add.  SwiGLU of a 4096 x 11008 pair
// at 192 rows (230 blocks of 96 weight rows): 51 us; without the MMAs 50, the
// weights alone 32 (HBM), the activations alone 20 (L2), the MMAs alone 33.
// Deeper rings, rings and waves of their own for each operand, eight waves per
// block and DMAs spread between the MMAs did not change that; what does is
// every CU having a share of the weights (172 blocks of 128 rows took 61 us),
// blocks out of step (below), and few split partials.
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// Softmax statistics of one row piece: max, sum e^(z-max), sum e^(z-max) (z-max).
struct SoftStat {
  float m, s, t;
};

// Merge of two pieces (b.m and a.m finite): rescale both to the larger max.
__device__ __forceinline__ SoftStat soft_merge(SoftStat a, SoftStat b) {
  const float m = fmaxf(a.m, b.m);
  const float da = a.m - m, db = b.m - m;
  const float ea = expf(da), eb = expf(db);
  return {m, ea * a.s + eb * b.s, ea * fmaf(a.s, da, a.t) + eb * fmaf(b.s, db, b.t)};
}

// Tile layout shared by the GEMM kernels: 16-byte chunk c of a 128-byte tile
// row r is stored in slot c ^ ((r >> 1) & 7).  An LDS pass of a 16-byte read
// serves 16 lanes; a fragment read has those lanes on 16 consecutive rows, so
// even and odd rows each cover the 8 slots and the 16 lanes hit 16 distinct
// bank groups (with c ^ (r & 7), rows r and r + 8 collide).
__device__ __forceinline__ int swz(int r) { return (r >> 1) & 7; }

// Cache slot (in rows of d elements) of packed row `row`: its sample's first
// slot plus its position.
__device__ __forceinline__ int64_t cache_slot(const GemmArgs& a, int row) {
  return (int64_t)(a.row_sample ? a.row_sample[row] : row) * a.kv_cap + a.pos[row];
}

// QKV epilogue of the streaming kernel: registers r and r + 8 (r < 8) of acc[i]
// hold the rotate-half partners n0 + 16 wh + 8 (r / 4) + 4 hi + r % 4 and 64
// columns on, of row tile i.  RoPE in place (kind bit 0), then bf16 through LDS:
// [row][column] rows to `out` and to the cache slots of `out2`, or (kind 2) V^T
// rows to `out`, whose rows M..ldvt-1 are written zero, and [row][column] rows to
// the cache.  In LDS column n0 + c is c, its partner 32 + c.
template <int MT, typename Acc, typename Trow>
__device__ __forceinline__ void stream_qkv_epilogue(const GemmArgs& a, const GroupView& G, int kind, void* out2,
                                                    uint8_t* ring, Acc& acc, int m0, int n0, int wh, int rows,
                                                    Trow trow) {
  constexpr int MH = MT / 2, BM = 32 * MT;
  const int tid = threadIdx.x, hi = (tid & 63) >> 5;
  const int c0 = 16 * wh + 4 * hi;  // local column of register 0
  if (kind & 1) {
#pragma unroll
    for (int i = 0; i < MH; ++i) {
      const int m = min(m0 + trow(i), G.M - 1);
      const int p = a.pos[G.rows ? G.rows[m] : m];
      const float4* cs = reinterpret_cast<const float4*>(a.rope + (int64_t)p * 64 + (n0 & 127) + c0);
      float4 x[2][2];
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        x[g][0] = cs[4 * g];
        x[g][1] = cs[4 * g + 1];
      }
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        const float c4[4] = {x[g][0].x, x[g][0].z, x[g][1].x, x[g][1].z};
        const float s4[4] = {x[g][0].y, x[g][0].w, x[g][1].y, x[g][1].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float2 y = rope_rotate(acc[i][4 * g + e], acc[i][4 * g + e + 8], c4[e], s4[e]);
          acc[i][4 * g + e] = y.x;
          acc[i][4 * g + e + 8] = y.y;
        }
      }
    }
  }
  uint16_t* st = reinterpret_cast<uint16_t*>(ring);
  uint16_t* out = reinterpret_cast<uint16_t*>(G.out);
  if (kind == 2 && out) {
    constexpr int VP = BM + 8;
    static_assert(64 * VP * 2 <= 64 * 1024, "V^T tile fits the ring");
#pragma unroll
    for (int i = 0; i < MH; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        st[(32 * (r >> 3) + c0 + 8 * ((r >> 2) & 1) + (r & 3)) * VP + trow(i)] =
            f32_to_bf16_bits(trow(i) < rows ? acc[i][r] : 0.f);
    __syncthreads();
    for (int c = tid; c < 64 * (BM / 8); c += 256) {
      const int col = c / (BM / 8), ch = c % (BM / 8);
      if (m0 + 8 * ch < a.ldvt)
        *reinterpret_cast<u32x4*>(out + (int64_t)(n0 + 64 * (col >> 5) + (col & 31)) * a.ldvt + m0 + 8 * ch) =
            *reinterpret_cast<const u32x4*>(st + col * VP + 8 * ch);
    }
    if (!out2) return;
    __syncthreads();
  }
  constexpr int QP = 72;  // row pitch (bf16)
#pragma unroll
  for (int i = 0; i < MH; ++i)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<uint2*>(st + trow(i) * QP + 32 * (g >> 1) + c0 + 8 * (g & 1)) =
          make_uint2((uint32_t)f32_to_bf16_bits(acc[i][4 * g]) | ((uint32_t)f32_to_bf16_bits(acc[i][4 * g + 1]) << 16),
                     (uint32_t)f32_to_bf16_bits(acc[i][4 * g + 2]) |
                         ((uint32_t)f32_to_bf16_bits(acc[i][4 * g + 3]) << 16));
  __syncthreads();
  for (int c = tid; c < rows * 8; c += 256) {
    const int row = c >> 3, ch = c & 7, m = m0 + row;
    const u32x4 v = *reinterpret_cast<const u32x4*>(st + row * QP + 8 * ch);
    const int col = n0 + 64 * (ch >> 2) + 8 * (ch & 3);
    if (kind != 2 && out) *reinterpret_cast<u32x4*>(out + (int64_t)m * G.ldo + col) = v;
    if (out2)
      *reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(out2) + cache_slot(a, G.rows ? G.rows[m] : m) * G.ldo +
                                col) = v;
  }
}

enum StreamMode { SM_PARTIAL, SM_SWIGLU, SM_LENS, SM_QKV };

template <int NW, int MT, int MODE>
__global__ void __launch_bounds__(256) gemm_stream_kernel(GemmArgs a) {
  constexpr int KB = 64;
  constexpr bool DUAL = MODE == SM_SWIGLU;
  // weights are read once: launches whose blocks take the whole K load them
  // non-temporal (measured 2-6 % faster there, no gain with split-K)
  constexpr bool kWeightNT = MODE != SM_PARTIAL;
  constexpr int BM = 32 * MT, WR = 32 * NW, MH = MT / 2;
  constexpr int BN = DUAL ? WR / 2 : WR;  // output columns per block
  constexpr int A_BYTES = BM * 128;
  constexpr int STAGE_BYTES = A_BYTES + WR * 128;  // activations, then the weight rows
  constexpr int STAGES = 4 * STAGE_BYTES <= 144 * 1024 ? 4 : 3, LEAD = STAGES - 1;
  constexpr int PER_IT = NW + MT;  // DMA instructions per wave per k-block
  constexpr int RING_BYTES = STAGES * STAGE_BYTES;
  static_assert(MT % 2 == 0, "row tiles split over two waves");
  static_assert(RING_BYTES <= 144 * 1024, "LDS of one block");
  __shared__ __attribute__((aligned(1024))) uint8_t ring[RING_BYTES];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hi = lane >> 5, lo = lane & 31;
  const int mh = wave & 1, wh = wave >> 1;
  constexpr bool KHALF = NW % 2 != 0;       // waves share the k-steps, not the weight tiles
  constexpr int NWW = KHALF ? NW : NW / 2;  // weight tiles of a wave, from tile u0
  const int u0 = KHALF ? 0 : NWW * wh;
  const TileCoord tc = decode_tile(a, xcd_remap(blockIdx.x, a.total_tiles), BM, BN);
  const GroupView G = group_view(a, tc.gi);
  const int M = G.M;
  if (tc.m0 >= M) return;  // a device row count below the launch's bound
  const int kbeg = tc.s * a.k_per_split;
  const int kend = min(a.K, kbeg + a.k_per_split);
  const int nkb = kend > kbeg ? (kend - kbeg) / KB : 0;
  // QKV: a block has 32 rotate-half pairs of one head, columns n0 + c and n0 + 64
  // + c; a weight tile holds 16 columns and then their 16 partners
  const int n0 = MODE == SM_QKV ? (tc.n0 & ~127) + (tc.n0 & 127) / 2 : tc.n0;

  // weight DMA: instruction q fills LDS weight rows 8 (NW wave + q) .. + 7; lane
  // l takes row l / 8 of them, slot l % 8
  const uint16_t* pw[NW];
#pragma unroll
  for (int q = 0; q < NW; ++q) {
    const int r = 8 * (NW * wave + q) + (lane >> 3), u = r >> 5, i = r & 31;
    const uint16_t* W = reinterpret_cast<const uint16_t*>(DUAL && i >= 16 ? G.W2 : G.W);
    const int row = DUAL ? n0 + 16 * u + (i & 15)
                         : (MODE == SM_QKV ? n0 + 16 * u + (i & 15) + (i >= 16 ? 64 : 0) : n0 + r);
    pw[q] = W + (int64_t)min(row, G.N - 1) * a.K + kbeg + 8 * ((lane & 7) ^ swz(r));
  }
  // activation DMA: instruction j of this wave fills tile rows 8g..8g+7,
  // g = wave*MT + j; lane l takes row 8g + l/8, slot l%8
  const uint16_t* pa[MT];
#pragma unroll
  for (int j = 0; j < MT; ++j) {
    const int g = wave * MT + j;
    const int r = min(tc.m0 + 8 * g + (lane >> 3), M - 1);
    const int src = G.rows ? G.rows[r] : r;
    const int c = (lane & 7) ^ swz(8 * g + (lane >> 3));
    pa[j] = reinterpret_cast<const uint16_t*>(G.A) + (int64_t)src * a.lda + kbeg + 8 * c;
  }

  floatx16 acc[NWW][MH];
#pragma unroll
  for (int u = 0; u < NWW; ++u)
#pragma unroll
    for (int i = 0; i < MH; ++i) acc[u][i] = floatx16{};

  const uint32_t ring_lds = lds_offset(ring);
  // Blocks with the whole K start at different k-blocks and wrap around: rows are
  // a power-of-two stride apart, and blocks in step ask the same few L2 and
  // memory channels (SwiGLU at 192 rows 55 -> 51 us, at 64 rows 39 -> 34; split
  // launches lose by it: their blocks start apart already)
  const int rot = a.split == 1 && nkb > 0 ? 5 * (tc.n0 / BN) % nkb : 0;
  // DMA instruction p (of PER_IT per wave) of the kb-th k-block into stage S
  auto issue_piece = [&](int kb, auto S, auto P) __attribute__((always_inline)) {
    constexpr int st = decltype(S)::value, p = decltype(P)::value;
    kb += rot;
    kb -= kb >= nkb ? nkb : 0;
    if constexpr (p < NW)
      dma16<kWeightNT>(pw[p] + kb * KB, ring_lds + st * STAGE_BYTES + A_BYTES + (wave * NW + p) * 1024);
    else
      dma16(pa[p - NW] + kb * KB, ring_lds + st * STAGE_BYTES + (wave * MT + p - NW) * 1024);
  };
  // MMAs of the k-block in stage S, the DMA of k-block kbn into stage SN spread
  // between them
  auto compute = [&](auto S, int kbn, auto SN) __attribute__((always_inline)) {
    constexpr int st = decltype(S)::value;
    const uint8_t* wt = ring + st * STAGE_BYTES + A_BYTES + lo * 128;
    const uint8_t* at = ring + st * STAGE_BYTES + (32 * MH * mh + lo) * 128;
    constexpr int NQ = KHALF ? 2 : 4;
    bf16x8 wf[2][NWW], af[2][MH];
    auto frags = [&](int q, bf16x8 (&w)[NWW], bf16x8 (&x)[MH]) __attribute__((always_inline)) {
      const int c = 16 * ((4 * hi + (KHALF ? 2 * wh : 0) + q) ^ swz(lo));
#pragma unroll
      for (int u = 0; u < NWW; ++u)
        w[u] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(wt + (u0 + u) * 32 * 128 + c));
#pragma unroll
      for (int i = 0; i < MH; ++i)
        x[i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(at + i * 32 * 128 + c));
    };
    frags(0, wf[0], af[0]);
    static_for<0, NQ>([&](auto Q) {
      constexpr int q = Q.value;
      if constexpr (q + 1 < NQ) frags(q + 1, wf[(q + 1) & 1], af[(q + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);
      static_for<0, NWW * MH>([&](auto T) {
        constexpr int t = T.value, i = t / NWW, u = t % NWW, n = q * NWW * MH + t, all = NQ * NWW * MH;
        acc[u][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[q & 1][u], af[q & 1][i], acc[u][i], 0, 0, 0);
        constexpr int p0 = n * PER_IT / all, p1 = (n + 1) * PER_IT / all;
        static_for<p0, p1>([&](auto P) { issue_piece(kbn, SN, P); });
        __builtin_amdgcn_sched_barrier(0);
      });
    });
  };

  if (nkb > 0) {
    static_for<0, LEAD>([&](auto S) {
      static_for<0, PER_IT>([&](auto P) { issue_piece(min((int)S.value, nkb - 1), S, P); });
    });
    dma_wait_barrier<(LEAD - 1) * PER_IT>();
    // k-block kb+LEAD goes to the slot that iteration kb-1 consumed (free since
    // its barrier); every iteration issues the same DMAs (the last k-block again
    // at the end), so the count of DMAs still in flight is exact
    auto body = [&](int kb, auto J) {
      constexpr int j = decltype(J)::value;
      compute(J, min(kb + LEAD, nkb - 1), std::integral_constant<int, (j + LEAD) % STAGES>{});
      dma_wait_barrier<(LEAD - 1) * PER_IT>();
    };
    int k0 = 0;
    for (; k0 + STAGES <= nkb; k0 += STAGES)
      static_for<0, STAGES>([&](auto J) { body(k0 + J.value, J); });
    const int rem = nkb - k0;
    static_for<0, STAGES>([&](auto J) {
      if (J.value < rem) body(k0 + J.value, J);
    });
    dma_wait_all();
  }

  // KHALF: add the two k halves.  The wh = 0 wave finishes the first OWN row
  // tiles, the wh = 1 wave the rest, each handing the other's over through LDS.
  // (The selects by wh are written out: a branch per half gets merged into one
  // with a dynamic register index, which lives in scratch.)
  constexpr int OWN = KHALF ? (MH + 1) / 2 : MH;
  static_assert(!KHALF || NW * MT * 4096 <= RING_BYTES, "hand-over fits the ring");
  __syncthreads();  // ring free
  floatx16 fin[NWW][OWN];
  if constexpr (KHALF) {
    auto pick = [&](int u, int j0, int j1) {  // wh ? acc[u][j1] : acc[u][j0]
      floatx16 v;
#pragma unroll
      for (int e = 0; e < 16; ++e) v[e] = wh ? acc[u][j1][e] : acc[u][j0][e];
      return v;
    };
    float* hand = reinterpret_cast<float*>(ring) + mh * MH * NW * 1024 + lane * 4;
#pragma unroll
    for (int j = 0; j < OWN; ++j)
#pragma unroll
      for (int u = 0; u < NW; ++u) {
        const floatx16 v = pick(u, OWN + j < MH ? OWN + j : j, j);
        if (wh || OWN + j < MH) {
#pragma unroll
          for (int q = 0; q < 4; ++q)
            *reinterpret_cast<floatx4*>(hand + (((wh ? j : OWN + j) * NW + u) * 4 + q) * 256) =
                floatx4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
        }
      }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < OWN; ++j)
#pragma unroll
      for (int u = 0; u < NW; ++u) {
        fin[u][j] = pick(u, j, OWN + j < MH ? OWN + j : j);
        if (!wh || OWN + j < MH) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const floatx4 v = *reinterpret_cast<const floatx4*>(hand + (((wh ? OWN + j : j) * NW + u) * 4 + q) * 256);
#pragma unroll
            for (int e = 0; e < 4; ++e) fin[u][j][4 * q + e] += v[e];
          }
        }
      }
    __syncthreads();
  } else {
#pragma unroll
    for (int u = 0; u < NWW; ++u)
#pragma unroll
      for (int j = 0; j < OWN; ++j) fin[u][j] = acc[u][j];
  }
  auto mine = [&](int j) { return !KHALF || !wh || OWN + j < MH; };

  // D layout: weight row 8 g + 4 hi + e of tile u in register 4 g + e, activation
  // row lo of the wave's row tile i.  Results go through LDS so that the stores are whole
  // row pieces.
  const int rows = min(BM, M - tc.m0);
  auto trow = [&](int j) { return 32 * (MH * mh + (KHALF && wh ? OWN : 0) + j) + lo; };
  if constexpr (DUAL) {
    // weight rows 0..15 of a tile are gate rows, 16..31 the up rows of the same
    // columns: registers r and r + 8 of one lane
    constexpr int OPITCH = BN + 8;
    static_assert(BM * OPITCH * 2 <= RING_BYTES, "output tile fits the ring");
    uint16_t* ot = reinterpret_cast<uint16_t*>(ring);
#pragma unroll
    for (int i = 0; i < OWN; ++i)
      if (mine(i)) {
#pragma unroll
        for (int u = 0; u < NWW; ++u)
#pragma unroll
          for (int g = 0; g < 2; ++g) {
            uint32_t w[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
              const int r = 4 * g + 2 * e;
              w[e] = (uint32_t)f32_to_bf16_bits(silu(fin[u][i][r]) * fin[u][i][r + 8]) |
                     ((uint32_t)f32_to_bf16_bits(silu(fin[u][i][r + 1]) * fin[u][i][r + 9]) << 16);
            }
            *reinterpret_cast<uint2*>(ot + trow(i) * OPITCH + 16 * (u0 + u) + 8 * g + 4 * hi) = make_uint2(w[0], w[1]);
          }
      }
    __syncthreads();
    uint16_t* op = reinterpret_cast<uint16_t*>(G.out) + (int64_t)tc.m0 * G.ldo + n0;
    constexpr int PIECES = BN / 8;
    for (int c = tid; c < rows * PIECES; c += 256) {
      const int row = c / PIECES, ch = c % PIECES;
      if (n0 + 8 * ch < G.N)
        *reinterpret_cast<u32x4*>(op + (int64_t)row * G.ldo + 8 * ch) =
            *reinterpret_cast<const u32x4*>(ot + row * OPITCH + 8 * ch);
    }
  } else if constexpr (MODE == SM_QKV) {
    static_assert(NW == 2, "a weight tile per wave half");
    stream_qkv_epilogue<MT>(a, G, sel3(tc.gi, a.g[0].kind, a.g[1].kind, a.g[2].kind),
                            sel3(tc.gi, a.g[0].out2, a.g[1].out2, a.g[2].out2), ring, fin[0], tc.m0, n0, wh, rows, trow);
  } else {
    // fp32 tile, row pitch WR + 4 floats
    constexpr int PITCH = WR + 4;
    static_assert(BM * PITCH * 4 <= RING_BYTES, "fp32 tile fits the ring");
    float* sm = reinterpret_cast<float*>(ring);
#pragma unroll
    for (int i = 0; i < OWN; ++i)
      if (mine(i)) {
#pragma unroll
        for (int u = 0; u < NWW; ++u)
#pragma unroll
          for (int g = 0; g < 4; ++g)
            *reinterpret_cast<floatx4*>(sm + trow(i) * PITCH + 32 * (u0 + u) + 8 * g + 4 * hi) =
                floatx4{fin[u][i][4 * g], fin[u][i][4 * g + 1], fin[u][i][4 * g + 2], fin[u][i][4 * g + 3]};
      }
    __syncthreads();
    if constexpr (MODE == SM_LENS) {
      // each row's 128 logits are reduced by 256/BM threads (64 rows: 4, 128: 2,
      // 192/256: 1) over consecutive column ranges, merged in fixed order
      constexpr int TPR = BM <= 64 ? 4 : (BM <= 128 ? 2 : 1);
      constexpr int CPT = 128 / TPR;
      const int row = tid / TPR, part = tid % TPR;
      SoftStat st{-INFINITY, 0.f, 0.f};
      if (row < BM) {
        const float* z = sm + row * PITCH + part * CPT;
        float mx = -INFINITY;
#pragma unroll
        for (int c = 0; c < CPT; c += 4) {
          const floatx4 v = *reinterpret_cast<const floatx4*>(z + c);
          mx = fmaxf(mx, fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3])));
        }
        float se = 0.f, te = 0.f;
#pragma unroll
        for (int c = 0; c < CPT; c += 4) {
          const floatx4 v = *reinterpret_cast<const floatx4*>(z + c);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float u = v[e] - mx;
            const float x = expf(u);
            se += x;
            te = fmaf(x, u, te);
          }
        }
        st = {mx, se, te};
      }
#pragma unroll
      for (int o = 1; o < TPR; o <<= 1) {
        const SoftStat other{__shfl_xor(st.m, o, 64), __shfl_xor(st.s, o, 64), __shfl_xor(st.t, o, 64)};
        st = (part & o) ? soft_merge(other, st) : soft_merge(st, other);
      }
      const int m = tc.m0 + row;
      if (row < BM && part == 0 && m < M)
        *reinterpret_cast<floatx4*>(reinterpret_cast<float*>(G.out) + ((int64_t)m * G.ldo + n0 / 128) * 4) =
            floatx4{st.m, st.s, st.t, 0.f};
    } else {
      // fp32 partial sums as 16-byte pieces
      float* op = reinterpret_cast<float*>(G.out) + tc.s * G.sstride + (int64_t)tc.m0 * G.ldo + n0;
      constexpr int PIECES = WR / 4;
      for (int c = tid; c < rows * PIECES; c += 256) {
        const int row = c / PIECES, ch = c % PIECES;
        if (n0 + 4 * ch < G.N)
          *reinterpret_cast<floatx4*>(op + (int64_t)row * G.ldo + 4 * ch) =
              *reinterpret_cast<const floatx4*>(sm + row * PITCH + 4 * ch);
      }
    }
  }
}

// ------------------------------------------------------------------ large row counts
// gemm_tile_kernel: the compute-bound regime (more than 256 rows).  A block
// computes BM = 64*MH rows against 256 weight rows (non-dual: 256 output
// columns; dual: the gate and up rows of 128 output columns) over its k range,
// in k-blocks of 64.  4 waves in 2 x 2, wave (mh, nh) owning rows
// [32 MH mh, 32 MH (mh + 1)) and 128 weight rows: non-dual LDS weight rows
// [128 nh, 128 nh + 128); dual output columns [64 nh, 64 nh + 64), i.e. gate
// rows [64 nh, +64) and up rows [128 + 64 nh, +64) of the stage, so every wave
// holds the gate and up sums of the same outputs and the SwiGLU epilogue needs
// no exchange.  Per k-step a wave reads MH + 4 fragments from LDS for 4 MH
// v_mfma_f32_32x32x16_bf16 (acc[i][t]: row tile i, weight tile t).
//
// Operands go global -> LDS by global_load_lds, rows of 128 B whose 16-byte
// chunks are permuted by swz(row): two activation stages, and two (256-row
// tiles) or three weight stages; the order of DMAs, MMAs and the one barrier
// per k-block is described at kblock below.  What bounds it: operand bytes from
// L2 (a block tile of 256 x 256 needs 32 B per clock per CU at the MFMA rate;
// L2 hits measured ~20 B per clock per CU), hence the large tile and the
// L2-friendly order.
// Row tiles entirely past M skip their MMAs; their rows read row M-1.
//
// Tile order: per group, split-major, then GM = 8 row tiles x all column
// tiles in column-major groups, so that the 32 blocks one XCD runs at a time
// (after the XCD remap) share 4 weight tiles and 8 activation tiles in its L2.
// Origin (first row, first output column) of logical tile `local` of a group
// with tm x tn tiles: groups of GM = 8 row tiles, column-major inside a group.
__device__ __forceinline__ int2 tile_origin(int local, int tm, int tn, int BM, int BN) {
  constexpr int GM = 8;
  const int grp = local / (GM * tn);
  const int first_m = grp * GM;
  const int gm = min(tm - first_m, GM);
  const int within = local - grp * GM * tn;
  return make_int2((first_m + within % gm) * BM, (within / gm) * BN);
}

template <int MH, bool DUAL, bool QKV = false>
__global__ void __launch_bounds__(256) gemm_tile_kernel(GemmArgs a) {
  constexpr int KB = 64;
  constexpr int BM = 64 * MH;
  constexpr int A_BYTES = BM * 128, W_BYTES = 256 * 128;
  constexpr int WST = MH <= 3 ? 3 : 2;  // weight stages (activations: two)
  constexpr int OPITCH = 136;  // dual epilogue: bf16 tile BM x 128, padded rows
  constexpr int STAGES_BYTES = 2 * A_BYTES + WST * W_BYTES;
  constexpr int RING_BYTES = STAGES_BYTES > BM * OPITCH * 2 ? STAGES_BYTES : BM * OPITCH * 2;
  // QKV epilogue: RoPE positions of the block's rows past the ring.  They
  // share its LDS array on purpose: with a second __shared__ object the
  // compiler can no longer tell the fragment reads from the in-flight
  // global_load_lds writes and waits for all loads before them.
  constexpr int POS_BYTES = QKV ? BM * 4 : 0;
  static_assert(RING_BYTES + POS_BYTES <= 145 * 1024, "LDS of one block");
  constexpr int A_PER_WAVE = BM / 32;  // DMA instructions (8 rows each) per wave and k-block
  __shared__ __attribute__((aligned(1024))) uint8_t ring[RING_BYTES + POS_BYTES];

  // wave-derived values are uniform: keep them (and the branches on them) scalar
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hi = lane >> 5, lo = lane & 31;
  const int mh = wave >> 1, nh = wave & 1;

  // Block -> (group, split, row tile, column tile).  SwiGLU launches may
  // start with tail pieces: blocks [0, tail_tiles * tail_split) compute piece
  // b % tail_split of the k range of tile (total_tiles + b / tail_split), the
  // rest the whole tiles [0, total_tiles).
  const int n_tail = a.tail_tiles * a.tail_split;
  const bool tail = (int)blockIdx.x < n_tail;
  int gi = 0, s, local, kps;
  if (tail) {
    s = blockIdx.x % a.tail_split;
    local = a.total_tiles + blockIdx.x / a.tail_split;
    kps = a.tail_kps;
  } else {
    const int t = xcd_remap(blockIdx.x - n_tail, a.total_tiles);
    if (a.ngroups > 1 && t >= a.g[1].tile_begin) gi = 1;
    if (a.ngroups > 2 && t >= a.g[2].tile_begin) gi = 2;
    const int tm = sel3(gi, a.g[0].tiles_m, a.g[1].tiles_m, a.g[2].tiles_m);
    const int tn = sel3(gi, a.g[0].tiles_n, a.g[1].tiles_n, a.g[2].tiles_n);
    local = t - sel3(gi, a.g[0].tile_begin, a.g[1].tile_begin, a.g[2].tile_begin);
    s = local / (tm * tn);
    local -= s * tm * tn;
    kps = a.k_per_split;
  }
  const GroupView G = group_view(a, gi);
  const int2 mn = tile_origin(local, sel3(gi, a.g[0].tiles_m, a.g[1].tiles_m, a.g[2].tiles_m),
                              sel3(gi, a.g[0].tiles_n, a.g[1].tiles_n, a.g[2].tiles_n), BM, DUAL ? 128 : 256);
  const int m0 = mn.x, n0 = mn.y;  // first row, first output column

  const int M = G.M;
  const int kbeg = s * kps;
  const int kend = min(a.K, kbeg + kps);
  const int nkb = kend > kbeg ? (kend - kbeg) / KB : 0;
  auto chunk_of = [&](int r) { return 8 * ((lane & 7) ^ swz(r)); };

  // activation DMA: instruction j of this wave fills tile rows 8g..8g+7,
  // g = wave*A_PER_WAVE + j; lane l takes row 8g + l/8, slot l%8
  const uint16_t* pa[A_PER_WAVE];
#pragma unroll
  for (int j = 0; j < A_PER_WAVE; ++j) {
    const int tr = 8 * (wave * A_PER_WAVE + j) + (lane >> 3);
    const int r = min(m0 + tr, M - 1);
    const int src = G.rows ? G.rows[r] : r;
    pa[j] = reinterpret_cast<const uint16_t*>(G.A) + (int64_t)src * a.lda + kbeg + chunk_of(tr);
  }
  // weight DMA: instruction j of this wave fills stage weight rows 8g..8g+7, g = 8*wave + j
  const uint16_t* pw[8];
  // QKV epilogue: RoPE positions of the block's rows, read once at the start
  int* spos = reinterpret_cast<int*>(ring + RING_BYTES);
  const int kind = sel3(gi, a.g[0].kind, a.g[1].kind, a.g[2].kind);
  if constexpr (QKV) {
    if (kind == 1 && tid < BM) {
      const int m = min(m0 + tid, M - 1);
      spos[tid] = a.pos[G.rows ? G.rows[m] : m];
    }
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int wr = 8 * (8 * wave + j) + (lane >> 3);  // 0..255
    const uint16_t* W;
    int row;
    if constexpr (DUAL) {
      W = reinterpret_cast<const uint16_t*>(wr < 128 ? G.W : G.W2);
      row = n0 + (wr & 127);
    } else {
      W = reinterpret_cast<const uint16_t*>(G.W);
      row = n0 + wr;
    }
    pw[j] = W + (int64_t)row * a.K + kbeg + chunk_of(wr);
  }

  // row tiles of this wave that hold rows < M (the rest skip their MMAs)
  const int live = __builtin_amdgcn_readfirstlane(min(MH, max(0, (M - m0 - 32 * MH * mh + 31) / 32)));

  floatx16 acc[MH][4];
#pragma unroll
  for (int i = 0; i < MH; ++i)
#pragma unroll
    for (int u = 0; u < 4; ++u) acc[i][u] = floatx16{};

  // DMA of this wave: piece p of the activations of k-block kb into activation
  // stage S, of the weights into weight stage S
  // LDS offset of the ring (the DMA takes its LDS destination from M0)
  const uint32_t ring_lds = lds_offset(ring);
  auto issue_a = [&](int kb, auto S, auto Pc) {
    constexpr int st = decltype(S)::value, p = decltype(Pc)::value;
    dma16(pa[p] + kb * KB, ring_lds + st * A_BYTES + (wave * A_PER_WAVE + p) * 1024);
  };
  auto issue_w = [&](int kb, auto S, auto Pc) {
    constexpr int st = decltype(S)::value, p = decltype(Pc)::value;
    dma16(pw[p] + kb * KB, ring_lds + 2 * A_BYTES + st * W_BYTES + (8 * wave + p) * 1024);
  };

  // weight tile u of the wave: LDS weight rows wrow(u) .. +31
  auto wrow = [&](int u) {
    if constexpr (DUAL) return (u < 2 ? 64 * nh + 32 * u : 128 + 64 * nh + 32 * (u - 2));
    else return 128 * nh + 32 * u;
  };

  // fragments of k-step q of the k-block in activation stage SA, weight stage SW
  auto frags = [&](auto SA, auto SW, int q, bf16x8 (&w)[4], bf16x8 (&x)[MH]) __attribute__((always_inline)) {
    const uint8_t* at = ring + decltype(SA)::value * A_BYTES + (32 * MH * mh + lo) * 128;
    const uint8_t* wt = ring + 2 * A_BYTES + decltype(SW)::value * W_BYTES + lo * 128;
    const int c = 16 * ((4 * hi + q) ^ swz(lo));
#pragma unroll
    for (int u = 0; u < 4; ++u)
      w[u] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(wt + wrow(u) * 128 + c));
#pragma unroll
    for (int i = 0; i < MH; ++i)
      x[i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(at + i * 32 * 128 + c));
  };
  bf16x8 wf[2][4], af[2][MH];
  // activation pieces of the next k-block issued in step 3 (the rest in the next step 0)
  constexpr int AH = WST == 2 ? A_PER_WAVE : A_PER_WAVE / 2;

  // One k-block kb in stages SA, SW.  On entry buffer 0 holds its step-0 fragments.
  // The barrier comes after step 2's MMAs, once step 3's fragments are in
  // registers: then its stages are free and k-block kb + 1 has landed (its step-0
  // fragments are read while step 3's MMAs run).  DMAs are issued between the
  // MMAs of a step: a burst stalls the wave.
  //  two weight stages (256-row tiles, whose stages fill the LDS): step 3 brings
  //    the activations of k-block kb + 2, the next step 0 its weights, and the
  //    barrier waits for all of them;
  //  three: the activations of kb + 2 in step 3 and the next step 0, the weights of
  //    kb + 2 in steps 1 and 2 of kb, still in flight across the barrier: they have
  //    a k-block longer to arrive.  Measured against two stages: 192-row tiles,
  //    down at 6014 rows 480 -> 422 us, QKV at 705 rows 101 -> 91; 128-row tiles,
  //    gate/up at 384 rows 90 -> 73.
  auto kblock = [&](auto SA, auto SW, int k1, int k2, auto FULL) __attribute__((always_inline)) {
    constexpr int sa = decltype(SA)::value, sw = decltype(SW)::value;
    using SA1 = std::integral_constant<int, 1 - sa>;
    using SW1 = std::integral_constant<int, (sw + 1) % WST>;
    using SW2 = std::integral_constant<int, (sw + 2) % WST>;
    // MMAs of step Q with n DMA pieces spread between their row tiles
    auto mmas = [&](auto Q, auto N, auto piece) __attribute__((always_inline)) {
      constexpr int q = decltype(Q)::value, n = decltype(N)::value;
      static_for<0, MH>([&](auto I) {
        constexpr int i = I.value;
        if (decltype(FULL)::value || i < live) {
#pragma unroll
          for (int u = 0; u < 4; ++u)
            acc[i][u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[q & 1][u], af[q & 1][i], acc[i][u], 0, 0, 0);
        }
        static_for<i * n / MH, (i + 1) * n / MH>(piece);
        __builtin_amdgcn_sched_barrier(0);
      });
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I3 = std::integral_constant<int, 3>;
    auto none = [&](auto) {};
    constexpr int AL = A_PER_WAVE - AH;  // 0 with two weight stages
    frags(SA, SW, 1, wf[1], af[1]);
    __builtin_amdgcn_sched_barrier(0);
    mmas(I0{}, std::integral_constant<int, WST == 2 ? 8 : AL>{}, [&](auto P) __attribute__((always_inline)) {
      if constexpr (WST == 3) issue_a(k1, SA1{}, std::integral_constant<int, AH + P.value>{});
      else issue_w(k1, SW1{}, P);
    });
    frags(SA, SW, 2, wf[0], af[0]);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (WST == 2) mmas(I1{}, I0{}, none);
    else mmas(I1{}, std::integral_constant<int, 4>{}, [&](auto P) __attribute__((always_inline)) { issue_w(k2, SW2{}, P); });
    frags(SA, SW, 3, wf[1], af[1]);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (WST == 2) {
      mmas(I2{}, I0{}, none);
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    } else {
      mmas(I2{}, std::integral_constant<int, 4>{}, [&](auto P) __attribute__((always_inline)) {
        issue_w(k2, SW2{}, std::integral_constant<int, 4 + P.value>{});
      });
      asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    }
    frags(SA1{}, SW1{}, 0, wf[0], af[0]);
    __builtin_amdgcn_sched_barrier(0);
    mmas(I3{}, std::integral_constant<int, AH>{}, [&](auto P) __attribute__((always_inline)) { issue_a(k2, SA, P); });
  };

  if (nkb > 0) {
    using S0 = std::integral_constant<int, 0>;
    using S1 = std::integral_constant<int, 1>;
    const int k1 = min(1, nkb - 1);
    static_for<0, A_PER_WAVE>([&](auto P) { issue_a(0, S0{}, P); });
    static_for<0, 8>([&](auto P) { issue_w(0, S0{}, P); });
    dma_wait_barrier();
    frags(S0{}, S0{}, 0, wf[0], af[0]);
    if constexpr (WST == 3) static_for<0, 8>([&](auto P) { issue_w(k1, S1{}, P); });
    static_for<0, AH>([&](auto P) { issue_a(k1, S1{}, P); });
    // Waves whose row tiles all hold rows < M (every block but the last row
    // tile) run a copy of the loop without the per-tile guards: a branch
    // inside the MMA groups splits the loop into basic blocks, across which
    // the compiler can only wait for every outstanding LDS read.
    auto run = [&](auto FULL) __attribute__((always_inline)) {
      constexpr int UN = WST == 2 ? 2 : 6;  // stages repeat after UN k-blocks
      int kb = 0;
      for (; kb + UN <= nkb; kb += UN)
        static_for<0, UN>([&](auto J) __attribute__((always_inline)) {
          kblock(std::integral_constant<int, J.value % 2>{}, std::integral_constant<int, J.value % WST>{},
                 min(kb + J.value + 1, nkb - 1), min(kb + J.value + 2, nkb - 1), FULL);
        });
      const int rem = nkb - kb;
      static_for<0, UN - 1>([&](auto J) __attribute__((always_inline)) {
        if (J.value < rem)
          kblock(std::integral_constant<int, J.value % 2>{}, std::integral_constant<int, J.value % WST>{},
                 min(kb + J.value + 1, nkb - 1), min(kb + J.value + 2, nkb - 1), FULL);
      });
    };
    if (live == MH) run(std::true_type{});
    else run(std::false_type{});
    dma_wait_all();
  }

  // The MMA takes the weight fragment as A and the activation fragment as B,
  // so its D layout puts one activation row in each lane (row lane % 32 of the
  // 32-row tile) and, in registers 4g..4g+3, the four consecutive output
  // columns 8 g + 4 (lane / 32) + [0, 4) of the 32-column tile: every lane
  // writes 16-byte (fp32) or 8-byte (bf16) row pieces.
  const int lrow = 32 * MH * mh + lo;  // tile row of acc[0][*]; acc[i][*] is 32 i further
  auto quad = [&](const floatx16& v, int g) { return floatx4{v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]}; };
  if constexpr (DUAL) {
    if (tail) {
      // fp32 partial sums of piece s: scratch[s][tail tile][BM][256], gate
      // columns 0..127 then up columns 128..255 of the tile's 128 outputs
      float* sp = reinterpret_cast<float*>(a.scratch) +
                  ((int64_t)s * a.tail_tiles + (local - a.total_tiles)) * BM * 256;
#pragma unroll
      for (int i = 0; i < MH; ++i) {
        const int row = lrow + 32 * i;
        if (m0 + row < M) {
#pragma unroll
          for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int g = 0; g < 4; ++g)
              *reinterpret_cast<floatx4*>(sp + row * 256 + (u >> 1) * 128 + 64 * nh + 32 * (u & 1) + 8 * g + 4 * hi) =
                  quad(acc[i][u], g);
        }
      }
      return;
    }
    // bf16 silu(g) * u staged as a BM x 128 tile, written as 16-byte row pieces
    __syncthreads();
    uint16_t* ot = reinterpret_cast<uint16_t*>(ring);
#pragma unroll
    for (int i = 0; i < MH; ++i)
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          uint32_t w[2];
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const int r = 4 * g + 2 * e;
            w[e] = (uint32_t)f32_to_bf16_bits(silu(acc[i][u][r]) * acc[i][u + 2][r]) |
                   ((uint32_t)f32_to_bf16_bits(silu(acc[i][u][r + 1]) * acc[i][u + 2][r + 1]) << 16);
          }
          *reinterpret_cast<uint2*>(ot + (lrow + 32 * i) * OPITCH + 64 * nh + 32 * u + 8 * g + 4 * hi) =
              make_uint2(w[0], w[1]);
        }
    __syncthreads();
    const int rows = min(BM, M - m0);
    uint16_t* op = reinterpret_cast<uint16_t*>(G.out) + (int64_t)m0 * G.ldo + n0;
    for (int c = tid; c < rows * 16; c += 256) {
      const int row = c >> 4, ch = c & 15;
      *reinterpret_cast<u32x4*>(op + (int64_t)row * G.ldo + 8 * ch) =
          *reinterpret_cast<const u32x4*>(ot + row * OPITCH + 8 * ch);
    }
  } else if constexpr (QKV) {
    // bf16 Q, K or V^T.  The wave's 128 output columns are one head, so the
    // rotate-half partner of column 32u + lo (u = 0, 1) is the same lane's
    // column 32(u + 2) + lo.  First RoPE in place on the accumulators, then
    // one 32-row tile at a time through the wave's own LDS area and out
    // as 16-byte pieces: [row][column] rows of Q and K, or [column][row] for
    // V^T whose rows M..ldvt-1 are written zero.  That loop and its barriers
    // run the same number of times in every wave.
    if (kind == 1) {
      // cos/sin rows of the block's BM rows into the ring (512 B per row, row
      // j at byte 512 j): one burst of global_load_lds, 2 rows per wave
      // instruction, then one wait instead of one table latency per tile
      static_assert(BM * 512 <= RING_BYTES, "RoPE rows fit in the ring");
      __syncthreads();  // spos written, every wave done with the last stage
#pragma unroll
      for (int t = 0; t < BM / 8; ++t) {
        const int row = 2 * (wave + 4 * t) + hi;
        const int p = spos[row];
        __builtin_amdgcn_global_load_lds(reinterpret_cast<const void*>(a.rope + (int64_t)p * 64 + 2 * lo),
                                         (__attribute__((address_space(3))) void*)(ring + 2 * (wave + 4 * t) * 512),
                                         16, 0, 0);
      }
      wait_vmcnt<0>();
      __syncthreads();
#pragma unroll
      for (int i = 0; i < MH; ++i) {
        if (i < live) {
          const uint8_t* cs = ring + (lrow + 32 * i) * 512;
#pragma unroll
          for (int r = 0; r < 16; ++r) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
              const int col = 32 * u + 8 * (r >> 2) + 4 * hi + (r & 3);
              const float2 c = *reinterpret_cast<const float2*>(cs + col * 8);
              const float2 y = rope_rotate(acc[i][u][r], acc[i][u + 2][r], c.x, c.y);
              acc[i][u][r] = y.x;
              acc[i][u + 2][r] = y.y;
            }
          }
        }
      }
    }
    constexpr int QP = 136, VP = 40;  // pitches (bf16) of the two layouts
    constexpr int WAREA = 32 * QP > 128 * VP ? 32 * QP : 128 * VP;
    static_assert(4 * WAREA * 2 <= RING_BYTES, "epilogue staging fits");
    uint16_t* sw = reinterpret_cast<uint16_t*>(ring) + wave * WAREA;
    const int col0 = n0 + 128 * nh;
    uint16_t* out = reinterpret_cast<uint16_t*>(G.out);
    uint16_t* out2 = reinterpret_cast<uint16_t*>(sel3(gi, a.g[0].out2, a.g[1].out2, a.g[2].out2));
    auto put_rows = [&](int i) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *reinterpret_cast<uint2*>(sw + lo * QP + 32 * u + 8 * g + 4 * hi) =
              make_uint2((uint32_t)f32_to_bf16_bits(acc[i][u][4 * g]) |
                             ((uint32_t)f32_to_bf16_bits(acc[i][u][4 * g + 1]) << 16),
                         (uint32_t)f32_to_bf16_bits(acc[i][u][4 * g + 2]) |
                             ((uint32_t)f32_to_bf16_bits(acc[i][u][4 * g + 3]) << 16));
    };
    // [row][column] rows of the tile at rb: to out (Q, K) and to the cache
    auto store_rows = [&](int rb) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int row = (lane >> 4) + 4 * j, ch = lane & 15;
        if (rb + row >= M) continue;
        const u32x4 v = *reinterpret_cast<const u32x4*>(sw + row * QP + 8 * ch);
        if (kind == 1 && out) *reinterpret_cast<u32x4*>(out + (int64_t)(rb + row) * G.ldo + col0 + 8 * ch) = v;
        if (out2)
          *reinterpret_cast<u32x4*>(out2 + cache_slot(a, G.rows ? G.rows[rb + row] : rb + row) * G.ldo + col0 + 8 * ch) = v;
      }
    };
#pragma unroll
    for (int i = 0; i < MH; ++i) {
      const int rb = m0 + 32 * (MH * mh + i);  // first row of the tile
      __syncthreads();
      if (i < live) {
        if (kind == 1) {
          put_rows(i);
        } else {
#pragma unroll
          for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int r = 0; r < 16; ++r)
              sw[(32 * u + 8 * (r >> 2) + 4 * hi + (r & 3)) * VP + lo] =
                  f32_to_bf16_bits(rb + lo < M ? acc[i][u][r] : 0.f);
        }
      }
      __syncthreads();
      if (i < live) {
        if (kind == 1) {
          store_rows(rb);
        } else if (out) {
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const int c = (lane >> 2) + 16 * j, ch = lane & 3;
            if (rb + 8 * ch < a.ldvt)
              *reinterpret_cast<u32x4*>(out + (int64_t)(col0 + c) * a.ldvt + rb + 8 * ch) =
                  *reinterpret_cast<const u32x4*>(sw + c * VP + 8 * ch);
          }
        }
      }
      if (kind == 2 && out2) {  // the values again, as rows for the cache
        __syncthreads();
        if (i < live) put_rows(i);
        __syncthreads();
        if (i < live) store_rows(rb);
      }
    }
  } else {
    // fp32 partial sums as 16-byte row pieces
    float* op = reinterpret_cast<float*>(G.out) + s * G.sstride;
#pragma unroll
    for (int i = 0; i < MH; ++i) {
      const int m = m0 + lrow + 32 * i;
      if (m < M) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int g = 0; g < 4; ++g)
            *reinterpret_cast<floatx4*>(op + (int64_t)m * G.ldo + n0 + wrow(u) + 8 * g + 4 * hi) = quad(acc[i][u], g);
      }
    }
  }
}

// Tail pieces of a SwiGLU launch: gate and up summed over the pieces in
// piece order, out = bf16(silu(g) * u).  Grid (rows of a tile, tail tiles) x 128.
__global__ void __launch_bounds__(128) swiglu_tail_reduce_kernel(GemmArgs a, int BM) {
  const int row = blockIdx.x, tt = blockIdx.y, c = threadIdx.x;
  const int2 mn = tile_origin(a.total_tiles + tt, a.g[0].tiles_m, a.g[0].tiles_n, BM, 128);
  const int m = mn.x + row;
  if (m >= a.g[0].M) return;
  const float* sp = reinterpret_cast<const float*>(a.scratch) + ((int64_t)tt * BM + row) * 256;
  const int64_t piece = (int64_t)a.tail_tiles * BM * 256;
  float g = 0.f, u = 0.f;
  for (int s = 0; s < a.tail_split; ++s) {
    g += sp[s * piece + c];
    u += sp[s * piece + 128 + c];
  }
  reinterpret_cast<uint16_t*>(a.g[0].out)[(int64_t)m * a.g[0].ldo + mn.y + c] = f32_to_bf16_bits(silu(g) * u);
}

// ------------------------------------------------------------------ decode rows
// gemv_kernel: at most 4 rows (greedy decoding, one row per sample).  The
// GEMM is then a stream of weight rows against a few activation rows: one
// block of 4 waves, the MB activation rows staged in LDS once (bf16), each
// wave owning NR weight rows (SwiGLU: NR/2 outputs, their gate and up rows)
// for the whole K.  Lane l takes the 16-byte chunks l, l + 64, ... of every
// row (1 KB per wave instruction, non-temporal: weights are read once), U
// chunks of each row in flight per iteration; fp32 FMAs, then one fixed-order
// wave sum per (row, activation row).  No split-K: the fp32 output is the
// finished sum.  A lane adds its chunks in ascending order whatever NR and U
// are, so they change the speed, not the bits.
// QKV (EPI_DECODE_QKV): NR = 2, the wave's rows are the rotate-half pair
// (c, c + 64) of one head, c = 128 (w / 64) + w % 64 for wave w of the launch.
template <int MB, bool DUAL, int NR, int U, bool QKV = false>
__global__ void __launch_bounds__(256) gemv_kernel(GemmArgs a) {
  static_assert(!QKV || (NR == 2 && !DUAL), "QKV: one rotate-half pair per wave");
  constexpr int NO = DUAL ? NR / 2 : NR;      // outputs per wave
  extern __shared__ __attribute__((aligned(16))) uint16_t xs[];  // [MB][K]
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int gi = 0;
  if (a.ngroups > 1 && (int)blockIdx.x >= a.g[1].tile_begin) gi = 1;
  if (a.ngroups > 2 && (int)blockIdx.x >= a.g[2].tile_begin) gi = 2;
  const GroupView G = group_view(a, gi);
  const int blk = blockIdx.x - sel3(gi, a.g[0].tile_begin, a.g[1].tile_begin, a.g[2].tile_begin);
  const int K = a.K, K8 = K / 8;
  if (a.norm_h) {
    // rows = bf16(h * rsqrt(mean(h^2) + eps) * w), summed in the order of the
    // RMSNorm kernel (float4 pieces tid + 256 j, wave sums, waves (0+1)+(2+3))
    __shared__ float red[4];
    const int K4 = K / 4;
    for (int m = 0; m < MB; ++m) {
      float4 v[8];
      const float4* hr = reinterpret_cast<const float4*>(a.norm_h + (int64_t)(m < G.M ? (G.rows ? G.rows[m] : m) : 0) * K);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int c = threadIdx.x + 256 * j;
        v[j] = (m < G.M && c < K4) ? hr[c] : make_float4(0.f, 0.f, 0.f, 0.f);
      }
      float ss = 0.f;
#pragma unroll
      for (int j = 0; j < 8; ++j)
        ss = fmaf(v[j].x, v[j].x, fmaf(v[j].y, v[j].y, fmaf(v[j].z, v[j].z, fmaf(v[j].w, v[j].w, ss))));
      ss = wave_sum(ss);
      if (lane == 0) red[wave] = ss;
      __syncthreads();
      const float tot = (red[0] + red[1]) + (red[2] + red[3]);
      const float inv = 1.0f / sqrtf(tot / (float)K + a.norm_eps);
      const float4* w4 = reinterpret_cast<const float4*>(a.norm_w);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int c = threadIdx.x + 256 * j;
        if (c < K4) {
          const float4 ww = w4[c];
          uint16_t* o = xs + (int64_t)m * K + 4 * c;
          o[0] = f32_to_bf16_bits(v[j].x * inv * ww.x);
          o[1] = f32_to_bf16_bits(v[j].y * inv * ww.y);
          o[2] = f32_to_bf16_bits(v[j].z * inv * ww.z);
          o[3] = f32_to_bf16_bits(v[j].w * inv * ww.w);
        }
      }
      __syncthreads();  // red is reused by the next row
    }
  } else {
    // activation rows (rows past M are zero)
    for (int c = threadIdx.x; c < MB * K8; c += 256) {
      const int m = c / K8, k8 = c - m * K8;
      u32x4 v = {0, 0, 0, 0};
      if (m < G.M) {
        const int src = G.rows ? G.rows[m] : m;
        v = *reinterpret_cast<const u32x4*>(reinterpret_cast<const uint16_t*>(G.A) + (int64_t)src * a.lda + 8 * k8);
      }
      *reinterpret_cast<u32x4*>(xs + (int64_t)m * K + 8 * k8) = v;
    }
    __syncthreads();
  }
  const int gw = blk * 4 + wave;  // wave of the group
  const int o0 = QKV ? 128 * (gw >> 6) + (gw & 63) : gw * NO;  // first output column of this wave
  if (o0 >= G.N) return;
  const uint16_t* wrow[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int o = QKV ? o0 + 64 * r : min(o0 + (DUAL ? r % NO : r), G.N - 1);
    const uint16_t* W = reinterpret_cast<const uint16_t*>(DUAL && r >= NO ? G.W2 : G.W);
    wrow[r] = W + (int64_t)o * K;
  }
  float acc[NR][MB];
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int m = 0; m < MB; ++m) acc[r][m] = 0.f;
  for (int c0 = lane; c0 < K8; c0 += 64 * U) {
    u32x4 wv[U][NR];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const int c = c0 + 64 * u;
        wv[u][r] = c < K8 ? __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(wrow[r] + 8 * c))
                          : u32x4{0, 0, 0, 0};
      }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int c = c0 + 64 * u;
      if (c >= K8) break;
#pragma unroll
      for (int m = 0; m < MB; ++m) {
        const u32x4 xv = *reinterpret_cast<const u32x4*>(xs + (int64_t)m * K + 8 * c);
        float x[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          x[2 * e] = __uint_as_float(xv[e] << 16);
          x[2 * e + 1] = __uint_as_float(xv[e] & 0xFFFF0000u);
        }
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            acc[r][m] = fmaf(__uint_as_float(wv[u][r][e] << 16), x[2 * e], acc[r][m]);
            acc[r][m] = fmaf(__uint_as_float(wv[u][r][e] & 0xFFFF0000u), x[2 * e + 1], acc[r][m]);
          }
      }
    }
  }
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int m = 0; m < MB; ++m) acc[r][m] = wave_sum(acc[r][m]);
  if (lane != 0) return;
  if constexpr (QKV) {
    const int kind = sel3(gi, a.g[0].kind, a.g[1].kind, a.g[2].kind);
#pragma unroll
    for (int m = 0; m < MB; ++m) {
      if (m >= G.M) break;
      const int p = a.pos[m];
      float y0 = acc[0][m], y1 = acc[1][m];
      if (kind & 1) {
        const float2 cs = a.rope[(int64_t)p * 64 + (o0 & 63)];
        const float2 y = rope_rotate(y0, y1, cs.x, cs.y);
        y0 = y.x;
        y1 = y.y;
      }
      uint16_t* dst = reinterpret_cast<uint16_t*>(G.out) + ((kind & 2) ? (int64_t)m * a.kv_cap + p : m) * G.ldo;
      dst[o0] = f32_to_bf16_bits(y0);
      dst[o0 + 64] = f32_to_bf16_bits(y1);
    }
    return;
  }
#pragma unroll
  for (int q = 0; q < NO; ++q) {
    const int o = o0 + q;
    if (o >= G.N) break;
#pragma unroll
    for (int m = 0; m < MB; ++m) {
      if (m >= G.M) break;
      if constexpr (DUAL)
        reinterpret_cast<uint16_t*>(G.out)[(int64_t)m * G.ldo + o] =
            f32_to_bf16_bits(silu(acc[q][m]) * acc[q + NO][m]);
      else if (a.epilogue == EPI_RESIDUAL_F32)
        reinterpret_cast<float*>(G.out)[(int64_t)m * G.ldo + o] += acc[q][m];
      else
        reinterpret_cast<float*>(G.out)[(int64_t)m * G.ldo + o] = acc[q][m];
    }
  }
}

// ------------------------------------------------------------------ fp32
// 16 R x 16 R outputs per block, R x R per thread, k in chunks of 64 through LDS
// (the next chunk's loads in flight behind the FMAs); every output adds its k
// in ascending order.  A small problem is one latency per chunk, so chunks of 64
// instead of 16 (Q, K, V, O and down of 48 rows, d = 128: 9.5 -> 6.8 us a launch on
// average); R = 2 halves the LDS reads per FMA
// where the grid still covers the CUs.
template <bool DUAL, int R>
__global__ void __launch_bounds__(256) gemm_f32_kernel(GemmArgs a) {
  constexpr int T = 16 * R, KC = 64, PITCH = KC + 4;
  __shared__ __attribute__((aligned(16))) float sA[T][PITCH];
  __shared__ __attribute__((aligned(16))) float sB[DUAL ? 2 * T : T][PITCH];
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  const TileCoord tc = decode_tile(a, blockIdx.x, T, T);
  const GroupView G = group_view(a, tc.gi);
  if (tc.m0 >= G.M) return;  // a device row count below the launch's bound
  const int K = a.K;
  // rows ty, ty + 16, .. of the tile, elements tx + 16 e of a chunk
  const float* pa[R];
  const float* pb[DUAL ? 2 * R : R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int m = min(tc.m0 + ty + 16 * r, G.M - 1), n = min(tc.n0 + ty + 16 * r, G.N - 1);
    pa[r] = reinterpret_cast<const float*>(G.A) + (int64_t)(G.rows ? G.rows[m] : m) * a.lda;
    pb[r] = reinterpret_cast<const float*>(G.W) + (int64_t)n * K;
    if constexpr (DUAL) pb[R + r] = reinterpret_cast<const float*>(G.W2) + (int64_t)n * K;
  }
  constexpr int NB = DUAL ? 2 * R : R;
  float ra[R][4], rb[NB][4];
  auto load = [&](int k0) {
    // (past K: any element of the row; the terms are left out below.  A load
    // under a bounds check of its own would wait for the one before it.)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int k = min(k0 + tx + 16 * e, K - 1);
#pragma unroll
      for (int r = 0; r < R; ++r) ra[r][e] = pa[r][k];
#pragma unroll
      for (int r = 0; r < NB; ++r) rb[r][e] = pb[r][k];
    }
  };
  float acc[R][R] = {}, acc2[DUAL ? R : 1][R] = {};
  load(0);
  for (int k0 = 0; k0 < K; k0 += KC) {
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 4; ++e) {
#pragma unroll
      for (int r = 0; r < R; ++r) sA[ty + 16 * r][tx + 16 * e] = ra[r][e];
#pragma unroll
      for (int r = 0; r < NB; ++r) sB[ty + 16 * r][tx + 16 * e] = rb[r][e];
    }
    __syncthreads();
    if (k0 + KC < K) load(k0 + KC);
    const int kn = min(KC, K - k0);
    auto step = [&](int kk) {
      floatx4 x[R], w[NB];
#pragma unroll
      for (int r = 0; r < R; ++r) x[r] = *reinterpret_cast<const floatx4*>(&sA[ty + 16 * r][kk]);
#pragma unroll
      for (int r = 0; r < NB; ++r) w[r] = *reinterpret_cast<const floatx4*>(&sB[tx + 16 * r][kk]);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (kk + e >= kn) break;  // K not a multiple of 4: no extra terms
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
          for (int j = 0; j < R; ++j) {
            acc[i][j] = fmaf(x[i][e], w[j][e], acc[i][j]);
            if constexpr (DUAL) acc2[i][j] = fmaf(x[i][e], w[R + j][e], acc2[i][j]);
          }
      }
    };
    if (kn == KC) {
#pragma unroll 4
      for (int kk = 0; kk < KC; kk += 4) step(kk);
    } else {
      for (int kk = 0; kk < kn; kk += 4) step(kk);
    }
  }
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const int m = tc.m0 + ty + 16 * i, n = tc.n0 + tx + 16 * j;
      if (m >= G.M || n >= G.N) continue;
      if constexpr (DUAL)
        reinterpret_cast<float*>(G.out)[(int64_t)m * G.ldo + n] = silu(acc[i][j]) * acc2[i][j];
      else
        reinterpret_cast<float*>(G.out)[tc.s * G.sstride + (int64_t)m * G.ldo + n] = acc[i][j];
    }
}

constexpr int kTargetBlocks = 256;

// Split-K of the tile and LDS-staged kernels.  Tile kernel (one block per CU):
// the largest split whose grid still fits in one wave of blocks; a second
// partial wave costs more than it hides.  LDS-staged kernel: split until the
// grid covers the chip.  Both double, never past split_max: it need not be a power
// of two, and the partial sums have room for that many slabs and no more.
int choose_split(int tiles, int K, int split_max, int kgran, bool one_wave) {
  int split = 1;
  if (one_wave) {
    while (2 * split <= split_max && tiles * split * 2 <= kTargetBlocks && K / (kgran * split * 2) >= 4) split *= 2;
  } else {
    while (2 * split <= split_max && tiles * split < kTargetBlocks && K / (kgran * split * 2) >= 4) split *= 2;
  }
  return split;
}

// Weight tiles per block and split of a streaming launch: the least of
//   waves of blocks x (k-blocks of a block x (NW + kStreamAct) + kStreamFixed)
//   + split x output columns x kStreamPartial
// in units of one 32-row weight tile's k-block (0.14 us on a CU): the 192
// activation rows of a k-block cost about 1.7 weight tiles, a block's prologue
// and epilogue about 20, and the partial sums are written here and read again by
// the next kernel.  At 192 rows it takes, per launch, NW 3 for SwiGLU (51 us; 4:
// 61), NW 2 and split 4 for O (16.2 us; 4 and 8: 17.3 and a norm 1 us longer), NW
// 4 and split 8 for down (30 us; 2 and 4: 36).  It depends on the columns and K
// only, never on the row count: launches sized for a row bound give the bits of
// launches sized for the live rows.
constexpr double kStreamAct = 1.7, kStreamFixed = 20.0, kStreamPartial = 5.2 / 4096;

struct StreamChoice {
  int nw, split;
};

StreamChoice stream_choice(const GemmArgs& a, int split_max, bool dual) {
  StreamChoice best{4, 1};
  double best_cost = 1e300;
  const int nkb = a.K / 64;
  for (int nw : {4, 3, 2}) {
    if (nw == 3 && !dual) continue;  // the hand-over of the k halves costs a short block more than it saves
    const int bn = dual ? 16 * nw : 32 * nw;
    int tiles = 0;
    double cols = 0;
    for (int i = 0; i < a.ngroups; ++i) {
      tiles += ceil_div(a.g[i].N, bn);
      cols += a.g[i].N;
    }
    for (int split = 1; split <= (dual ? 1 : split_max) && (split == 1 || nkb / split >= 4); ++split) {
      const double cost = ceil_div(tiles * split, kTargetBlocks) * (ceil_div(nkb, split) * (nw + kStreamAct) + kStreamFixed) +
                          (dual ? 0.0 : split * cols * kStreamPartial);
      if (cost < best_cost) {
        best_cost = cost;
        best = StreamChoice{nw, split};
      }
    }
  }
  return best;
}

void fill_tiles(GemmArgs& a, int BM, int BN) {
  int t = 0;
  for (int i = 0; i < a.ngroups; ++i) {
    GemmGroup& g = a.g[i];
    g.tiles_m = ceil_div(g.M, BM);
    g.tiles_n = ceil_div(g.N, BN);  // only the streaming kernel takes a ragged last tile
    g.tile_begin = t;
    t += g.tiles_m * g.tiles_n * a.split;
  }
  a.total_tiles = t;
}

int tiles_for(const GemmArgs& a, int BM, int BN) {
  int t = 0;
  for (int i = 0; i < a.ngroups; ++i) t += ceil_div(a.g[i].M, BM) * (a.g[i].N / BN);
  return t;
}

template <int BM, int BN, int WGM, int WGN, bool DUAL>
void launch_cfg(const GemmArgs& a, hipStream_t st) {
  gemm_bf16_kernel<BM, BN, WGM, WGN, 4, DUAL><<<a.total_tiles, 256, 0, st>>>(a);
}

template <int NW, int MODE>
void launch_stream(const GemmArgs& a, int maxM, hipStream_t st) {
  switch (std::max(1, ceil_div(maxM, 64))) {
    case 1: gemm_stream_kernel<NW, 2, MODE><<<a.total_tiles, 256, 0, st>>>(a); break;
    case 2: gemm_stream_kernel<NW, 4, MODE><<<a.total_tiles, 256, 0, st>>>(a); break;
    case 3: gemm_stream_kernel<NW, 6, MODE><<<a.total_tiles, 256, 0, st>>>(a); break;
    default: gemm_stream_kernel<NW, 8, MODE><<<a.total_tiles, 256, 0, st>>>(a); break;
  }
}

// The streaming kernel stores 16-byte pieces of output rows and multiplies whole
// 64-k blocks.
bool stream_fits(const GemmArgs& a, int maxM, bool dual) {
  if (maxM > 256 || a.K % 64) return false;
  const int per16 = dual ? 8 : 4;
  for (int i = 0; i < a.ngroups; ++i) {
    const GemmGroup& g = a.g[i];
    if (g.N % 16 || reinterpret_cast<uintptr_t>(g.out) % 16 || g.ldo % per16 || g.split_stride % per16) return false;
  }
  return true;
}

// More than 256 rows: gemm_tile_kernel when the shapes fit it (N a multiple of
// the block's output columns, K of 64, 16-byte aligned bf16 output rows for
// the SwiGLU epilogue).  The row tile (256, 192 or 128) minimises the number
// of waves of blocks (one block per CU) times the cost of a block; split-K only
// fills a grid that would leave CUs idle.  A full wave at K = 5120 was measured at
// 140, 97 and about 80 us (320 : 222 : 183).  The costs 320 : 240 : 190 lean to the
// larger tiles, which read less in launches of many waves.  Measured where the two
// disagree, one layer, leaned and not: QKV of 3136 rows 722 and 751 us, of 6200
// 1517 and 1544, of 2350 (d = 5120) 783 and 808; gate/up loses by it at a split
// last wave: 600 rows 341 and 331, 1400 rows 691 and 678, 1050 (d = 5120) 802 and
// 782, 6014 rows 2663 and 2656.
bool tile_path_fits(const GemmArgs& a, bool dual) {
  if (a.K % 64) return false;
  for (int i = 0; i < a.ngroups; ++i) {
    const GemmGroup& g = a.g[i];
    if (g.N % (dual ? 128 : 256)) return false;
    if (dual && (reinterpret_cast<uintptr_t>(g.out) % 16 || g.ldo % 8)) return false;
    // fp32 partial sums leave as 16-byte row pieces
    if (!dual && a.epilogue != EPI_QKV_BF16 &&
        (reinterpret_cast<uintptr_t>(g.out) % 16 || g.ldo % 4 || g.split_stride % 4))
      return false;
  }
  return true;
}

struct TileChoice {
  int mh, split, tail, tail_split;
  double cost;
};

TileChoice tile_choice(const GemmArgs& a, int split_max, bool dual) {
  const int bn = dual ? 128 : 256;
  TileChoice best{4, 1, 0, 0, 1e300};
  for (int mh : {4, 3, 2}) {
    const int bm = 64 * mh;
    const int tiles = tiles_for(a, bm, bn);
    const int split = dual ? 1 : choose_split(tiles, a.K, split_max, 64, true);
    const double block = mh == 4 ? 320 : (mh == 3 ? 240 : 190);
    double cost = (double)ceil_div(tiles * split, kTargetBlocks) * block / split;
    int tail = 0, ts = 0;
    // SwiGLU, one group: a last wave at most a quarter full is split along k
    // into pieces that run beside the first wave (fp32 partials in scratch)
    const int r = tiles % kTargetBlocks;
    if (dual && a.ngroups == 1 && tiles > kTargetBlocks && r > 0 && r <= kTargetBlocks / 4 && a.scratch) {
      const int nkb = a.K / 64;
      int s = std::min(16, std::min(nkb / 2, kTargetBlocks / r));
      while (s >= 2 && (size_t)r * s * bm * 256 * 4 > a.scratch_bytes) --s;
      if (s >= 2) {
        const double c2 = (double)(tiles / kTargetBlocks) * block + block * (1.0 / s + 0.1);
        if (c2 < cost) {
          cost = c2;
          tail = r;
          ts = s;
        }
      }
    }
    if (cost < best.cost) best = TileChoice{mh, split, tail, ts, cost};
  }
  return best;
}

hipError_t launch_tile(GemmArgs& a, int split_max, bool dual, hipStream_t st) {
  const int bn = dual ? 128 : 256;
  const TileChoice tc = tile_choice(a, split_max, dual);
  const int best_mh = tc.mh, best_split = tc.split, best_tail = tc.tail, best_ts = tc.tail_split;
  const bool qkv = a.epilogue == EPI_QKV_BF16;
  a.split = best_split;
  a.k_per_split = ceil_div(a.K / 64, a.split) * 64;
  fill_tiles(a, 64 * best_mh, bn);
  a.tail_tiles = best_tail;
  a.tail_split = best_ts;
  a.tail_kps = best_ts ? ceil_div(a.K / 64, best_ts) * 64 : 0;
  a.total_tiles -= best_tail;  // whole tiles; the tail tiles follow them in logical order
  const int blocks = a.total_tiles + best_tail * best_ts;
  if (blocks == 0) return hipSuccess;
  switch (best_mh * 2 + (dual ? 1 : 0)) {
    case 8: qkv ? gemm_tile_kernel<4, false, true><<<blocks, 256, 0, st>>>(a)
                : gemm_tile_kernel<4, false><<<blocks, 256, 0, st>>>(a); break;
    case 9: gemm_tile_kernel<4, true><<<blocks, 256, 0, st>>>(a); break;
    case 6: qkv ? gemm_tile_kernel<3, false, true><<<blocks, 256, 0, st>>>(a)
                : gemm_tile_kernel<3, false><<<blocks, 256, 0, st>>>(a); break;
    case 7: gemm_tile_kernel<3, true><<<blocks, 256, 0, st>>>(a); break;
    case 4: qkv ? gemm_tile_kernel<2, false, true><<<blocks, 256, 0, st>>>(a)
                : gemm_tile_kernel<2, false><<<blocks, 256, 0, st>>>(a); break;
    default: gemm_tile_kernel<2, true><<<blocks, 256, 0, st>>>(a); break;
  }
  if (best_tail) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    swiglu_tail_reduce_kernel<<<dim3(64 * best_mh, best_tail), 128, 0, st>>>(a, 64 * best_mh);
  }
  return hipGetLastError();
}

// At most 4 rows: gemv_kernel, no split (the output holds the finished sums).
// Decode rows: one weight row per wave with 16 chunks in flight (SwiGLU: the
// gate and up rows of one output, 8 chunks each), four waves per block.  With
// 4 rows (2 outputs) and 4 chunks per wave, a wave fetched its rows in several
// dependent rounds and the O and down projections filled only 256 blocks:
// 3.40 ms per decode step then, 3.13 now; 32 / 16 chunks (more registers,
// fewer waves per SIMD) measured 3.55 ms.
hipError_t launch_gemv(GemmArgs& a, int maxM, bool dual, hipStream_t st) {
  a.split = 1;
  a.k_per_split = a.K;
  const bool qkv = a.epilogue == EPI_DECODE_QKV;
  const int per_block = qkv ? 8 : 4;  // outputs per block
  int t = 0;
  for (int i = 0; i < a.ngroups; ++i) {
    a.g[i].tile_begin = t;
    t += ceil_div(a.g[i].N, per_block);
  }
  a.total_tiles = t;
  if (t == 0 || maxM == 0) return hipSuccess;
  const int mb = maxM <= 1 ? 1 : (maxM <= 2 ? 2 : 4);
  const size_t sh = (size_t)mb * a.K * 2;
  if (qkv) {
    switch (mb) {
      case 1: gemv_kernel<1, false, 2, 8, true><<<t, 256, sh, st>>>(a); break;
      case 2: gemv_kernel<2, false, 2, 8, true><<<t, 256, sh, st>>>(a); break;
      default: gemv_kernel<4, false, 2, 8, true><<<t, 256, sh, st>>>(a); break;
    }
    return hipGetLastError();
  }
  if (!dual) {
    switch (mb) {
      case 1: gemv_kernel<1, false, 1, 16><<<t, 256, sh, st>>>(a); break;
      case 2: gemv_kernel<2, false, 1, 16><<<t, 256, sh, st>>>(a); break;
      default: gemv_kernel<4, false, 1, 16><<<t, 256, sh, st>>>(a); break;
    }
    return hipGetLastError();
  }
  switch (mb) {
    case 1: gemv_kernel<1, true, 2, 8><<<t, 256, sh, st>>>(a); break;
    case 2: gemv_kernel<2, true, 2, 8><<<t, 256, sh, st>>>(a); break;
    default: gemv_kernel<4, true, 2, 8><<<t, 256, sh, st>>>(a); break;
  }
  return hipGetLastError();
}

}  // namespace

namespace {
bool gemv_fits(int maxM, int K) { return maxM <= 4 && K % 8 == 0 && (size_t)4 * K * 2 <= 160 * 1024; }
int max_rows(const GemmArgs& a) {
  int maxM = 0;
  for (int i = 0; i < a.ngroups; ++i) maxM = std::max(maxM, a.g[i].M);
  return maxM;
}
// a group whose rows come from a device count (streaming, LDS-staged, fp32 kernels only)
bool has_row_count(const GemmArgs& a) {
  for (int i = 0; i < a.ngroups; ++i)
    if (a.g[i].m_dev) return true;
  return false;
}
}  // namespace

bool gemm_qkv_fused(const GemmArgs& a, int split_max) {
  const int maxM = max_rows(a);
  if (gemv_fits(maxM, a.K) || a.K % 64) return false;
  for (int i = 0; i < a.ngroups; ++i)
    if (a.g[i].N % 128) return false;
  if (maxM <= 256) return true;
  return !has_row_count(a) && tile_path_fits(a, false) && tile_choice(a, split_max, false).split == 1;
}

// Few queries (only the text rows, say) beside many keys and values: as tiles of
// the same launch they may open a wave of blocks of their own, alone the
// streaming kernel takes them in 24 us (64 rows, d = 4096) to 46 us (256).  Q goes
// apart up to two 64-row steps of it, where the launch without it is enough
// cheaper.  The line is measured, QKV per layer in one launch and in two, d = 4096:
// 64 queries of 1921 rows 153 and 141 us, of 4417 291 and 285, of 5953 365 and 365, of
// 6144 409 and 374; 128 of 2945 rows 203 and 205 (not apart), of 4417 291 and 291, of
// 6144 411 and 381; 192 of 4417 290 and 301, of 6144 412 and 389; 256 of 6014 372 and 391.
// A wave costs 190 to 320 here and less in truth (its few blocks have the chip to
// themselves), hence the margin: 64 queries of 2049 rows take 152 us in one launch, 174
// in two.  Both launches run unsplit, whatever split the keys and values alone
// would have taken.
bool gemm_qkv_q_apart(const GemmArgs& a, int split_max) {
  if (a.ngroups != 3 || a.g[0].M <= 4 || a.g[0].M > 128 || max_rows(a) <= 256 || !gemm_qkv_fused(a, split_max))
    return false;
  GemmArgs kv = a;
  kv.ngroups = 2;
  kv.g[0] = a.g[1];
  kv.g[1] = a.g[2];
  const double q_cost = 100 + 40 * ceil_div(a.g[0].M, 64);
  return tile_choice(kv, 1, false).cost + q_cost < tile_choice(a, 1, false).cost;
}

hipError_t launch_gemm_bf16(GemmArgs& a, int split_max, hipStream_t st) {
  const int maxM = max_rows(a);
  if (a.epilogue == EPI_LENS_STATS) {
    if (maxM > 256 || a.K % 64) return hipErrorInvalidValue;
    for (int i = 0; i < a.ngroups; ++i)
      if (a.g[i].N % 128) return hipErrorInvalidValue;
    a.split = 1;
    a.k_per_split = a.K;
    fill_tiles(a, 256, 128);
    if (a.total_tiles == 0) return hipSuccess;
    launch_stream<4, SM_LENS>(a, maxM, st);
    return hipGetLastError();
  }
  const bool dual = a.epilogue == EPI_SWIGLU;
  const bool gemv_ok = gemv_fits(maxM, a.K);
  if (a.epilogue == EPI_QKV_BF16) {
    // whole sums in one block, whole heads, 16-byte stores.  (Whether a split
    // would pay is the caller's question to gemm_qkv_fused, of all groups; this may
    // be some of them.)
    if (!gemm_qkv_fused(a, 1) || !a.rope || !a.pos) return hipErrorInvalidValue;
    for (int i = 0; i < a.ngroups; ++i) {
      const GemmGroup& g = a.g[i];
      if (reinterpret_cast<uintptr_t>(g.out) % 16 || reinterpret_cast<uintptr_t>(g.out2) % 16 || g.ldo % 8 ||
          (g.kind != 1 && g.kind != 2) || (g.out2 && a.kv_cap < 1))
        return hipErrorInvalidValue;
      if (g.kind == 2 && g.out && (a.ldvt % 32 || a.ldvt < g.M)) return hipErrorInvalidValue;
    }
    if (maxM > 256) return launch_tile(a, 1, false, st);
    a.split = 1;
    a.k_per_split = a.K;
    fill_tiles(a, 256, 64);
    if (a.total_tiles == 0) return hipSuccess;
    launch_stream<2, SM_QKV>(a, maxM, st);
    return hipGetLastError();
  }
  if (a.epilogue == EPI_RESIDUAL_F32 || a.epilogue == EPI_DECODE_QKV || a.norm_h) {
    // only the decode-row kernel applies a residual or cache epilogue or a
    // fused norm (the norm holds a row of at most 8192 floats in registers)
    if (!gemv_ok || (a.norm_h && (!a.norm_w || a.K > 8192))) return hipErrorInvalidValue;
  }
  if (a.epilogue == EPI_DECODE_QKV) {
    if (!a.rope || !a.pos || a.kv_cap < 1) return hipErrorInvalidValue;
    for (int i = 0; i < a.ngroups; ++i)
      if (a.g[i].N % 128 || a.g[i].a_rows) return hipErrorInvalidValue;
  }
  if ((gemv_ok || (maxM > 256 && tile_path_fits(a, dual))) && has_row_count(a)) return hipErrorInvalidValue;
  if (gemv_ok) return launch_gemv(a, maxM, dual, st);
  if (maxM > 256 && tile_path_fits(a, dual)) return launch_tile(a, split_max, dual, st);
  if (stream_fits(a, maxM, dual)) {
    const StreamChoice sc = stream_choice(a, split_max, dual);
    a.split = sc.split;
    a.k_per_split = ceil_div(a.K / 64, a.split) * 64;
    fill_tiles(a, 256, (dual ? 16 : 32) * sc.nw);
    if (a.total_tiles == 0) return hipSuccess;
    switch (sc.nw * 2 + (dual ? 1 : 0)) {
      case 4: launch_stream<2, SM_PARTIAL>(a, maxM, st); break;
      case 5: launch_stream<2, SM_SWIGLU>(a, maxM, st); break;
      case 7: launch_stream<3, SM_SWIGLU>(a, maxM, st); break;
      case 8: launch_stream<4, SM_PARTIAL>(a, maxM, st); break;
      default: launch_stream<4, SM_SWIGLU>(a, maxM, st); break;
    }
    return hipGetLastError();
  }
  // Shapes the tile kernel does not take (past 256 rows; K and N are multiples of
  // 64 and the outputs aligned, so the streaming kernel takes the rest)
  const int BM = 128;
  int BN = dual ? 64 : 128;
  for (int i = 0; i < a.ngroups; ++i) {
    if (a.g[i].N % 64) return hipErrorInvalidValue;
    if (a.g[i].N % 128) BN = 64;  // a vocabulary of 32064, say
  }
  if (a.K % 32) return hipErrorInvalidValue;
  a.split = dual ? 1 : choose_split(tiles_for(a, BM, BN), a.K, split_max, 32, false);
  a.k_per_split = ceil_div(a.K / 32, a.split) * 32;
  fill_tiles(a, BM, BN);
  if (a.total_tiles == 0) return hipSuccess;
  if (dual) launch_cfg<128, 64, 2, 2, true>(a, st);
  else if (BN == 64) launch_cfg<128, 64, 2, 2, false>(a, st);
  else launch_cfg<128, 128, 2, 2, false>(a, st);
  return hipGetLastError();
}

hipError_t launch_gemm_f32(GemmArgs& a, int split_max, hipStream_t st) {
  (void)split_max;
  if (a.epilogue != EPI_PARTIAL_F32 && a.epilogue != EPI_SWIGLU) return hipErrorInvalidValue;
  a.split = 1;
  a.k_per_split = a.K;
  // 32 x 32 tiles once there are two of them per CU
  int big = 0;
  for (int i = 0; i < a.ngroups; ++i) big += ceil_div(a.g[i].M, 32) * ceil_div(a.g[i].N, 32);
  const int T = big >= 512 ? 32 : 16;
  int t = 0;
  for (int i = 0; i < a.ngroups; ++i) {
    GemmGroup& g = a.g[i];
    g.tiles_m = ceil_div(g.M, T);
    g.tiles_n = ceil_div(g.N, T);
    g.tile_begin = t;
    t += g.tiles_m * g.tiles_n;
  }
  a.total_tiles = t;
  if (t == 0) return hipSuccess;
  const bool dual = a.epilogue == EPI_SWIGLU;
  if (T == 32) {
    if (dual) gemm_f32_kernel<true, 2><<<t, 256, 0, st>>>(a);
    else gemm_f32_kernel<false, 2><<<t, 256, 0, st>>>(a);
  } else {
    if (dual) gemm_f32_kernel<true, 1><<<t, 256, 0, st>>>(a);
    else gemm_f32_kernel<false, 1><<<t, 256, 0, st>>>(a);
  }
  return hipGetLastError();
}

}  // namespace spider
