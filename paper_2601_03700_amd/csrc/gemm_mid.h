// bf16 GEMMs with too few 256x256 tiles to fill the chip: smaller tiles
// (gemm_tile.h), 128x256 with one workgroup per CU or 128x128 with two, and
// tiles cut along K.
//
// Most tiles run in one piece with the fused epilogue.  When the tiles do not
// fill a whole round of the chip, the ones left over (all of them when there
// are few) are cut along K into S pieces each; a piece writes its f32 sums to
// the workspace, and mid_reduce_kernel adds a tile's pieces in order
// (deterministic) and applies the epilogue.  The host makes the plan for
// every number of row tiles (MidTable); the device's row count picks the
// entry, so all workgroups and the reduction agree without a read-back.
//
// What bounds it: with few tiles the latency of a k stage (one 256x256 tile
// of K = 4096 takes 73 us however few there are), with many the loads through
// L2: 128x128 tiles move twice the bytes per MFMA of 256x256 ones (without
// the loads a full chip of them runs at 1.50 PFLOP/s, with them at 1.03;
// 128x256: 1.13, 256x256: 1.25).  Measured, us, 256x256 tiles -> this file:
// 7B width (4096, 11008), 333 rows, QKV / O / gate-up / down 85 / 73 / 93 /
// 198 -> 60 / 27 / 80 / 50; 150 rows 81 / 74 / 81 / 200 -> 45 / 20 / 62 / 43;
// width 1600, 750 rows 55 / 38 / 66 / 107 -> 24 / 18 / 35 / 30.
#pragma once

#include "gemm_tile.h"

namespace adept {

constexpr int kMidRows = 128;        // rows of a tile (both geometries)
constexpr int kMidMaxTm = 32;        // row tiles up to which a plan may cut tiles
constexpr int kMidMinStages = 6;     // k stages per piece at least
constexpr int kMidMaxS = 16;         // pieces per tile at most

// By the number of row tiles tm = 1..kMidMaxTm (entry tm - 1; more: nothing is
// cut): the last `tail` tiles in raster order are cut into S pieces each.
struct MidTable {
  uint16_t tail[kMidMaxTm];
  uint8_t S[kMidMaxTm];
};
struct MidPlan {
  int n_full, tail, S;
  __host__ __device__ int full_blocks() const { return (n_full + 7) / 8 * 8; }
  __host__ __device__ int tail_blocks() const { return (tail * S + 7) / 8 * 8; }
};
__host__ __device__ inline MidPlan mid_plan(const MidTable& mt, int tiles_m, int tiles_n) {
  const int T = tiles_m * tiles_n;
  if (tiles_m > kMidMaxTm) return MidPlan{T, 0, 1};
  const int tail = mt.tail[tiles_m - 1];
  return MidPlan{T - tail, tail, mt.S[tiles_m - 1]};
}

// Epilogues whose tiles are cut: the decoder layer's.  The encoder, the mapper
// and the head give no workspace, and theirs stay whole.
constexpr bool mid_cuts(int epi) { return epi != EPI_STORE && epi != EPI_GELU; }

// Host: the plan table of a geometry (128 or 256 columns) for rows up to
// M_max, and the bounds over it.  split == false: nothing is cut.
struct MidBound {
  int blocks, tail, pieces;
};
MidBound mid_table(int cols, int M_max, int tiles_n, int KT, bool split, MidTable* out);
// output columns per tile: SwiGLU's tiles hold gate and up columns of half as many
inline int mid_tiles_n(int cols, int N, int epi) {
  return epi == EPI_SWIGLU ? N / (cols / 2) : ceil_div(N, cols);
}

namespace {

// Piece e of the cut tiles, in groups of tiles_m tiles (one column tile's
// row tiles, which share its weights): within a group the tiles are fastest,
// then the pieces, so the workgroups of one XCD that run together read the
// same weight slices.
__device__ __forceinline__ void mid_piece(const MidPlan& pl, int e, int tiles_m, int* i, int* s) {
  const int gsz = tiles_m * pl.S;
  const int g = e / gsz, r = e - g * gsz;
  const int in_g = min(tiles_m, pl.tail - g * tiles_m);
  *s = r / in_g;
  *i = g * tiles_m + r % in_g;
}

template <int EPI, int HD, bool EXT, class GT>
__global__ __launch_bounds__(GT::kThreads, GT::kTN == 128 ? 2 : 1) void gemm_mid_kernel(
    GP p, MidTable table, float* ws) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int M = p.M_dev ? min(*p.M_dev, p.M_max) : p.M_max;
  if (M <= 0) return;
  const int tiles_m = (M + kMidRows - 1) / kMidRows;
  const int KT = p.K / BK;
  const MidPlan pl = mid_plan(table, tiles_m, p.tiles_n);
  // ids go to the 8 XCDs round-robin: XCD x takes the x-th contiguous eighth
  // of the whole tiles, then of the pieces
  int b = blockIdx.x, t, k0 = 0, k1 = KT, mt, nt;
  float* part = nullptr;
  const int fb = pl.full_blocks();
  if (b < fb) {
    t = (b & 7) * (fb >> 3) + (b >> 3);
    if (t >= pl.n_full) return;
  } else {
    b -= fb;
    const int tb = pl.tail_blocks();
    if (b >= tb) return;
    const int e = (b & 7) * (tb >> 3) + (b >> 3);
    if (e >= pl.tail * pl.S) return;
    int i, s;
    mid_piece(pl, e, tiles_m, &i, &s);
    t = pl.n_full + i;
    k0 = s * KT / pl.S;
    k1 = (s + 1) * KT / pl.S;
    part = ws + ((int64_t)i * pl.S + s) * (kMidRows * GT::kTN);
  }
  raster_tile(t, tiles_m, p.tiles_n, &mt, &nt);
  gemm_tile<EPI, false, HD, EXT, GT, mid_cuts(EPI)>(p, smem, 0, mt, nt, M, p.B, k0, k1 - k0, part);
}

// Sum of the pieces of a cut tile of C columns at (row r, columns c..c+3);
// four loads in flight.
template <int C>
__device__ __forceinline__ float4 mid_sum(const float* __restrict__ tile, int S, int r, int c) {
  const float* q = tile + r * C + c;
  float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int s = 0; s < S; s += 4) {
    float4 y[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      y[u] = *reinterpret_cast<const float4*>(q + (int64_t)min(s + u, S - 1) * (kMidRows * C));
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (s + u < S) { x.x += y[u].x; x.y += y[u].y; x.z += y[u].z; x.w += y[u].w; }
  }
  return x;
}

// One thread per (row, 4 outputs) of the cut tiles: workgroup (slab, i) takes
// some rows of cut tile i.
template <int EPI, int C>
__global__ __launch_bounds__(256) void mid_reduce_kernel(GP p, MidTable table,
                                                         const float* __restrict__ ws) {
  constexpr int W = EPI == EPI_SWIGLU ? C / 2 : C;   // outputs per tile row
  constexpr int kSlab = 1024 / W;                    // rows per workgroup
  const int M = p.M_dev ? min(*p.M_dev, p.M_max) : p.M_max;
  if (M <= 0) return;
  const int tiles_m = (M + kMidRows - 1) / kMidRows;
  const MidPlan pl = mid_plan(table, tiles_m, p.tiles_n);
  const int i = blockIdx.y;
  if (i >= pl.tail) return;
  int mt, nt;
  raster_tile(pl.n_full + i, tiles_m, p.tiles_n, &mt, &nt);
  const int r = blockIdx.x * kSlab + threadIdx.x / (W / 4), c = (threadIdx.x % (W / 4)) * 4;
  const int m = mt * kMidRows + r, n = nt * W + c;
  if (m >= M || n >= p.N) return;
  const float* tile = ws + (int64_t)i * pl.S * (kMidRows * C);
  // SwiGLU tile columns: 64 gate, then 64 up of the same outputs, per 128
  const int tc = EPI == EPI_SWIGLU ? (c >> 6) * 128 + (c & 63) : c;
  const float sc = p.row_scale ? p.row_scale[m] : 1.0f;
  const float4 x4 = mid_sum<C>(tile, pl.S, r, tc);
  epilogue4<EPI>(p, m, n, sc, x4, [&](int dc) { return mid_sum<C>(tile, pl.S, r, tc + dc); },
                 [&]() { return mid_sum<C>(tile, pl.S, r, tc + 64); });
}

// The reduction's name in timings: epilogue and columns of a tile
template <int EPI, int C> constexpr const char* mid_reduce_name() {
  constexpr bool L = C == 256;
  return EPI == EPI_QKV      ? (L ? "mid_reduce_qkv_256" : "mid_reduce_qkv_128")
         : EPI == EPI_RESID  ? (L ? "mid_reduce_resid_256" : "mid_reduce_resid_128")
         : EPI == EPI_SWIGLU ? (L ? "mid_reduce_swiglu_256" : "mid_reduce_swiglu_128")
                             : (L ? "mid_reduce_gelu_tanh_256" : "mid_reduce_gelu_tanh_128");
}

template <int EPI, int HD, bool EXT, class GT>
adept_status mid_launch_x(const GP& p, const char* name, float* ws, const MidTable& table,
                          const MidBound& b, hipStream_t s) {
  static bool attr_set = false;
  ADEPT_TRY(lds_limit((const void*)gemm_mid_kernel<EPI, HD, EXT, GT>, GT::kLds, &attr_set,
                      "gemm_mid LDS limit"));
  {
    TimedLaunch tl(name ? name : "gemm_mid", s);
    hipLaunchKernelGGL((gemm_mid_kernel<EPI, HD, EXT, GT>), dim3(b.blocks), dim3(GT::kThreads),
                       GT::kLds, s, p, table, ws);
  }
  ADEPT_CHECK_LAUNCH("gemm_mid");
  if constexpr (mid_cuts(EPI)) {
    if (b.tail > 0) {
      constexpr int kSlab = 1024 / (EPI == EPI_SWIGLU ? GT::kTN / 2 : GT::kTN);
      TimedLaunch tl(mid_reduce_name<EPI, GT::kTN>(), s);
      hipLaunchKernelGGL((mid_reduce_kernel<EPI, GT::kTN>), dim3(kMidRows / kSlab, b.tail),
                         dim3(256), 0, s, p, table, ws);
    }
    return launch_status("mid_reduce");
  }
  return ADEPT_OK;
}

template <int EPI, int HD, class GT>
adept_status mid_launch(const GP& p, const char* name, float* ws, const MidTable& table,
                        const MidBound& b, hipStream_t s) {
  return tile_needs_ext(p, EPI, GT::kTN) ? mid_launch_x<EPI, HD, true, GT>(p, name, ws, table, b, s)
                                         : mid_launch_x<EPI, HD, false, GT>(p, name, ws, table, b, s);
}

template <class GT>
adept_status gemm_mid(GP p, int epi, const char* name, float* ws, size_t ws_bytes, hipStream_t s) {
  constexpr int C = GT::kTN;
  p.tiles_m = ceil_div(p.M_max, kMidRows);
  p.tiles_n = mid_tiles_n(C, p.N, epi);
  const int KT = p.K / BK;
  MidTable t{};
  const bool split = mid_cuts(epi) && ws_bytes > 0 &&
                     ws_bytes >= mid_ws_bytes(p.M_max, p.N, p.K, epi);
  MidBound b = mid_table(C, p.M_max, p.tiles_n, KT, split, &t);
  if ((size_t)b.pieces * kMidRows * C * sizeof(float) > ws_bytes)
    b = mid_table(C, p.M_max, p.tiles_n, KT, false, &t);
  switch (epi) {
    case EPI_STORE: return mid_launch<EPI_STORE, 0, GT>(p, name, ws, t, b, s);
    case EPI_QKV:
      return p.head_dim == 128 ? mid_launch<EPI_QKV, 128, GT>(p, name, ws, t, b, s)
                               : mid_launch<EPI_QKV, 64, GT>(p, name, ws, t, b, s);
    case EPI_RESID: return mid_launch<EPI_RESID, 0, GT>(p, name, ws, t, b, s);
    case EPI_SWIGLU: return mid_launch<EPI_SWIGLU, 0, GT>(p, name, ws, t, b, s);
    case EPI_GELU: return mid_launch<EPI_GELU, 0, GT>(p, name, ws, t, b, s);
    case EPI_GELU_TANH: return mid_launch<EPI_GELU_TANH, 0, GT>(p, name, ws, t, b, s);
    default: set_error("gemm: bad epilogue"); return ADEPT_E_INVALID;
  }
}

}  // namespace
}  // namespace adept
