// Dense and grouped GEMMs of the hot path, C[m][n] = sum_k A[m][k] B[n][k]
// (B in nn.Linear [out][in] order, so both operands are K-contiguous).
//
// bf16 path: gemm_tile.h's 256x256 tile when the rows are many; the 128x256 and
// 128x128 tiles of gemm_mid.h otherwise; the skinny path below for 17 to 64 rows
// of wide layers, gemm_direct.hip for the rest of them.
//
// Workgroups are mapped to tiles XCD by XCD: the hardware deals consecutive
// workgroup ids round-robin to the 8 XCDs, so the id is remapped to give each
// XCD a contiguous block of tiles, rastered in groups of 8 row tiles; the
// workgroups resident on one XCD then share A and B k-slices in its L2.
//
// The grouped variant is the decoupled KV generation of Eq. 9: one
// workgroup per (layer r, 256-row tile, column tile) item, the items built on
// the device from the exited rows sorted by exit layer (rows with i* < r form
// a prefix); B is [Wk_r; Wv_r] with layer r's gain folded in, the row scale is
// 1/rms(s~), and the epilogue writes K (with RoPE) and V into cache[r].
#include <algorithm>

#include "gemm_tile.h"

namespace adept {
namespace {

constexpr int BM = 256, BN = 256;
using GeoL = Geo<256, 256>;
constexpr int kThreads = GeoL::kThreads;
constexpr size_t kLdsBytes = GeoL::kLds;

// XCD-aware tile order (see the header comment).
__device__ __forceinline__ void tile_of(int bid, int tiles_m, int tiles_n, int* mt, int* nt) {
  const int T = tiles_m * tiles_n;
  int t = bid;
  if ((T & 7) == 0) t = (bid & 7) * (T >> 3) + (bid >> 3);
  raster_tile(t, tiles_m, tiles_n, mt, nt);
}

// The grid is sized for M_max; the tiles are numbered over the rows that are
// actually active (device count), so when tokens exit the remaining tiles
// still spread over all XCDs and the surplus workgroups return at once.
template <int EPI, int HD, bool EXT>
__global__ __launch_bounds__(kThreads, 1) void gemm_bf16_kernel(GP p) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int M = p.M_dev ? min(*p.M_dev, p.M_max) : p.M_max;
  const int tiles_m = (M + BM - 1) / BM;
  if ((int)blockIdx.x >= tiles_m * p.tiles_n) return;
  int mt, nt;
  tile_of(blockIdx.x, tiles_m, p.tiles_n, &mt, &nt);
  gemm_tile<EPI, false, HD, EXT, GeoL, false>(p, smem, 0, mt, nt, M, p.B, 0, p.K / BK, nullptr);
}

// Grouped GEMM of the KV generation: one workgroup per item of the
// device-built list of (layer, row tile) items times the column tiles,
// rastered in groups of 8 row tiles.  Workgroup ids go to the 8 XCDs
// round-robin, so XCD x takes the x-th contiguous eighth of the item list and
// the tiles running together on an XCD share one layer's weight slices in its
// L2; ids past the device-built count return at once.  (A persistent form
// that took items from per-XCD counters kept the loop's state in registers
// and spilled 196 bytes per lane around the K loop; one item per workgroup
// compiles as the plain GEMM does, without scratch, and runs 2 % faster.)
template <int HD, bool EXT, class GT>
__global__ __launch_bounds__(GT::kThreads, GT::kTN == 128 ? 2 : 1) void gemm_kv_flat_kernel(GP p) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  constexpr int kSub = BM / GT::kTM;   // row tiles of an item: 256 rows
  const int n_work = *p.n_work * kSub;
  const int total = n_work * p.tiles_n;
  const int chunk = (total + 7) >> 3;
  const int t = (int)(blockIdx.x & 7) * chunk + (int)(blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= chunk || t >= total) return;
  int w, nt;
  raster_tile(t, n_work, p.tiles_n, &w, &nt);
  const int packed = p.work[w / kSub];
  const int layer = packed >> 16, mt = (packed & 0xffff) * kSub + w % kSub;
  const int m = p.grp_m[layer];
  if (kSub > 1 && mt * GT::kTM >= m) return;   // the item's second half is empty
  gemm_tile<EPI_KV, true, HD, EXT, GT, false>(p, smem, layer, mt, nt, m,
                                              p.B + (int64_t)(layer - 1) * p.b_layer_stride, 0,
                                              p.K / BK, nullptr);
}

template <int HD, bool EXT, class GT>
adept_status launch_kv_x(GP p, int max_work, hipStream_t s) {
  static bool attr_set = false;
  ADEPT_TRY(lds_limit((const void*)gemm_kv_flat_kernel<HD, EXT, GT>, GT::kLds, &attr_set,
                      "kv LDS limit"));
  p.tiles_n = ceil_div(p.N, GT::kTN);
  // one workgroup per tile: the host bound on them, rounded to whole XCD rounds
  const int flat = (max_work * (BM / GT::kTM) * p.tiles_n + 7) / 8 * 8;
  {
    TimedLaunch tl(GT::kTN == 256 ? "gemm_kv_flat_kernel<256x256>" : "gemm_kv_flat_kernel<128x128>", s);
    hipLaunchKernelGGL((gemm_kv_flat_kernel<HD, EXT, GT>), dim3(flat), dim3(GT::kThreads), GT::kLds,
                       s, p);
  }
  return launch_status("gemm_kv_grouped");
}

template <class GT>
adept_status launch_kv(const GP& p, int max_work, hipStream_t s) {
  const bool ext = tile_needs_ext(p, EPI_KV, GT::kTN) || p.bias;
  if (p.head_dim == 128)
    return ext ? launch_kv_x<128, true, GT>(p, max_work, s) : launch_kv_x<128, false, GT>(p, max_work, s);
  return ext ? launch_kv_x<64, true, GT>(p, max_work, s) : launch_kv_x<64, false, GT>(p, max_work, s);
}

// Sets a kernel's dynamic-LDS limit once per process.
adept_status allow_lds(const void* kernel, bool* done, const char* what) {
  return lds_limit(kernel, kLdsBytes, done, what);
}

template <int EPI, int HD, bool EXT>
adept_status launch_bf16_x(const GP& p, hipStream_t s, const char* name) {
  static bool attr_set = false;
  ADEPT_TRY(allow_lds((const void*)gemm_bf16_kernel<EPI, HD, EXT>, &attr_set,
                      "gemm_bf16 LDS limit"));
  {
    TimedLaunch tl(name ? name : "gemm_bf16", s);
    hipLaunchKernelGGL((gemm_bf16_kernel<EPI, HD, EXT>), dim3(p.tiles_m * p.tiles_n),
                       dim3(kThreads), kLdsBytes, s, p);
  }
  return launch_status("gemm_bf16");
}

bool needs_ext(const GP& p, int epi) { return tile_needs_ext(p, epi, BN); }

template <int EPI, int HD>
adept_status launch_bf16(const GP& p, hipStream_t s, const char* name) {
  return needs_ext(p, EPI) ? launch_bf16_x<EPI, HD, true>(p, s, name)
                           : launch_bf16_x<EPI, HD, false>(p, s, name);
}

// ---------------------------------------------------------------------------
// Skinny path (17 to 64 rows of wide layers: decode; fewer rows and narrower
// layers: gemm_direct.hip).  The weights are streamed from HBM once; M is too
// small for the 256x256 tile to give the chip enough workgroups.  The work is a flattened space of units: a unit is one
// 64-column tile of the partial space (N columns, or the
// F gate columns followed by the F up columns for SWIGLU) times one 64-deep
// k step.  The units are cut into G equal contiguous ranges, one per
// workgroup (stream-K), so that every workgroup streams the same number of
// weight bytes and the grid is one even wave of about two workgroups per CU;
// a range is never longer than a tile's k extent, so it covers at most two
// tiles (two segments).  Each (workgroup, segment) writes one 64x64 fp32
// partial tile; skinny_epilogue_kernel sums a tile's partials in workgroup
// order (deterministic) and applies the same epilogues as the tiled path.
// ---------------------------------------------------------------------------
constexpr int kSkinnyM = 64;      // rows of a skinny pass (decode: one per sequence)
constexpr int kSkStages = 4;      // LDS ring depth
constexpr int kSkStage = 2 * 64 * 128;   // A and B, 64 rows x 64 k each: 16 KiB
constexpr int kSkPart = kSkinnyM * kSkinnyBN;   // floats of one partial tile
constexpr int kSkGroups = 512;    // target grid: two workgroups per CU

// Skinny GEMM (M <= 64): workgroup w multiplies the units [w*U, w*U + U) and
// writes the partial tile of each segment to part[w][segment][m][c].  The
// pass streams B (the weights) once, so it is HBM-bound: A and B reach LDS by
// direct loads of whole 128-byte rows (eight lanes per row, one cache line),
// four stages deep, and the four waves each take a 32x32 block of the 64x64
// tile.  The two segments of a range share one load pipeline (the second
// tile's first stages are in flight while the first tile's last ones are
// multiplied); the first segment's accumulators are held in registers and
// both partial tiles are written at the end, so no store sits among the
// loads that the stage waits count.
__global__ __launch_bounds__(256, 2) void gemm_skinny_kernel(GP p, int nb, SkSplit sp,
                                                             float* __restrict__ part) {
  __shared__ __attribute__((aligned(1024))) char sm[kSkStages * kSkStage];
  const int M = p.M_dev ? min(*p.M_dev, p.M_max) : p.M_max;
  if (M <= 0) return;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int64_t u0 = (int64_t)blockIdx.x * sp.U;
  const int n = (int)(min(sp.total, u0 + sp.U) - u0);   // >= 1: G = ceil(total / U)
  // a range is never longer than a tile's k extent (U <= KT): tiles t0, t1
  const int t0 = (int)(u0 / sp.KT), kb0 = (int)(u0 - (int64_t)t0 * sp.KT);
  const int n0 = min(n, sp.KT - kb0);   // k steps in tile t0; the rest are in t0 + 1
  const int rA = wm * 32 + (lane & 31), rB = wn * 32 + (lane & 31);
  const int swz = (lane >> 1) & 7;
  // direct-load instruction j (0..3) of wave w: operand (A for waves 0-1, B
  // for 2-3), rows 8q .. 8q+7 with q = (4w + j) mod 8; lane l -> row 8q + l/8,
  // stored position l%8, logical chunk (l%8) ^ ((row >> 1) & 7).  src0 / src1
  // point at k step 0 of tile t0 / t0 + 1 (the same A row for both), so the
  // loop only selects one and adds the k offset.
  const bf16* src0[4];
  const bf16* src1[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int q = (4 * wave + j) & 7;
    const int r = 8 * q + (lane >> 3);
    const int ch = (lane & 7) ^ ((r >> 1) & 7);
    if (wave < 2) {
      const int m = min(r, M - 1);   // clamped: loaded, never stored
      const int row = p.a_rows ? p.a_rows[m] : m;
      const bf16* abase = (p.a_sel && (p.a_sel[row] & 1)) ? p.A2 : p.A;
      src0[j] = src1[j] = abase + (int64_t)row * p.lda + ch * 8;
    } else {
      // tile t0 + 1 past the last tile (then n0 == n) is never loaded
      const int na = t0 * kSkinnyBN + r;
      const int nb1 = (int64_t)(t0 + 1) * sp.KT < sp.total ? na + kSkinnyBN : na;
      src0[j] = (na >= nb ? p.B2 + (int64_t)(na - nb) * p.ldb : p.B + (int64_t)na * p.ldb) + ch * 8;
      src1[j] = (nb1 >= nb ? p.B2 + (int64_t)(nb1 - nb) * p.ldb : p.B + (int64_t)nb1 * p.ldb) +
                ch * 8;
    }
  }
  auto issue = [&](int i) {   // stage i of the range into ring slot i % kSkStages
    const bool second = i >= n0;
    const int k = (second ? i - n0 : kb0 + i) * BK;
    char* slot = sm + (i % kSkStages) * kSkStage + (wave >> 1) * 8192;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      dma16((second ? src1[j] : src0[j]) + k, slot + ((4 * wave + j) & 7) * 1024);
  };
  // the stages [i0, i1) of the range into acc
  auto run = [&](f32x16_t& acc, int i0, int i1) {
    for (int it = i0; it < i1; ++it) {
      // stage it has landed once at most the later stages' loads are in
      // flight; near the end of the range fewer stages follow it
      if (it + kSkStages - 2 < n) wait_vm<4 * (kSkStages - 2)>();
      else wait_dma();
      stage_barrier();   // publishes stage it; every wave is done with stage it-1
      if (it + kSkStages - 1 < n) issue(it + kSkStages - 1);   // into stage it-1's slot
      const char* st = sm + (it % kSkStages) * kSkStage;
#pragma unroll
      for (int ks = 0; ks < BK / 16; ++ks) {
        const int ch = (2 * ks + (lane >> 5)) ^ swz;
        const bf16x8_t a = *reinterpret_cast<const bf16x8_t*>(st + (rA * 8 + ch) * 16);
        const bf16x8_t b = *reinterpret_cast<const bf16x8_t*>(st + 8192 + (rB * 8 + ch) * 16);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
      }
    }
  };
  f32x16_t acc0, acc1;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc0[v] = acc1[v] = 0.0f;
#pragma unroll
  for (int s = 0; s < kSkStages - 1; ++s)
    if (s < n) issue(s);
  run(acc0, 0, n0);
  run(acc1, n0, n);
  // every load has landed (the last stage waited for all of them)
  // C layout: value v is row 8*(v/4) + 4*(lane/32) + v%4 of the block, column lane%32
  float* dst = part + (int64_t)blockIdx.x * 2 * kSkPart;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int r = wm * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
    dst[r * kSkinnyBN + wn * 32 + (lane & 31)] = acc0[v];
  }
  if (n0 < n) {
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int r = wm * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
      dst[kSkPart + r * kSkinnyBN + wn * 32 + (lane & 31)] = acc1[v];
    }
  }
}

// Sum of the partials of row m, partial-space columns c..c+3: the
// workgroups whose ranges meet c's tile, in ascending order; a workgroup
// whose range starts in that tile holds it as segment 0, one that starts in
// the tile before as segment 1.
__device__ __forceinline__ float4 skinny_sum(const float* __restrict__ part, const SkSplit& sp,
                                             int m, int c) {
  const int t = c / kSkinnyBN, col = c - t * kSkinnyBN;
  const int64_t u0 = (int64_t)t * sp.KT;
  const int w0 = (int)(u0 / sp.U), w1 = (int)((u0 + sp.KT - 1) / sp.U);
  float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int w = w0; w <= w1; ++w) {
    const int seg = (int64_t)w * sp.U >= u0 ? 0 : 1;
    const float4 y = *reinterpret_cast<const float4*>(part + ((int64_t)w * 2 + seg) * kSkPart +
                                                      m * kSkinnyBN + col);
    x.x += y.x; x.y += y.y; x.z += y.z; x.w += y.w;
  }
  return x;
}

// One thread per (row, 4 output columns).
template <int EPI>
__global__ __launch_bounds__(256) void skinny_epilogue_kernel(GP p, int nout, SkSplit sp,
                                                              const float* __restrict__ part) {
  const int M = p.M_dev ? min(*p.M_dev, p.M_max) : p.M_max;
  const int g4 = nout / 4;
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int m = (int)(idx / g4), n = (int)(idx % g4) * 4;
  if (m >= M) return;
  const float sc = p.row_scale ? p.row_scale[m] : 1.0f;
  const float4 x4 = skinny_sum(part, sp, m, n);
  epilogue4<EPI>(p, m, n, sc, x4, [&](int dc) { return skinny_sum(part, sp, m, n + dc); },
                 [&]() { return skinny_sum(part, sp, m, nout + n); });
}

// The residual epilogue with the next step over its result rows: one
// workgroup of 1024 threads per row m (rows of at most 4096; thread t owns
// columns 4t..4t+3, so every partial of the row is in flight at once).  From
// the bf16 results (the values a separate pass would read back), summed lane
// by lane, across the wave, then over the 16 waves in order:
//  * ROW_RINV: rinv_out[m] = 1/sqrt(mean(v^2) + eps) (the next RMSNorm's
//    factor), f32;
//  * ROW_LN: ln_out[m] = (v - mean) / sqrt(var + eps) (LayerNorm without its
//    affine part, two passes over the registers), f32;
//  * ROW_EXIT: the GLOBAL exit test of the row against its inertia I:
//    <v,v>, <I,I>, <v,I> in double (every product of two floats is exact),
//    the decision of Eq. 8, then I += v/|v| (as adept_exit_test).
enum { ROW_RINV = 0, ROW_LN = 1, ROW_EXIT = 2 };
template <int MODE>
__global__ __launch_bounds__(1024) void skinny_resid_row_kernel(GP p, int nout, SkSplit sp,
                                                                const float* __restrict__ part) {
  __shared__ float wsum[16];
  __shared__ float total;
  __shared__ double dsum[16][3];
  __shared__ double dtot[3];
  const int M = p.M_dev ? min(*p.M_dev, p.M_max) : p.M_max;
  const int m = blockIdx.x;
  if (m >= M) return;
  const float sc = p.row_scale ? p.row_scale[m] : 1.0f;
  const int n = threadIdx.x * 4;
  const bool live = n < nout;
  float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  if (live) {
    const float4 x4 = skinny_sum(part, sp, m, n);
    const float4 bx = bias4(p.bias, n);
    const float x[4] = {x4.x * sc + bx.x, x4.y * sc + bx.y, x4.z * sc + bx.z, x4.w * sc + bx.w};
    const int64_t off = (int64_t)p.rows[m] * p.ldc + n;
    const bf16x4_t r = *reinterpret_cast<const bf16x4_t*>(p.resid + off);
    bf16x4_t o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      o[e] = f2bf(x[e] + bf2f(r[e]));
      v[e] = bf2f(o[e]);
    }
    *reinterpret_cast<bf16x4_t*>(reinterpret_cast<bf16*>(p.C) + off) = o;
  }
  auto block_sum = [&](float x) {
    x = wave_sum_f32(x);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = x;
    __syncthreads();
    if (threadIdx.x == 0) {
      float t = 0.0f;
#pragma unroll
      for (int w = 0; w < 16; ++w) t += wsum[w];
      total = t;
    }
    __syncthreads();
    const float t = total;
    __syncthreads();   // wsum and total are reused by the next sum
    return t;
  };
  if (MODE == ROW_EXIT) {
    const int row = p.rows[m];
    float* ir = p.ex.inertia + (int64_t)row * nout;
    f32x4_t i4 = {0.f, 0.f, 0.f, 0.f};
    if (live) i4 = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>(ir + n));
    const float iv[4] = {i4[0], i4[1], i4[2], i4[3]};
    double s3[3] = {0.0, 0.0, 0.0};   // <v,v>, <I,I>, <v,I>
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const double a = v[e], b = iv[e];
      s3[0] = fma(a, a, s3[0]);
      s3[1] = fma(b, b, s3[1]);
      s3[2] = fma(a, b, s3[2]);
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) s3[q] = wave_sum_f64(s3[q]);
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
      for (int q = 0; q < 3; ++q) dsum[threadIdx.x >> 6][q] = s3[q];
    }
    __syncthreads();
    if (threadIdx.x < 3) {
      double t = 0.0;
#pragma unroll
      for (int w = 0; w < 16; ++w) t += dsum[w][threadIdx.x];
      dtot[threadIdx.x] = t;
    }
    __syncthreads();
    const double nh = sqrt(dtot[0]), nr = sqrt(dtot[1]);
    const double den = nh * nr;
    const double sim = den > 0.0 ? dtot[2] / den : __longlong_as_double(0x7ff8000000000000ll);
    if (threadIdx.x == 0) {
      p.ex.exit_flag[m] = exit_decision(sim >= p.ex.delta, p.ex.layer, p.ex.min_exit_layer,
                                        p.ex.n_layers, p.ex.force_layer, row) ? 1 : 0;
      if (p.ex.sim_out) p.ex.sim_out[m] = sim;
    }
    if (live && nh > 0.0) {
      const double inv = 1.0 / nh;
      f32x4_t o4;
#pragma unroll
      for (int e = 0; e < 4; ++e) o4[e] = (float)((double)iv[e] + (double)v[e] * inv);
      __builtin_nontemporal_store(o4, reinterpret_cast<f32x4_t*>(ir + n));
    }
  } else if (MODE == ROW_RINV) {
    float ss = 0.0f;
#pragma unroll
    for (int e = 0; e < 4; ++e) ss = fmaf(v[e], v[e], ss);
    const float t = block_sum(ss);
    if (threadIdx.x == 0) p.rinv_out[m] = 1.0f / sqrtf(t / (float)nout + p.row_eps);
  } else {
    const float mean = block_sum((v[0] + v[1]) + (v[2] + v[3])) / (float)nout;
    float q = 0.0f;
    if (live) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float t = v[e] - mean;
        q = fmaf(t, t, q);
      }
    }
    const float r = 1.0f / sqrtf(block_sum(q) / (float)nout + p.row_eps);
    if (live) {
      bf16x4_t y;
#pragma unroll
      for (int e = 0; e < 4; ++e) y[e] = f2bf((v[e] - mean) * r);
      *reinterpret_cast<bf16x4_t*>(p.ln_out + (int64_t)m * nout + n) = y;
    }
  }
}

template <int EPI>
adept_status launch_skinny(const GP& p, int Nt, int nout, hipStream_t s, const char* name,
                           float* part) {
  const SkSplit sp = skinny_split(Nt, p.K);
  {
    TimedLaunch tl(name ? name : "gemm_skinny", s);
    hipLaunchKernelGGL(gemm_skinny_kernel, dim3(sp.G), dim3(256), 0, s, p,
                       EPI == EPI_SWIGLU ? nout : Nt, sp, part);
  }
  ADEPT_CHECK_LAUNCH("gemm_skinny");
  if (EPI == EPI_RESID && (p.ln_out || p.rinv_out || p.has_exit)) {
    const dim3 g(p.M_max), b(1024);
    if (p.has_exit)
      ADEPT_LAUNCH(skinny_resid_row_kernel<ROW_EXIT>, g, b, 0, s, p, nout, sp, part);
    else if (p.ln_out)
      ADEPT_LAUNCH(skinny_resid_row_kernel<ROW_LN>, g, b, 0, s, p, nout, sp, part);
    else
      ADEPT_LAUNCH(skinny_resid_row_kernel<ROW_RINV>, g, b, 0, s, p, nout, sp, part);
    return launch_status("skinny_resid_row");
  }
  const int64_t total = (int64_t)p.M_max * (nout / 4);
  ADEPT_LAUNCH(skinny_epilogue_kernel<EPI>, dim3((unsigned)((total + 255) / 256)), dim3(256), 0,
               s, p, nout, sp, part);
  return launch_status("skinny_epilogue");
}

bool aligned8(const void* p) { return ((uintptr_t)p & 7u) == 0; }

bool aligned_operands(const GemmArgs& g) {
  return aligned16(g.A) && aligned16(g.B) && (!g.B2 || aligned16(g.B2)) &&
         (!(g.a_sel || (g.list && g.list->exit_layer)) || (g.A2 && aligned16(g.A2))) &&
         g.lda % 8 == 0 && g.ldb % 8 == 0;
}

}  // namespace

SkSplit skinny_split(int Nt, int K) {
  SkSplit sp;
  sp.KT = K / BK;
  sp.total = (int64_t)(Nt / kSkinnyBN) * sp.KT;
  if (sp.total <= 0) {   // no work (the entry rejects K or N below one tile)
    sp.G = 0;
    sp.U = 1;
    return sp;
  }
  const int64_t g = std::max<int64_t>(1, std::min<int64_t>(kSkGroups, sp.total));
  // at least four k steps (32 KiB of weights) against each 16 KiB partial tile
  sp.U = (int)std::min<int64_t>(std::max<int64_t>((sp.total + g - 1) / g, 4), sp.KT);
  sp.G = (int)((sp.total + sp.U - 1) / sp.U);
  return sp;
}

size_t skinny_ws_bytes(int Nt, int K) {
  return (size_t)skinny_split(Nt, K).G * 2 * kSkPart * sizeof(float);
}

bool gemm_skinny_row_norm(const GemmArgs& g) {
  return g.epi == EPI_RESID && !gemm_direct_fits(g) && g.M_max > 0 && g.M_max <= kSkinnyM &&
         g.skinny_ws && g.N > 0 && g.N % 64 == 0 && g.N <= 4096 && g.K > 0 && g.K % BK == 0 &&
         skinny_ws_bytes(g.N, g.K) <= g.skinny_ws_bytes;
}

adept_status gemm(adept_dtype dt, const GemmArgs& g, hipStream_t s) {
  if (g.M_max <= 0) return ADEPT_OK;
  const bool direct = gemm_direct_fits(g);
  if ((g.row_norm || g.list) && !direct) {
    set_error("gemm: row_norm and list only where gemm_direct_fits");
    return ADEPT_E_INVALID;
  }
  if ((g.rinv_out || g.ln_out || g.exit) &&
      (!gemm_skinny_row_norm(g) || (!!g.rinv_out + !!g.ln_out + !!g.exit) > 1 ||
       (g.ln_out && !aligned8(g.ln_out)) ||
       (g.exit && (!g.exit->inertia || !aligned16(g.exit->inertia) || !g.exit->exit_flag)))) {
    set_error("gemm: one of rinv_out / ln_out (8-byte aligned) / exit (16-byte aligned inertia, "
              "flags) only on the skinny residual path (see gemm_skinny_row_norm)");
    return ADEPT_E_INVALID;
  }
  if (dt != ADEPT_BF16) {
    set_error("gemm: bf16 entry called with another dtype");
    return ADEPT_E_INVALID;
  }
  if (g.K <= 0 || g.K % BK != 0) {
    set_error("gemm: K=%d not a positive multiple of %d", g.K, BK);
    return ADEPT_E_UNSUPPORTED;
  }
  // the last 256-column tile may be ragged (N a multiple of 64); SwiGLU pairs
  // 64 gate with 64 up columns per wave, so its N is a multiple of 128
  const int ncols = g.epi == EPI_SWIGLU ? 128 : 64;
  if (g.N <= 0 || g.N % ncols != 0) {
    set_error("gemm: N=%d not a positive multiple of %d", g.N, ncols);
    return ADEPT_E_UNSUPPORTED;
  }
  if ((g.epi == EPI_QKV) &&
      (g.d_q % 64 != 0 ||
       (g.rope_cos && (g.d_q % 128 != 0 || (g.head_dim != 64 && g.head_dim != 128))) ||
       (!g.rope_cos && !g.bias && g.d_q % 128 != 0))) {
    set_error("gemm: QKV epilogue needs d_q %% 64 == 0 (d_q %% 128 == 0 and head_dim 64/128 "
              "with RoPE or without a bias)");
    return ADEPT_E_UNSUPPORTED;
  }
  if (g.bias && (g.epi == EPI_SWIGLU || g.epi == EPI_KV || !aligned8(g.bias))) {
    set_error("gemm: bias needs an 8-byte aligned [N] vector and no SWIGLU / KV epilogue");
    return ADEPT_E_UNSUPPORTED;
  }
  if (!aligned_operands(g)) {
    set_error("gemm: operands must be 16-byte aligned with leading dims a multiple of 8");
    return ADEPT_E_INVALID;
  }
  if (direct) return gemm_direct(g, s);
  GP p = to_gp(g);
  if (g.M_max <= kSkinnyM && g.skinny_ws && g.epi != EPI_KV) {
    const int Nt = g.epi == EPI_SWIGLU ? 2 * g.N : g.N;
    if (skinny_ws_bytes(Nt, g.K) <= g.skinny_ws_bytes) {
      switch (g.epi) {
        case EPI_STORE: return launch_skinny<EPI_STORE>(p, Nt, g.N, s, g.name, g.skinny_ws);
        case EPI_QKV: return launch_skinny<EPI_QKV>(p, Nt, g.N, s, g.name, g.skinny_ws);
        case EPI_RESID: return launch_skinny<EPI_RESID>(p, Nt, g.N, s, g.name, g.skinny_ws);
        case EPI_SWIGLU: return launch_skinny<EPI_SWIGLU>(p, Nt, g.N, s, g.name, g.skinny_ws);
        case EPI_GELU: return launch_skinny<EPI_GELU>(p, Nt, g.N, s, g.name, g.skinny_ws);
        case EPI_GELU_TANH:
          return launch_skinny<EPI_GELU_TANH>(p, Nt, g.N, s, g.name, g.skinny_ws);
        default: break;
      }
    }
  }
  const size_t ws_bytes = g.skinny_ws ? g.skinny_ws_bytes : 0;
  switch (mid_choose(p, g.epi, ws_bytes)) {
    case kTile128x256: return gemm_mid_128x256(p, g.epi, g.name, g.skinny_ws, ws_bytes, s);
    case kTile128x128: return gemm_mid_128x128(p, g.epi, g.name, g.skinny_ws, ws_bytes, s);
    default: break;
  }
  p.tiles_m = ceil_div(g.M_max, BM);
  p.tiles_n = g.epi == EPI_SWIGLU ? g.N / 128 : ceil_div(g.N, BN);
  switch (g.epi) {
    case EPI_STORE: return launch_bf16<EPI_STORE, 0>(p, s, g.name);
    case EPI_QKV:
      return g.head_dim == 128 ? launch_bf16<EPI_QKV, 128>(p, s, g.name)
                               : launch_bf16<EPI_QKV, 64>(p, s, g.name);
    case EPI_RESID: return launch_bf16<EPI_RESID, 0>(p, s, g.name);
    case EPI_SWIGLU: return launch_bf16<EPI_SWIGLU, 0>(p, s, g.name);
    case EPI_GELU: return launch_bf16<EPI_GELU, 0>(p, s, g.name);
    case EPI_GELU_TANH: return launch_bf16<EPI_GELU_TANH, 0>(p, s, g.name);
    default: set_error("gemm: bad epilogue"); return ADEPT_E_INVALID;
  }
}

// Grouped bf16 GEMM of the KV generation (see the header comment).  g.row_scale
// is indexed by the sorted position.
adept_status gemm_kv_grouped(const GemmArgs& g, const int32_t* work, const int32_t* n_work,
                             int max_work, const int32_t* grp_m,
                             const int32_t* srows,
                             int64_t b_layer_stride, int64_t cache_layer_stride, hipStream_t s) {
  if (max_work <= 0) return ADEPT_OK;
  if (!aligned_operands(g)) {
    set_error("kv_generate: operands must be 16-byte aligned");
    return ADEPT_E_INVALID;
  }
  if (g.N <= 0 || g.N % 64 != 0 || (g.bias && !aligned8(g.bias)) ||
      (!g.bias && g.d_q % 128 != 0)) {
    set_error("kv_generate: 2*H*hd must be a multiple of 64 (128 per section without a bias), "
              "the bias 8-byte aligned");
    return ADEPT_E_UNSUPPORTED;
  }
  GP p = to_gp(g);
  p.work = work; p.n_work = n_work; p.grp_m = grp_m; p.srows = srows;
  p.b_layer_stride = b_layer_stride;
  p.cache_layer_stride = cache_layer_stride;
  // Few tiles (one or two skipped layers): a tile's latency is the time, so
  // 128x128 tiles, two per CU.  Two layers, 20 to 30 % of the rows leaving after
  // the first: 7B width, 333 rows 636 -> 608 us, 1500 rows 1311 -> 1291; width
  // 1600, 750 rows 351 -> 315, 7200 rows (377 tiles) 1263 -> 1244.  With more
  // tiles the smaller ones' loads through L2 bind: 600 rows over 24 layers of
  // the 7B width 841 -> 909 us, 4096 rows 2970 -> 3970.
  if ((int64_t)max_work * ceil_div(g.N, BN) <= 512) return launch_kv<Geo<128, 128>>(p, max_work, s);
  return launch_kv<GeoL>(p, max_work, s);
}

}  // namespace adept
