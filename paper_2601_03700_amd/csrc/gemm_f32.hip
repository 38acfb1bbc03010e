// f32 GEMMs (small configurations), C[m][n] = sum_k A[m][k] B[n][k] with the
// decoder's epilogues, on the f32 matrix instruction (f32 products and sums).
//
// Main form: one workgroup per 16 x 16 outputs (QKV and SwiGLU: per 16 x 2 x 16,
// a block of columns and its rotary partner, or gate and up), its four or
// sixteen waves taking every fourth or sixteenth 32-deep piece of K; the waves'
// sums meet in LDS, in wave order, where the epilogue runs, with the row's RMSNorm factor formed
// from the A values on the way when asked.  The shapes are small (128 x 256,
// K = 1024): what bounds them is the chip they leave idle and the chain of
// dependent loads, so the tile is the smallest the instruction gives, K is
// spread over the waves and no second kernel follows.  Measured at 128 rows of
// the tiny decoder: K = 1024, N = 256: 119 us (8 workgroups of 64 x 64, plain
// FMAs) -> 7; a layer's GEMMs with their epilogue and norm kernels 400 -> 25.
//
// General form (outputs of many 64x64 tiles, K or leading dimensions not multiples
// of 4, unaligned operands, rotary heads not a multiple of 32): 64x64-tiled FMA GEMM into a
// float scratch buffer followed by an element-wise epilogue kernel.
#include "gemm_tile.h"

namespace adept {
namespace {

// EPI_KV, the KV generation (blockIdx.z: layer - 1): K and V of the listed rows
// that exited before the layer, with the layer's norm gain when it is not
// folded into the weights.
struct KvF32 {
  const int32_t* exit_layer;
  const float* gain;      // [n_layers][K], nullable
};

template <int EPI, bool NORM, int W>
__global__ __launch_bounds__(64 * W) void gemm_f32_mfma_kernel(GP p, KvF32 kv) {
  constexpr bool kCache = EPI == EPI_QKV || EPI == EPI_KV;
  constexpr int NB = kCache || EPI == EPI_SWIGLU ? 2 : 1;
  __shared__ float red[W][NB][16][17];
  __shared__ float ssq[W][16];
  const int M = p.M_dev ? min(*p.M_dev, p.M_max) : p.M_max;
  const int m0 = blockIdx.x * 16;
  if (m0 >= M) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r16 = lane & 15, q = lane >> 4;
  const float* A = reinterpret_cast<const float*>(p.A);
  const float* B = reinterpret_cast<const float*>(p.B);
  // first output column of the block(s): QKV takes 16 columns of the first half
  // of a head and the 16 that rotate with them
  const int half = p.head_dim >> 1;
  int n0 = blockIdx.y * 16;
  if (kCache) n0 = n0 / half * p.head_dim + n0 % half;
  const int am = min(m0 + r16, M - 1);   // clamped: never stored
  const int arow = p.a_rows ? p.a_rows[am] : am;
  const float* gain = nullptr;
  if (EPI == EPI_KV) {
    const int layer = blockIdx.z + 1;
    if (!__any(kv.exit_layer[arow] < layer)) return;   // the same rows in every wave
    B += (int64_t)blockIdx.z * p.b_layer_stride;
    if (kv.gain) gain = kv.gain + (int64_t)blockIdx.z * p.K + 4 * q;
  }
  const float* ar = A + (int64_t)arow * p.lda + 4 * q;
  const float* br[NB];
  const int bn = min(n0 + r16, p.N - 1);
  br[0] = B + (int64_t)bn * p.ldb + 4 * q;
  if (kCache) br[NB - 1] = B + (int64_t)(n0 + half + r16) * p.ldb + 4 * q;
  if (EPI == EPI_SWIGLU)
    br[NB - 1] = reinterpret_cast<const float*>(p.B2) + (int64_t)bn * p.ldb + 4 * q;
  // the epilogue's inputs of this thread's output (row r, column c), loaded
  // beside the operands: each would be one more memory latency at the end
  const int r = threadIdx.x >> 4, c = threadIdx.x & 15;
  const int m = m0 + r, n = n0 + c, mc = min(m, M - 1);
  int row = 0, slot = 0;
  float res = 0.0f, cs = 1.0f, sn = 0.0f, sc = 1.0f;
  if (!NORM && p.row_scale) sc = p.row_scale[mc];
  if (EPI == EPI_RESID) {
    row = p.rows[mc];
    if (n < p.N) res = reinterpret_cast<const float*>(p.resid)[(int64_t)row * p.ldc + n];
  }
  if (kCache) {
    row = p.rows[mc];
    slot = p.slot ? p.slot[row] : row;
    if (p.rope_cos) {
      const int64_t t = (int64_t)p.pos[row] * half + n % p.head_dim;   // n < hd/2 in its head
      cs = p.rope_cos[t];
      sn = p.rope_sin[t];
    }
  }
  f32x4_t acc[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) acc[b] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float ss = 0.0f;
  // lane (row r16, q) holds k = k0 + 16 h + 4 q + 0..3 of both operands, so the
  // instruction's four k are 4 q + e of the four q, for e = 0..3.  Two of the
  // wave's 32-deep pieces are loaded at once.
  constexpr int U = 2, kStep = 32 * W;
#pragma unroll 1
  for (int kb = 32 * wave; kb < p.K; kb += U * kStep) {
    float4 a[U][2], b[NB][U][2];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int k = kb + u * kStep + 16 * h;
        const bool in = k + 4 * q < p.K;
        const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int x = 0; x < NB; ++x)
          b[x][u][h] = in ? *reinterpret_cast<const float4*>(br[x] + k) : z;
        a[u][h] = in ? *reinterpret_cast<const float4*>(ar + k) : z;
      }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (kb + u * kStep >= p.K) break;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        float av[4] = {a[u][h].x, a[u][h].y, a[u][h].z, a[u][h].w};
        if (NORM) {
#pragma unroll
          for (int e = 0; e < 4; ++e) ss = fmaf(av[e], av[e], ss);
        }
        const int k = kb + u * kStep + 16 * h;
        if (EPI == EPI_KV && gain && k + 4 * q < p.K) {
          const float4 gv = *reinterpret_cast<const float4*>(gain + k);
          av[0] *= gv.x; av[1] *= gv.y; av[2] *= gv.z; av[3] *= gv.w;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
#pragma unroll
          for (int x = 0; x < NB; ++x) {
            const float bv[4] = {b[x][u][h].x, b[x][u][h].y, b[x][u][h].z, b[x][u][h].w};
            acc[x] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[e], bv[e], acc[x], 0, 0, 0);
          }
        }
      }
    }
  }
#pragma unroll
  for (int c = 0; c < NB; ++c)
#pragma unroll
    for (int v = 0; v < 4; ++v) red[wave][c][4 * q + v][r16] = acc[c][v];
  if (NORM) {
    ss += __shfl_xor(ss, 16, 64);
    ss += __shfl_xor(ss, 32, 64);
    if (q == 0) ssq[wave][r16] = ss;
  }
  __syncthreads();
  if (threadIdx.x >= 256 || m >= M || n >= p.N) return;
  float x[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    x[b] = 0.0f;
#pragma unroll
    for (int w = 0; w < W; ++w) x[b] += red[w][b][r][c];
  }
  if (NORM) {
    float t = 0.0f;
#pragma unroll
    for (int w = 0; w < W; ++w) t += ssq[w][r];
    sc = 1.0f / sqrtf(t / (float)p.K + p.row_eps);
  }
  float* C = reinterpret_cast<float*>(p.C);
  if (EPI == EPI_STORE) {
    C[(int64_t)m * p.ldc + n] = x[0] * sc;
  } else if (EPI == EPI_RESID) {
    C[(int64_t)row * p.ldc + n] = res + x[0] * sc;
  } else if (EPI == EPI_SWIGLU) {
    C[(int64_t)m * p.ldc + n] = silu(x[0] * sc) * (x[NB - 1] * sc);
  } else {   // EPI_QKV, EPI_KV
    int sec = n / p.d_q;
    const int cin = n - sec * p.d_q;
    if (EPI == EPI_KV) ++sec;   // 0 Q, 1 K, 2 V
    const int64_t lay = EPI == EPI_KV ? (int64_t)blockIdx.z * p.cache_layer_stride : 0;
    if (EPI == EPI_KV && kv.exit_layer[row] > (int)blockIdx.z) return;
    float* dst = sec == 0 ? reinterpret_cast<float*>(p.q_out) + (int64_t)m * p.d_q
                          : reinterpret_cast<float*>(sec == 1 ? p.k_cache : p.v_cache) + lay +
                                (int64_t)slot * p.d_q;
    float lo = x[0] * sc, hi = x[NB - 1] * sc;
    if (sec < 2 && p.rope_cos) {   // rotate-half RoPE of columns cin and cin + hd/2
      const float y = lo;
      lo = y * cs - hi * sn;
      hi = hi * cs + y * sn;
    }
    dst[cin] = lo;
    dst[cin + half] = hi;
  }
}

// Sixteen waves for the two-block epilogues, whose rows are norms and weights of
// K = 256 (QKV 10.0 -> 8.6 us, gate/up 14.2 -> 12.9, K/V generation 11.4 ->
// 10.0 at 128 rows); four for the others (O and down projections 11.8, with
// sixteen 12.4: the sums of more waves cost what the shorter chain gains).
template <int EPI>
adept_status launch_f32_grid(const GP& p, const KvF32& kv, const dim3& grid, bool norm,
                             hipStream_t s) {
  constexpr int W = EPI == EPI_QKV || EPI == EPI_KV || EPI == EPI_SWIGLU ? 16 : 4;
  const dim3 block(64 * W);
  if (norm) ADEPT_LAUNCH((gemm_f32_mfma_kernel<EPI, true, W>), grid, block, 0, s, p, kv);
  else ADEPT_LAUNCH((gemm_f32_mfma_kernel<EPI, false, W>), grid, block, 0, s, p, kv);
  return launch_status("gemm_f32");
}

template <int EPI> adept_status launch_f32_epi(const GP& p, bool norm, hipStream_t s) {
  const int cols = EPI == EPI_QKV ? p.N / 2 : p.N;
  return launch_f32_grid<EPI>(p, KvF32{}, dim3(ceil_div(p.M_max, 16), ceil_div(cols, 16)), norm, s);
}

adept_status launch_f32(const GemmArgs& g, hipStream_t s) {
  const GP p = to_gp(g);
  switch (g.epi) {
    case EPI_STORE: return launch_f32_epi<EPI_STORE>(p, g.row_norm, s);
    case EPI_RESID: return launch_f32_epi<EPI_RESID>(p, g.row_norm, s);
    case EPI_SWIGLU: return launch_f32_epi<EPI_SWIGLU>(p, g.row_norm, s);
    default: return launch_f32_epi<EPI_QKV>(p, g.row_norm, s);
  }
}

// ---------------------------------------------------------------------------
// general form
// ---------------------------------------------------------------------------
constexpr int FT = 64, FK = 16;

__global__ __launch_bounds__(256) void gemm_f32_kernel(int M_max, const int32_t* M_dev, int N,
                                                       int K, const float* __restrict__ A,
                                                       const int32_t* __restrict__ a_rows,
                                                       int64_t lda, const float* __restrict__ B,
                                                       int64_t ldb, float* __restrict__ C,
                                                       int64_t ldc) {
  __shared__ float sA[FK][FT + 1];
  __shared__ float sB[FK][FT + 1];
  const int M = M_dev ? min(*M_dev, M_max) : M_max;
  const int m0 = blockIdx.x * FT, n0 = blockIdx.y * FT;
  if (m0 >= M) return;
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  float acc[4][4] = {};
  for (int k0 = 0; k0 < K; k0 += FK) {
    for (int e = threadIdx.x; e < FT * FK; e += 256) {
      const int r = e / FK, c = e % FK;
      int m = m0 + r;
      if (m >= M) m = m0;
      const int arow = a_rows ? a_rows[m] : m;
      sA[c][r] = (k0 + c < K) ? A[(int64_t)arow * lda + k0 + c] : 0.0f;
      const int n = n0 + r;
      sB[c][r] = (n < N && k0 + c < K) ? B[(int64_t)n * ldb + k0 + c] : 0.0f;
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < FK; ++c) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = sA[c][ty * 4 + i];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = sB[c][tx * 4 + j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = m0 + ty * 4 + i;
    if (m >= M) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = n0 + tx * 4 + j;
      if (n < N) C[(int64_t)m * ldc + n] = acc[i][j];
    }
  }
}

// Element-wise epilogue over the f32 scratch T[m][n] (n < n_out), after the
// per-row scale.
__global__ void epilogue_f32_kernel(int epi, int M_max, const int32_t* M_dev, int n_out,
                                    const float* __restrict__ T, int64_t ldt, GP p) {
  const int M = M_dev ? min(*M_dev, M_max) : M_max;
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int m = (int)(idx / n_out), n = (int)(idx % n_out);
  if (m >= M) return;
  const float sc = p.row_scale ? p.row_scale[m] : 1.0f;
  const float* t = T + (int64_t)m * ldt;
  float* C = reinterpret_cast<float*>(p.C);
  if (epi == EPI_STORE) {
    C[(int64_t)m * p.ldc + n] = t[n] * sc;
  } else if (epi == EPI_RESID) {
    const int64_t row = p.rows[m];
    C[row * p.ldc + n] = reinterpret_cast<const float*>(p.resid)[row * p.ldc + n] + t[n] * sc;
  } else if (epi == EPI_SWIGLU) {
    C[(int64_t)m * p.ldc + n] = silu(t[n] * sc) * (t[p.N + n] * sc);
  } else {  // EPI_QKV
    const int sec = n / p.d_q, cin = n - sec * p.d_q;
    const int row = p.rows[m];
    float* dst;
    if (sec == 0) dst = reinterpret_cast<float*>(p.q_out) + (int64_t)m * p.d_q;
    else dst = reinterpret_cast<float*>(sec == 1 ? p.k_cache : p.v_cache) + (int64_t)p.slot[row] * p.d_q;
    if (sec == 2) {
      dst[cin] = t[n] * sc;
    } else {
      const int hd = p.head_dim, half = hd / 2;
      const int c = cin % hd, kk = c % half;
      const int ps = p.pos[row];
      const float cs = p.rope_cos[(int64_t)ps * half + kk], sn = p.rope_sin[(int64_t)ps * half + kk];
      const float x = t[n] * sc;
      const float y = (c < half ? t[n + half] : t[n - half]) * sc;
      dst[cin] = c < half ? x * cs - y * sn : x * cs + y * sn;
    }
  }
}

}  // namespace

// Rows and columns past the grid's 65535 y blocks, or leading dimensions that
// break the 16-byte loads, take the general form, and so do outputs of many 64x64
// tiles: a 16x16 block reads its operands four times as often as the general
// form's tile, and once that has one or two workgroups per CU this decides.  The
// two-block epilogues share the A block, so their line lies at twice the tiles.
// Two layers, us, this kernel throughout / general form throughout / by this
// rule: width 768, 512 rows 1637 / 2846 / 1644, 2048 rows 7772 / 5322 / 5316;
// width 4096, 128 rows 6511 / 12622 / 6508, 1024 rows 51800 / 24122 / 24041.
bool gemm_f32_fused(const GemmArgs& g) {
  const bool two = g.epi == EPI_QKV || g.epi == EPI_SWIGLU;
  if ((int64_t)ceil_div(g.M_max, FT) * ceil_div(g.N, FT) >= (two ? 512 : 256)) return false;
  const bool kind = g.epi == EPI_STORE || g.epi == EPI_RESID || g.epi == EPI_SWIGLU ||
                    (g.epi == EPI_QKV && g.head_dim % 32 == 0 && g.d_q % g.head_dim == 0);
  return kind && g.N > 0 && g.N <= 16 * 65535 && g.K > 0 && g.K % 4 == 0 && g.lda % 4 == 0 &&
         g.ldb % 4 == 0 && aligned16(g.A) && aligned16(g.B) && (!g.B2 || aligned16(g.B2));
}

adept_status kvgen_f32_fused(const GemmArgs& g, int n_layers, const int32_t* exit_layer,
                             const float* gain, int64_t b_layer_stride,
                             int64_t cache_layer_stride, bool* ran, hipStream_t s) {
  *ran = g.head_dim % 32 == 0 && g.N <= 32 * 65535 && n_layers <= 65535 && g.K % 4 == 0 &&
         g.lda % 4 == 0 && g.ldb % 4 == 0 && b_layer_stride % 4 == 0 && aligned16(g.A) &&
         aligned16(g.B) && (!gain || aligned16(gain));
  if (!*ran) return ADEPT_OK;
  GP p = to_gp(g);
  p.b_layer_stride = b_layer_stride;
  p.cache_layer_stride = cache_layer_stride;
  return launch_f32_grid<EPI_KV>(p, KvF32{exit_layer, gain},
                                 dim3(ceil_div(p.M_max, 16), p.N / 32, n_layers), true, s);
}

// f32 GEMM + element-wise epilogue; tmp holds M_max x (N or 2N for SWIGLU) floats.
adept_status gemm_f32(const GemmArgs& g, float* tmp, hipStream_t s) {
  if (g.M_max <= 0) return ADEPT_OK;
  if (gemm_f32_fused(g)) return launch_f32(g, s);
  if (g.row_norm) {
    set_error("gemm_f32: row_norm only where gemm_f32_fused holds");
    return ADEPT_E_INVALID;
  }
  const int nt = g.epi == EPI_SWIGLU ? 2 * g.N : g.N;
  dim3 block(256);
  dim3 grid(ceil_div(g.M_max, FT), ceil_div(g.N, FT));
  ADEPT_LAUNCH(gemm_f32_kernel, grid, block, 0, s, g.M_max, g.M_dev, g.N, g.K,
               (const float*)g.A, g.a_rows, g.lda, (const float*)g.B, g.ldb, tmp, (int64_t)nt);
  ADEPT_CHECK_LAUNCH("gemm_f32");
  if (g.epi == EPI_SWIGLU) {
    ADEPT_LAUNCH(gemm_f32_kernel, grid, block, 0, s, g.M_max, g.M_dev, g.N, g.K,
                 (const float*)g.A, g.a_rows, g.lda, (const float*)g.B2, g.ldb, tmp + g.N,
                 (int64_t)nt);
    ADEPT_CHECK_LAUNCH("gemm_f32");
  }
  GP p = to_gp(g);
  const int64_t total = (int64_t)g.M_max * g.N;
  ADEPT_LAUNCH(epilogue_f32_kernel, dim3((unsigned)((total + 255) / 256)), block, 0, s, g.epi,
               g.M_max, g.M_dev, g.N, (const float*)tmp, (int64_t)nt, p);
  return launch_status("epilogue_f32");
}

// f32 GEMM written straight to C (no epilogue, no row scale): C[m][n] = A[m] . B[n].
adept_status gemm_f32_direct(const GemmArgs& g, hipStream_t s) {
  if (g.M_max <= 0) return ADEPT_OK;
  if (gemm_f32_fused(g)) return launch_f32(g, s);
  dim3 grid(ceil_div(g.M_max, FT), ceil_div(g.N, FT));
  ADEPT_LAUNCH(gemm_f32_kernel, grid, dim3(256), 0, s, g.M_max, g.M_dev, g.N, g.K,
               (const float*)g.A, g.a_rows, g.lda, (const float*)g.B, g.ldb, (float*)g.C, g.ldc);
  return launch_status("gemm_f32");
}

}  // namespace adept
