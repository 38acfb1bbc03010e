// bf16 GEMMs of at most 64 rows (decode, short prompts, the head of a few
// rows): one kernel, operands straight from global memory to the registers of
// v_mfma_f32_16x16x32_bf16, epilogue included.
//
// A workgroup of eight waves owns 16 or 32 weight rows (NB blocks of 16) and
// all M activation rows (MB blocks of 16).  Its waves take every eighth
// 64-deep (one cache line) piece of K; their f32 sums meet in LDS, in wave
// order, where the epilogue runs.  The weights cross HBM once, non-temporal;
// the activations (at most 64 rows) come from L2.  With the weights as the
// instruction's first operand a lane ends up with four consecutive output
// columns of one row, the unit the epilogues work on.
//
// What bounds these GEMMs is the weights' HBM time for wide layers and, for
// narrow ones, the chain of a kernel: its start, the row count, the row list,
// the operands, the hand-over of the sums.  So there is one kernel where a
// split over K with partial tiles in memory took two, the first weight loads
// are issued before the row count is known, and the row's RMSNorm factor and
// the row list of the fused decode schedule are formed on the way instead of
// by kernels of their own.  Measured, us, GEMM and epilogue kernel of the
// split form -> this one: 7B width, 1 row, a layer's four GEMMs with their
// norms and row list 131 -> 102 (4.5 TB/s of weights in gate/up); width 1600,
// 24 rows, QKV / first MLP 13.5 / 13.0 -> 11.0 / 10.3; width 768, 48 rows, biased
// QKV 9.4 -> 6.8, in the skinny path's order (SPLIT) 8.0.
#include "gemm_tile.h"

namespace adept {
namespace {

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// What the epilogue of one thread's four columns (n.. of row m) reads, loaded
// beside the first operands: each would be one more memory latency at the end.
struct DirPre {
  int m, n, row, slot;
  bool out;          // this lane stores (SwiGLU: the gate lanes)
  bf16x4_t bias, resid;
  float4 cs, sn;
  float sc;
};

// NB == 1 with a pair epilogue (rotary halves, gate and up): the 16 rows of the
// block are 8 of the first kind and their 8 partners.
//
// SPLIT: the sums in the order of the skinny path (gemm.hip), bit for bit: K in
// the segments its split sp gives these columns' tile, each one chain from zero,
// added up in ascending order.  The waves take every eighth segment.
template <int EPI, int NB, int MB, int W, int U, bool SPLIT>
__global__ __launch_bounds__(64 * W) void gemm_direct_kernel(GP p, RowList rl, int row_norm,
                                                             SkSplit sp) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  float4* red = reinterpret_cast<float4*>(smem);      // [wave or segment][MB * NB][64]
  __shared__ float ssq[W][MB * 16];
  __shared__ int32_t list[64];
  __shared__ uint8_t from2[64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r16 = lane & 15, q = lane >> 4;
  const int KT = p.K / BK;
  const bool rope = EPI == EPI_QKV && p.rope_cos;
  const bool pair = EPI == EPI_SWIGLU || rope;
  // the first kind's first column, rows per kind, and the distance to the
  // second kind (SwiGLU's is in B2)
  const int per = pair && NB == 1 ? 8 : 16;
  int n0, dn = 16;
  if (rope) {
    dn = p.head_dim >> 1;
    const int cpb = dn / per;   // blocks per head
    n0 = (int)blockIdx.x / cpb * p.head_dim + (int)blockIdx.x % cpb * per;
  } else {
    n0 = blockIdx.x * (EPI == EPI_SWIGLU ? per : 16 * NB);
  }
  // raw list entries: loaded before the row count is known, used below it
  int raw[MB];
#pragma unroll
  for (int y = 0; y < MB; ++y)
    raw[y] = !rl.exit_layer && p.a_rows ? p.a_rows[min(16 * y + r16, p.M_max - 1)] : 16 * y + r16;
  constexpr int XB = EPI == EPI_SWIGLU ? 1 : NB;
  constexpr int G = (MB * XB + W - 1) / W;            // epilogue groups of a wave
  DirPre pre[G];
  constexpr bool kRows = EPI == EPI_RESID || EPI == EPI_QKV;
#pragma unroll
  for (int i = 0; i < G; ++i) {
    const int t = wave + W * i, y = t / XB;
    pre[i].m = 16 * y + r16;
    pre[i].row = kRows && !rl.exit_layer ? p.rows[min(pre[i].m, p.M_max - 1)] : 0;
  }
  int el = INT_MAX, act = 0;
  if (rl.exit_layer) {
    if (lane < rl.n_tok) {
      el = rl.exit_layer[lane];
      act = rl.act[lane];
    }
  }
  // SPLIT: the segments of K, numbered from sp's first workgroup of the tile that
  // holds these columns
  [[maybe_unused]] const int u0 = SPLIT ? n0 / kSkinnyBN * KT : 0, w0 = SPLIT ? u0 / sp.U : 0;
  const int nseg = SPLIT ? (u0 + KT - 1) / sp.U - w0 + 1 : W;
  auto lo_of = [&](int s) { return max((w0 + s) * sp.U - u0, 0); };
  auto hi_of = [&](int s) { return min((w0 + s + 1) * sp.U - u0, KT); };
  const bf16* br[NB];
  {
    const bool two = NB == 1 && pair && r16 >= 8;   // a lane of the second kind
    const int r = two ? r16 - 8 : r16;
    br[0] = (EPI == EPI_SWIGLU && two ? p.B2 + (int64_t)(n0 + r) * p.ldb
                                      : p.B + (int64_t)(n0 + r + (two ? dn : 0)) * p.ldb) + 8 * q;
    if constexpr (NB == 2)
      br[1] = (EPI == EPI_SWIGLU ? p.B2 + (int64_t)(n0 + r16) * p.ldb
                                 : p.B + (int64_t)(n0 + dn + r16) * p.ldb) + 8 * q;
  }
  u32x4_t bw[2][U][NB][2], aw[2][U][MB][2];
  // a stage: up to U pieces of K from c0 on, below hi
  constexpr int kStep = SPLIT ? 1 : W;
  auto load_b = [&](int c0, int hi, u32x4_t (&b)[U][NB][2]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int c = c0 + u * kStep;
      if (c >= hi) continue;   // uniform over the wave
#pragma unroll
      for (int x = 0; x < NB; ++x)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          b[u][x][h] = __builtin_nontemporal_load(
              reinterpret_cast<const u32x4_t*>(br[x] + (int64_t)c * BK + 32 * h));
    }
  };
  if constexpr (SPLIT) {
    if (wave < nseg) load_b(lo_of(wave), hi_of(wave), bw[0]);
  } else {
    load_b(wave, KT, bw[0]);
  }

  // the rows: active rows, then (row list) the rows that exited before the
  // layer, in one ballot of at most 64 token rows
  int M = p.M_dev ? min(*p.M_dev, rl.exit_layer ? rl.max_act : p.M_max) : p.M_max;
  if (rl.ticket && blockIdx.x == 0 && threadIdx.x < 2) rl.ticket[threadIdx.x] = 0ull;
  const bf16* ar[MB];
  if (rl.exit_layer) {
    const int na = M;
    const bool ex = el < rl.layer;
    const uint64_t gone = __ballot(ex);
    M = min(na + __popcll(gone), 64);
    if (wave == 0) {
      const int at = na + __popcll(gone & ((1ull << lane) - 1));
      if (lane < na) {
        list[lane] = act;
        from2[lane] = 0;
      }
      if (ex && at < 64) {
        list[at] = lane;
        from2[at] = (el & 1) != ((rl.layer - 1) & 1);
      }
    }
    __syncthreads();
    if (M <= 0) return;
#pragma unroll
    for (int y = 0; y < MB; ++y) {
      const int m = min(16 * y + r16, M - 1);
      ar[y] = (from2[m] ? p.A2 : p.A) + (int64_t)list[m] * p.lda + 8 * q;
    }
#pragma unroll
    for (int i = 0; i < G; ++i) pre[i].row = list[min(pre[i].m, M - 1)];
  } else {
    if (M <= 0) return;
#pragma unroll
    for (int y = 0; y < MB; ++y) {
      // rows past the count: row 0, computed and never stored
      const int row = 16 * y + r16 < M ? raw[y] : 0;
      ar[y] = ((p.a_sel && (p.a_sel[row] & 1)) ? p.A2 : p.A) + (int64_t)row * p.lda + 8 * q;
    }
#pragma unroll
    for (int i = 0; i < G; ++i)
      if (pre[i].m >= M) pre[i].row = 0;
  }
  auto load_a = [&](int c0, int hi, u32x4_t (&a)[U][MB][2]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int c = c0 + u * kStep;
      if (c >= hi) continue;
#pragma unroll
      for (int y = 0; y < MB; ++y)
        if (y == 0 || 16 * y < M) {
#pragma unroll
          for (int h = 0; h < 2; ++h)
            a[u][y][h] = *reinterpret_cast<const u32x4_t*>(ar[y] + (int64_t)c * BK + 32 * h);
        }
    }
  };
  if constexpr (SPLIT) {
    if (wave < nseg) load_a(lo_of(wave), hi_of(wave), aw[0]);
  } else {
    load_a(wave, KT, aw[0]);
  }
  // the epilogue's inputs
#pragma unroll
  for (int i = 0; i < G; ++i) {
    DirPre& e = pre[i];
    const int t = wave + W * i, x = t % XB;
    const int kind = per == 8 ? q >> 1 : x;           // of a pair
    e.out = t < MB * XB && e.m < M && !(EPI == EPI_SWIGLU && kind);
    e.n = n0 + (per == 8 ? (EPI == EPI_SWIGLU ? 0 : kind * dn) + 4 * (q & 1) : x * dn + 4 * q);
    e.sc = 1.0f;
    e.bias = bf16x4_t{0, 0, 0, 0};
    if (!e.out) continue;
    if (p.row_scale) e.sc = p.row_scale[e.m];
    if (p.bias) e.bias = *reinterpret_cast<const bf16x4_t*>(p.bias + e.n);
    if constexpr (EPI == EPI_RESID)
      e.resid = *reinterpret_cast<const bf16x4_t*>(p.resid + (int64_t)e.row * p.ldc + e.n);
    if constexpr (EPI == EPI_QKV) {
      e.slot = p.slot ? p.slot[e.row] : e.row;
      if (rope) {
        const int64_t o = (int64_t)p.pos[e.row] * dn + (e.n & (dn - 1));
        e.cs = rope4(p.rope_cos + o);
        e.sn = rope4(p.rope_sin + o);
      }
    }
  }
  f32x4_t acc[MB][NB];
  float ss[MB];
#pragma unroll
  for (int y = 0; y < MB; ++y) {
    ss[y] = 0.0f;
#pragma unroll
    for (int x = 0; x < NB; ++x) acc[y][x] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  }
  auto step = [&](int c0, int hi, u32x4_t (&a)[U][MB][2], u32x4_t (&b)[U][NB][2]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (c0 + u * kStep >= hi) continue;
#pragma unroll
      for (int y = 0; y < MB; ++y)
        if (y == 0 || 16 * y < M) {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const bf16x8_t av = __builtin_bit_cast(bf16x8_t, a[u][y][h]);
#pragma unroll
            for (int x = 0; x < NB; ++x)
              acc[y][x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                  __builtin_bit_cast(bf16x8_t, b[u][x][h]), av, acc[y][x], 0, 0, 0);
            if (row_norm) {
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const float lo = __uint_as_float(a[u][y][h][e] << 16);
                const float hi = __uint_as_float(a[u][y][h][e] & 0xffff0000u);
                ss[y] = fmaf(lo, lo, ss[y]);
                ss[y] = fmaf(hi, hi, ss[y]);
              }
            }
          }
        }
    }
  };
  auto hand_over = [&](int s) {   // the sums of segment s
#pragma unroll
    for (int y = 0; y < MB; ++y)
#pragma unroll
      for (int x = 0; x < NB; ++x)
        red[(s * MB * NB + y * NB + x) * 64 + lane] =
            make_float4(acc[y][x][0], acc[y][x][1], acc[y][x][2], acc[y][x][3]);
  };
  if constexpr (SPLIT) {
    // stage (s, c): pieces c.. of segment s; the next one may open the wave's
    // next segment, whose loads then pass the hand-over
    auto next = [&](int& s, int& c) {
      c += U;
      if (c >= hi_of(s)) {
        s += W;
        c = lo_of(s);
      }
    };
    auto finish = [&](int s) {
      hand_over(s);
#pragma unroll
      for (int y = 0; y < MB; ++y)
#pragma unroll
        for (int x = 0; x < NB; ++x) acc[y][x] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    };
    int s = wave, c = lo_of(wave);
#pragma unroll 1
    while (s < nseg) {
      int s1 = s, c1 = c;
      next(s1, c1);
      if (s1 < nseg) {
        load_b(c1, hi_of(s1), bw[1]);
        load_a(c1, hi_of(s1), aw[1]);
      }
      step(c, hi_of(s), aw[0], bw[0]);
      if (s1 != s) finish(s);
      s = s1;
      c = c1;
      if (s >= nseg) break;
      next(s1, c1);
      if (s1 < nseg) {
        load_b(c1, hi_of(s1), bw[0]);
        load_a(c1, hi_of(s1), aw[0]);
      }
      step(c, hi_of(s), aw[1], bw[1]);
      if (s1 != s) finish(s);
      s = s1;
      c = c1;
    }
  } else {
    const int mine = KT > wave ? (KT - wave + W - 1) / W : 0;   // this wave's pieces of K
    const int iters = (mine + U - 1) / U;
    auto at = [&](int it) { return it * U * W + wave; };
#pragma unroll 1
    for (int it = 0; it < iters; it += 2) {
      if (it + 1 < iters) {
        load_b(at(it + 1), KT, bw[1]);
        load_a(at(it + 1), KT, aw[1]);
      }
      step(at(it), KT, aw[0], bw[0]);
      if (it + 1 < iters) {
        if (it + 2 < iters) {
          load_b(at(it + 2), KT, bw[0]);
          load_a(at(it + 2), KT, aw[0]);
        }
        step(at(it + 1), KT, aw[1], bw[1]);
      }
    }
    hand_over(wave);   // a wave without pieces: zeros
  }
  if (row_norm) {
#pragma unroll
    for (int y = 0; y < MB; ++y) {
      float s = ss[y];
      s += __shfl_xor(s, 16, 64);
      s += __shfl_xor(s, 32, 64);
      if (q == 0) ssq[wave][16 * y + r16] = s;
    }
  }
  __syncthreads();
  // lane l of block (y, x): row 16 y + l % 16, four columns by l / 16
  auto sum = [&](int blk, int l) {
    float4 t = SPLIT ? make_float4(0.f, 0.f, 0.f, 0.f) : red[blk * 64 + l];
    auto add = [&](int w) {
      const float4 o = red[(w * MB * NB + blk) * 64 + l];
      t.x += o.x; t.y += o.y; t.z += o.z; t.w += o.w;
    };
    if constexpr (SPLIT) {
#pragma unroll 4
      for (int w = 0; w < nseg; ++w) add(w);
    } else {
#pragma unroll
      for (int w = 1; w < W; ++w) add(w);
    }
    return t;
  };
#pragma unroll
  for (int i = 0; i < G; ++i) {
    const DirPre& e = pre[i];
    if (!e.out) continue;
    const int t = wave + W * i, y = t / XB, x = t % XB;
    float sc = e.sc;
    if (row_norm) {
      float s = 0.0f;
#pragma unroll
      for (int w = 0; w < W; ++w) s += ssq[w][e.m];
      sc = 1.0f / sqrtf(s / (float)p.K + p.row_eps);
    }
    const float4 x4 = sum(y * NB + x, lane);
    const float bx[4] = {bf2f(e.bias[0]), bf2f(e.bias[1]), bf2f(e.bias[2]), bf2f(e.bias[3])};
    float v[4] = {x4.x * sc + bx[0], x4.y * sc + bx[1], x4.z * sc + bx[2], x4.w * sc + bx[3]};
    bf16x4_t o;
    if constexpr (EPI == EPI_STORE) {
      if (p.c_f32) {
        *reinterpret_cast<float4*>(reinterpret_cast<float*>(p.C) + (int64_t)e.m * p.ldc + e.n) =
            make_float4(v[0], v[1], v[2], v[3]);
        continue;
      }
    }
    bf16* dst = reinterpret_cast<bf16*>(p.C) + (int64_t)(EPI == EPI_RESID ? e.row : e.m) * p.ldc + e.n;
    if constexpr (EPI == EPI_SWIGLU) {
      const float4 y4 = per == 8 ? sum(y, lane ^ 32) : sum(y * NB + NB - 1, lane);
      const float u[4] = {y4.x * sc, y4.y * sc, y4.z * sc, y4.w * sc};
#pragma unroll
      for (int c = 0; c < 4; ++c) o[c] = f2bf(silu(v[c]) * u[c]);
    } else if constexpr (EPI == EPI_QKV) {
      const int sec = e.n / p.d_q, cin = e.n - sec * p.d_q;
      dst = (sec == 0 ? p.q_out + (int64_t)e.m * p.d_q
                      : (sec == 2 ? p.v_cache : p.k_cache) + (int64_t)e.slot * p.d_q) + cin;
      if (rope && sec != 2) {
        const bool first = per == 8 ? q < 2 : x == 0;
        const float4 y4 = per == 8 ? sum(y, lane ^ 32) : sum(y * NB + (x ^ (NB - 1)), lane);
        const float4 by = bias4(p.bias, first ? e.n + dn : e.n - dn);
        const float w[4] = {y4.x * sc + by.x, y4.y * sc + by.y, y4.z * sc + by.z, y4.w * sc + by.w};
        const float cv[4] = {e.cs.x, e.cs.y, e.cs.z, e.cs.w};
        const float sv[4] = {e.sn.x, e.sn.y, e.sn.z, e.sn.w};
#pragma unroll
        for (int c = 0; c < 4; ++c)
          o[c] = f2bf(first ? v[c] * cv[c] - w[c] * sv[c] : v[c] * cv[c] + w[c] * sv[c]);
      } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) o[c] = f2bf(v[c]);
      }
    } else {
      if constexpr (EPI == EPI_GELU) gelu_erf(v);
#pragma unroll
      for (int c = 0; c < 4; ++c)
        o[c] = f2bf(EPI == EPI_GELU_TANH   ? gelu_tanh(v[c])
                    : EPI == EPI_RESID     ? v[c] + bf2f(e.resid[c])
                                           : v[c]);
    }
    *reinterpret_cast<bf16x4_t*>(dst) = o;
  }
}

// LDS of a SPLIT workgroup's sums: at most this (beside the static arrays)
constexpr size_t kSplitLds = 128 * 1024;
// the most segments a tile has
int split_segments(const SkSplit& sp) {
  return sp.KT % sp.U == 0 ? sp.KT / sp.U : (sp.KT + sp.U - 2) / sp.U + 1;
}

template <int EPI, int NB, int MB, int W, int U, bool SPLIT>
adept_status dir_launch(const GP& p, const RowList& rl, int row_norm, const char* name,
                        hipStream_t s) {
  SkSplit sp{};
  int parts = W;
  if (SPLIT) {
    sp = skinny_split(p.N, p.K);
    parts = split_segments(sp);
  }
  const size_t red = (size_t)parts * MB * NB * 1024;
  static bool attr_set = false;
  if (SPLIT || red > 48 * 1024)
    ADEPT_TRY(lds_limit((const void*)gemm_direct_kernel<EPI, NB, MB, W, U, SPLIT>,
                        SPLIT ? kSplitLds : red, &attr_set, "gemm_direct LDS limit"));
  const int cols = EPI == EPI_SWIGLU ? 8 * NB : 16 * NB;
  {
    TimedLaunch tl(name ? name : "gemm_direct", s);
    hipLaunchKernelGGL((gemm_direct_kernel<EPI, NB, MB, W, U, SPLIT>), dim3(p.N / cols),
                       dim3(64 * W), red, s, p, rl, row_norm, sp);
  }
  return launch_status("gemm_direct");
}

// 32 weight rows per workgroup where they still give half the chip one: the
// activations are read half as often (24 rows, width 1600: QKV 14.0 -> 11.0 us
// with 150 workgroups, but the O and down projections 12.4 -> 18.1 with 50)
bool dir_wide(int N, int epi) { return (epi == EPI_SWIGLU ? N / 16 : N / 32) >= 128; }

template <int EPI, bool SPLIT>
adept_status dir_rows(const GP& p, const RowList& rl, int row_norm, const char* name,
                      hipStream_t s) {
  const int M = rl.exit_layer ? rl.n_tok : p.M_max;
  // one piece of K in flight per stage for QKV, whose workgroups (768 of them at
  // the 7B width) are short and start with the row list: more of them per CU
  // (28 -> 24 us); two for the others (down and O projections 18 -> 15.6).
  // SPLIT: a wave's segment is four pieces at least and few waves have one (three
  // at K = 768), so its loads are issued together (twelve layers of width 768:
  // 12 rows 524 -> 500 us, 40 rows 687 -> 661)
  if (M <= 16)
    return dir_launch<EPI, 1, 1, 8, SPLIT ? 4 : EPI == EPI_QKV ? 1 : 2, SPLIT>(p, rl, row_norm, name,
                                                                               s);
  const bool wide = dir_wide(p.N, EPI);
  if (M <= 32)
    return wide ? dir_launch<EPI, 2, 2, 8, 2, SPLIT>(p, rl, row_norm, name, s)
                : dir_launch<EPI, 1, 2, 8, SPLIT ? 4 : 2, SPLIT>(p, rl, row_norm, name, s);
  return wide ? dir_launch<EPI, 2, 4, 8, 1, SPLIT>(p, rl, row_norm, name, s)
              : dir_launch<EPI, 1, 4, 8, SPLIT ? 2 : 1, SPLIT>(p, rl, row_norm, name, s);
}

}  // namespace

// Up to 16 rows, or up to 64 of narrow layers.  With more rows each workgroup
// reads up to 64 activation rows for 16 or 32 weight rows, and the load path of
// the CUs binds: at the 7B widths and 64 rows 35 to 73 us a GEMM, 16 to 43 for
// the skinny path's two kernels; at width 1600 (10 M weights) a decode step of
// 24 rows 4000 us against 4530, of 40 4471 against 4661, of 48 the same, of 64
// 5412 against 5141; two layers of width 1600, 40 / 48 / 64 rows 152 / 162 / 185
// against 156 / 153 / 160.  Past 40 rows the line lies below the least width that
// lost (LayerNorm family, width 1024, 4.2 M: 48 / 64 rows 122 / 137 against 124 /
// 128), at the widest that was measured to win (width 768, 2.36 M: 108 / 118
// against 118 / 121); steps of the RMSNorm family would win up to 5.8 M (width 1024,
// 48 rows 103 against 127).  A step takes the form for all its GEMMs or none
// (layer.hip, encoder.hip).
// Plain stores (the head) of wide layers stream better through the tiles of
// gemm_mid.h (6 rows, 32000 x 4096: 52 us, 58 here).
bool gemm_direct_fits(int M_max, int n_weights, int K, int epi) {
  const int64_t weights = (int64_t)n_weights * K;
  const bool narrow = weights <= (M_max <= 40 ? 12 << 20 : 2400000);
  return M_max > 0 && M_max <= kDirectRows && epi != EPI_KV &&
         (narrow || (M_max <= 16 && epi != EPI_STORE));
}

bool gemm_direct_split_fits(int M_max, int N, int K, int epi) {
  if (epi == EPI_SWIGLU || !gemm_direct_fits(M_max, N, K, epi) || N % kSkinnyBN != 0) return false;
  const SkSplit sp = skinny_split(N, K);
  const int mb = M_max <= 16 ? 1 : M_max <= 32 ? 2 : 4, nb = M_max > 16 && dir_wide(N, epi) ? 2 : 1;
  return sp.G > 0 && (size_t)split_segments(sp) * mb * nb * 1024 <= kSplitLds;
}

bool gemm_direct_fits(const GemmArgs& g) {
  if (g.few_rows == kFewSkinny) return false;
  if (g.few_rows == kFewSplit) return !g.rope_cos && gemm_direct_split_fits(g.M_max, g.N, g.K, g.epi);
  return gemm_direct_fits(g.M_max, g.epi == EPI_SWIGLU ? 2 * g.N : g.N, g.K, g.epi);
}

adept_status gemm_direct(const GemmArgs& g, hipStream_t s) {
  const GP p = to_gp(g);
  const RowList rl = g.list ? *g.list : RowList{};
  const int rn = g.row_norm ? 1 : 0;
  if (g.few_rows == kFewSplit) {
    switch (g.epi) {
      case EPI_QKV: return dir_rows<EPI_QKV, true>(p, rl, rn, g.name, s);
      case EPI_RESID: return dir_rows<EPI_RESID, true>(p, rl, rn, g.name, s);
      case EPI_GELU: return dir_rows<EPI_GELU, true>(p, rl, rn, g.name, s);
      default: break;
    }
    set_error("gemm: few_rows = split without this epilogue");
    return ADEPT_E_INVALID;
  }
  switch (g.epi) {
    case EPI_STORE: return dir_rows<EPI_STORE, false>(p, rl, rn, g.name, s);
    case EPI_QKV: return dir_rows<EPI_QKV, false>(p, rl, rn, g.name, s);
    case EPI_RESID: return dir_rows<EPI_RESID, false>(p, rl, rn, g.name, s);
    case EPI_SWIGLU: return dir_rows<EPI_SWIGLU, false>(p, rl, rn, g.name, s);
    case EPI_GELU: return dir_rows<EPI_GELU, false>(p, rl, rn, g.name, s);
    case EPI_GELU_TANH: return dir_rows<EPI_GELU_TANH, false>(p, rl, rn, g.name, s);
    default: set_error("gemm: bad epilogue"); return ADEPT_E_INVALID;
  }
}

}  // namespace adept
