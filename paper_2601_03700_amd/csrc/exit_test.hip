// Token-level exit test (Section 4.1, Eq. 7-8; local metric of Appendix H.3).
//
// One wavefront per active row.  Per chunk c each lane holds E consecutive
// elements of h starting at element (c*64 + lane)*E, with E = 4 for the
// global metric (8 bytes of bf16 h beside one contiguous 16-byte vector of
// the f32 inertia) and E = 16/sizeof(T) for the local one, so that every
// load and store instruction of the wave covers one contiguous span.  The
// values stay in registers in their stored form between the reduction and
// the inertia update; the three sums <h,h>, <r,r>, <h,r> are accumulated in
// double (every product of two float values is exact in double), a xor
// butterfly reduces across the wave and the decision is taken in double.
// For the global metric the inertia row is then updated from the registers,
// so each byte of h and of the inertia crosses HBM once (read h, read +
// write inertia).  Every access is streaming (non-temporal): nothing the
// kernel touches is read again before it has left the caches.  The combined
// metric (both cosines must reach the threshold) reads h, h_prev and the
// inertia with the global metric's grouping (4 elements per lane and chunk)
// and keeps five sums.
#include "common.h"

namespace adept {
namespace {

constexpr int kWavesPerBlock = 4;
constexpr int kMaxChunks = 32;
constexpr int kMaxChunksBoth = 16;   // three row streams in registers

enum Mode { kLocal = 0, kGlobal = 1, kBoth = 2 };

struct ExitParams {
  double delta;
  int min_exit_layer, n_layers, layer, d;
};

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
template <int BYTES> struct Raw;
template <> struct Raw<8> { using type = u32x2; };
template <> struct Raw<16> { using type = u32x4; };

// Element i of a raw vector of T, as float.
template <typename T, typename R> __device__ __forceinline__ float elem(const R& r, int i) {
  if constexpr (sizeof(T) == 4) {
    return __uint_as_float(r[i]);
  } else {
    const uint32_t w = r[i >> 1];
    return __uint_as_float((i & 1) ? (w & 0xffff0000u) : (w << 16));
  }
}

template <typename T, int CH, int MODE>
__global__ __launch_bounds__(64 * kWavesPerBlock)
void exit_test_kernel(
    ExitParams p, int max_active, const int32_t* __restrict__ rows,
    const int32_t* __restrict__ n_active,
    const T* __restrict__ h_cur, const T* __restrict__ h_prev, float* __restrict__ inertia,
    const int32_t* __restrict__ force_layer, uint8_t* __restrict__ exit_flag,
    double* __restrict__ sim_out) {
  constexpr bool GLOBAL = MODE != kLocal;   // reads and updates the inertia
  constexpr bool BOTH = MODE == kBoth;      // also reads h_prev
  constexpr int E = GLOBAL ? 4 : 16 / (int)sizeof(T);
  using HRaw = typename Raw<E * sizeof(T)>::type;
  using RRaw = u32x4;   // 4 f32 of the inertia, or E values of h_prev
  const int lane = threadIdx.x & 63;
  const int k = blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
  if (k >= min(*n_active, max_active)) return;
  const int row = rows[k];
  const int nvec = p.d / E;
  const T* hr = h_cur + (int64_t)row * p.d;
  const uint32_t* rr = GLOBAL ? reinterpret_cast<const uint32_t*>(inertia + (int64_t)row * p.d)
                              : reinterpret_cast<const uint32_t*>(h_prev + (int64_t)row * p.d);

  const T* pr = BOTH ? h_prev + (int64_t)row * p.d : nullptr;   // combined metric only

  HRaw hv[CH];
  RRaw rv[CH];
  HRaw pv[BOTH ? CH : 1];
  // Loads are not predicated: a lane past the end of the row re-reads the
  // row's last vector and contributes zeros (predicated loads leave the
  // register allocator with partially defined values and cost spills).
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const int vi = min(c * 64 + lane, nvec - 1);
    hv[c] = __builtin_nontemporal_load(reinterpret_cast<const HRaw*>(hr + vi * E));
    rv[c] = __builtin_nontemporal_load(reinterpret_cast<const RRaw*>(rr) + vi);
    if constexpr (BOTH) pv[c] = __builtin_nontemporal_load(reinterpret_cast<const HRaw*>(pr + vi * E));
  }
  double s_hh = 0.0, s_rr = 0.0, s_hr = 0.0, s_pp = 0.0, s_hp = 0.0;
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const bool live = c * 64 + lane < nvec;
#pragma unroll
    for (int v = 0; v < E; ++v) {
      const double a = live ? elem<T>(hv[c], v) : 0.0f;
      const double b = live ? (GLOBAL ? elem<float>(rv[c], v) : elem<T>(rv[c], v)) : 0.0f;
      s_hh = fma(a, a, s_hh);
      s_rr = fma(b, b, s_rr);
      s_hr = fma(a, b, s_hr);
      if constexpr (BOTH) {
        const double q = live ? elem<T>(pv[c], v) : 0.0f;
        s_pp = fma(q, q, s_pp);
        s_hp = fma(a, q, s_hp);
      }
    }
    // chunk by chunk: the conversions to double are not hoisted (and held
    // in registers) ahead of the chunk that needs them
    __builtin_amdgcn_sched_barrier(0);
  }
  s_hh = wave_sum_f64(s_hh);
  s_rr = wave_sum_f64(s_rr);
  s_hr = wave_sum_f64(s_hr);
  if constexpr (BOTH) {
    s_pp = wave_sum_f64(s_pp);
    s_hp = wave_sum_f64(s_hp);
  }

  const double kNaN = __longlong_as_double(0x7ff8000000000000ll);
  const double nh = sqrt(s_hh), nr = sqrt(s_rr);
  const double den = nh * nr;
  double sim = den > 0.0 ? s_hr / den : kNaN;
  bool pass = sim >= p.delta;
  if constexpr (BOTH) {
    // the local cosine must pass too; the reported similarity is the
    // smaller of the two (NaN if either is undefined)
    const double den_l = nh * sqrt(s_pp);
    const double sim_l = den_l > 0.0 ? s_hp / den_l : kNaN;
    pass = pass && sim_l >= p.delta;
    sim = (sim != sim || sim_l != sim_l) ? kNaN : fmin(sim, sim_l);
  }
  const bool ex = exit_decision(pass, p.layer, p.min_exit_layer, p.n_layers, force_layer, row);
  if (lane == 0) {
    exit_flag[k] = ex ? 1 : 0;
    if (sim_out) sim_out[k] = sim;
  }
  if (GLOBAL && nh > 0.0) {
    const double inv = 1.0 / nh;
    float* iw = inertia + (int64_t)row * p.d;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      // opaque to the optimiser: the values are converted again here rather
      // than kept in double registers since the reduction
      asm volatile("" : "+v"(hv[c]), "+v"(rv[c]));
      const int vi = c * 64 + lane;
      if (vi < nvec) {
        u32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          o[e] = __float_as_uint(
              (float)((double)elem<float>(rv[c], e) + (double)elem<T>(hv[c], e) * inv));
        __builtin_nontemporal_store(o, reinterpret_cast<u32x4*>(iw) + vi);
      }
    }
  }
}

template <typename T, int MODE>
adept_status launch_exit(int ch, const ExitParams& p, int max_active, const int32_t* rows,
                         const int32_t* n_active, const void* h_cur, const void* h_prev,
                         float* inertia, const int32_t* force, uint8_t* flag, double* sim,
                         hipStream_t s) {
  dim3 grid(ceil_div(max_active, kWavesPerBlock)), block(64 * kWavesPerBlock);
  const T* hc = (const T*)h_cur;
  const T* hp = (const T*)h_prev;
#define ADEPT_EXIT_CASE(C)                                                                     \
  case C:                                                                                      \
    ADEPT_LAUNCH((exit_test_kernel<T, C, MODE>), grid, block, 0, s, p, max_active, rows, n_active, \
                       hc, hp, inertia, force, flag, sim);                                     \
    break;
  switch (MODE == kBoth && ch > kMaxChunksBoth ? 0 : ch) {
    ADEPT_EXIT_CASE(1)
    ADEPT_EXIT_CASE(2)
    ADEPT_EXIT_CASE(4)
    ADEPT_EXIT_CASE(8)
    ADEPT_EXIT_CASE(16)
    case 32:
      if constexpr (MODE != kBoth) {
        ADEPT_LAUNCH((exit_test_kernel<T, 32, MODE>), grid, block, 0, s, p, max_active, rows,
                     n_active, hc, hp, inertia, force, flag, sim);
        break;
      }
      [[fallthrough]];
    default:
      set_error("exit_test: unsupported chunk count %d", ch);
      return ADEPT_E_UNSUPPORTED;
  }
#undef ADEPT_EXIT_CASE
  return launch_status("exit_test");
}

// The GLOBAL exit test and the active-list update of at most 64 active rows in
// one launch (decode, short prompts), with what an encoder layer does around
// them: the second LayerNorm of the rows before (LN), the early stop of a
// sequence with its [CLS] row and the dead keys after.  One workgroup per row:
// a row's 4 elements per thread and chunk are in flight at once, and the sums
// of the exit test are kept in double as in exit_test_kernel.
//
// The workgroup that finishes last splits the list: the rows' decisions meet
// in ticket[0] (one bit per list entry), their number in ticket[1], both by
// device-scope atomics; a workgroup counts itself once the atomic that set its
// bit has returned, so the one that counts n finds every bit.  Nothing else is
// handed over (the flags are stored by the last workgroup), so no cache has to
// be written back in between.  Both words are zero at the start.
//
// Separate kernels are a launch, a row count and a list read each: at 24 rows
// of 1600 the exit test took 12.7 us in the down projection's epilogue and the
// compaction 4.0; together 4.3.  An encoder layer's five (48 rows of 768):
// LayerNorm 4.0, exit test 4.2, early stop 1.8, compaction 4.2, dead keys 1.4;
// together 7.9.
struct SmallExit {
  const int32_t* rows;
  const int32_t* n_active;
  int max_active;
  bf16* h;                     // layer output, by token row (LN: normalised in place)
  float* inertia;
  const int32_t* force_layer;
  uint8_t* exit_flag;
  double* sim_out;
  int32_t *next, *n_next, *exited, *n_exited, *exit_layer;
  unsigned long long* ticket;
  const bf16 *ln_g, *ln_b;     // LN
  float ln_eps;
  int cls_seq_len;             // > 0: early stop
  uint8_t* key_live;           // nullable
};

constexpr int kSmallThreads = 256;

template <int CH, bool LN>
__global__ __launch_bounds__(kSmallThreads) void exit_compact_kernel(ExitParams p, SmallExit a) {
  __shared__ double ds[4][3];
  const int n = min(*a.n_active, a.max_active);
  const int k = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (k >= n) {
    if (k == 0 && tid == 0) {
      *a.n_next = 0;
      *a.n_exited = 0;
    }
    return;
  }
  const int row = a.rows[k];
  const int nvec = p.d / 4;
  bf16* hr = a.h + (int64_t)row * p.d;
  float* ir = a.inertia + (int64_t)row * p.d;
  float v[CH][4];
  f32x4_t iv[CH];
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const int i = min(c * kSmallThreads + tid, nvec - 1);
    const bf16x4_t x = *reinterpret_cast<const bf16x4_t*>(hr + 4 * i);
    iv[c] = *reinterpret_cast<const f32x4_t*>(ir + 4 * i);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[c][e] = bf2f(x[e]);
  }
  if constexpr (LN) {
    // every wave forms the row's statistics, with the sums of layernorm_row_vec
    // (the LayerNorm of longer lists): the rows come out the same bit for bit
    float w[2 * CH][8];
    const float ls = layernorm_load<2 * CH>(hr, p.d, lane, w);
    const float2 st = layernorm_stats<2 * CH>(w, ls, p.d, a.ln_eps, lane);
    const float mean = st.x, r = st.y;
    __syncthreads();   // the row has been read before it is normalised in place
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int i = min(c * kSmallThreads + tid, nvec - 1);
      const bf16x4_t g = *reinterpret_cast<const bf16x4_t*>(a.ln_g + 4 * i);
      const bf16x4_t b = *reinterpret_cast<const bf16x4_t*>(a.ln_b + 4 * i);
      bf16x4_t o;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        o[e] = f2bf(fmaf((v[c][e] - mean) * r, bf2f(g[e]), bf2f(b[e])));
        v[c][e] = bf2f(o[e]);
      }
      if (c * kSmallThreads + tid < nvec) *reinterpret_cast<bf16x4_t*>(hr + 4 * i) = o;
    }
  }
  double s3[3] = {0.0, 0.0, 0.0};   // <h,h>, <I,I>, <h,I>
#pragma unroll
  for (int c = 0; c < CH; ++c)
    if (c * kSmallThreads + tid < nvec) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const double x = v[c][e], y = iv[c][e];
        s3[0] = fma(x, x, s3[0]);
        s3[1] = fma(y, y, s3[1]);
        s3[2] = fma(x, y, s3[2]);
      }
    }
#pragma unroll
  for (int j = 0; j < 3; ++j) s3[j] = wave_sum_f64(s3[j]);
  if (lane == 0) {
#pragma unroll
    for (int j = 0; j < 3; ++j) ds[wave][j] = s3[j];
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 3; ++j) s3[j] = (ds[0][j] + ds[1][j]) + (ds[2][j] + ds[3][j]);
  const double nh = sqrt(s3[0]), den = nh * sqrt(s3[1]);
  const double sim = den > 0.0 ? s3[2] / den : __longlong_as_double(0x7ff8000000000000ll);
  unsigned long long mask = 0;
  int last = 0;
  if (tid == 0) {
    if (a.sim_out) a.sim_out[k] = sim;
    unsigned long long one = 1ull;
    if (exit_decision(sim >= p.delta, p.layer, p.min_exit_layer, p.n_layers, a.force_layer, row)) {
      const unsigned long long old = __hip_atomic_fetch_or(&a.ticket[0], 1ull << k,
                                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      asm volatile("" : "+v"(one) : "v"(old));   // counted after the bit is set
    }
    last = __hip_atomic_fetch_add(&a.ticket[1], one, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
           (unsigned long long)(n - 1);
    if (last) {
      asm volatile("" ::: "memory");
      mask = __hip_atomic_fetch_or(&a.ticket[0], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  if (nh > 0.0) {
    const double inv = 1.0 / nh;
#pragma unroll
    for (int c = 0; c < CH; ++c)
      if (c * kSmallThreads + tid < nvec) {
        f32x4_t o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (float)((double)iv[c][e] + (double)v[c][e] * inv);
        *reinterpret_cast<f32x4_t*>(ir + 4 * (c * kSmallThreads + tid)) = o;
      }
  }
  if (wave != 0 || !__shfl(last, 0, 64)) return;
  // the last workgroup's first wave: entry `lane` of the list
  mask = __shfl(mask, 0, 64);
  const bool on = lane < n;
  const int mr = on ? a.rows[lane] : -1;
  if (a.cls_seq_len > 0) {
    // a row leaves when its sequence's first row leaves or is no longer listed
    const int cls = on ? mr - mr % a.cls_seq_len : -2;
    bool stop = on;
    for (int j = 0; j < n; ++j)
      if (__shfl(mr, j, 64) == cls) stop = (mask >> j) & 1ull;
    mask |= __ballot(on && stop);
  }
  const bool gone = (mask >> lane) & 1ull;
  const int below = __popcll(mask & ((1ull << lane) - 1ull));
  if (on) {
    a.exit_flag[lane] = gone ? 1 : 0;
    if (gone) {
      a.exited[below] = mr;
      a.exit_layer[mr] = p.layer;
      if (a.key_live) a.key_live[mr] = 0;
    } else {
      a.next[lane - below] = mr;
    }
  }
  if (lane == 0) {
    const int ex = __popcll(mask);
    *a.n_exited = ex;
    *a.n_next = n - ex;
  }
}

// All-at-once variant (Appendix H.2).  Key of an active row: (position + 1)
// in the high word, its list index in the low word; the largest key of a
// sequence names its last prompt token.
__global__ __launch_bounds__(256) void prompt_level_clear(unsigned long long* __restrict__ key,
                                                          int n_seq) {
  const int b = blockIdx.x * 256 + threadIdx.x;
  if (b < n_seq) key[b] = 0ull;
}

__global__ __launch_bounds__(256) void prompt_level_pick(
    const int32_t* __restrict__ rows, const int32_t* __restrict__ n_active, int max_active,
    const int32_t* __restrict__ seq, const int32_t* __restrict__ pos, int n_seq,
    unsigned long long* __restrict__ key) {
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k >= min(*n_active, max_active)) return;
  const int row = rows[k];
  const int b = seq[row];
  if (b < 0 || b >= n_seq) return;
  atomicMax(&key[b], ((unsigned long long)(uint32_t)(pos[row] + 1) << 32) | (uint32_t)k);
}

__global__ __launch_bounds__(256) void prompt_level_apply(
    const int32_t* __restrict__ rows, const int32_t* __restrict__ n_active, int max_active,
    const int32_t* __restrict__ seq, int n_seq, const unsigned long long* __restrict__ key,
    uint8_t* flag) {
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k >= min(*n_active, max_active)) return;
  const int b = seq[rows[k]];
  if (b < 0 || b >= n_seq) return;
  // the deciding row rewrites its own flag with the value it already holds
  flag[k] = flag[(uint32_t)key[b]];
}

}  // namespace
}  // namespace adept

using namespace adept;

extern "C" size_t adept_exit_prompt_level_workspace_bytes(int n_seq) {
  return n_seq > 0 ? (size_t)n_seq * sizeof(unsigned long long) : 0;
}

extern "C" adept_status adept_exit_prompt_level(const int32_t* active_rows,
                                                const int32_t* n_active, int max_active,
                                                const int32_t* seq, const int32_t* pos, int n_seq,
                                                uint8_t* exit_flag, void* workspace,
                                                size_t workspace_bytes, void* stream) {
  ADEPT_REQUIRE(max_active >= 0 && n_seq >= 0, "exit_prompt_level: negative size");
  ADEPT_REQUIRE(active_rows && n_active && seq && pos && exit_flag,
                "exit_prompt_level: NULL tensor");
  if (max_active == 0 || n_seq == 0) return ADEPT_OK;
  const size_t need = adept_exit_prompt_level_workspace_bytes(n_seq);
  if (!workspace || workspace_bytes < need || ((uintptr_t)workspace & 7)) {
    set_error("exit_prompt_level: workspace of %zu bytes (8-byte aligned) needed", need);
    return ADEPT_E_WORKSPACE;
  }
  hipStream_t s = as_stream(stream);
  auto* key = (unsigned long long*)workspace;
  ADEPT_LAUNCH(prompt_level_clear, dim3(ceil_div(n_seq, 256)), dim3(256), 0, s, key, n_seq);
  ADEPT_CHECK_LAUNCH("prompt_level_clear");
  ADEPT_LAUNCH(prompt_level_pick, dim3(ceil_div(max_active, 256)), dim3(256), 0, s, active_rows,
               n_active, max_active, seq, pos, n_seq, key);
  ADEPT_CHECK_LAUNCH("prompt_level_pick");
  ADEPT_LAUNCH(prompt_level_apply, dim3(ceil_div(max_active, 256)), dim3(256), 0, s, active_rows,
               n_active, max_active, seq, n_seq, key, exit_flag);
  return launch_status("prompt_level_apply");
}

extern "C" adept_status adept_exit_test(adept_dtype dt, int d_model, int layer,
                                        const adept_exit_cfg* cfg, const int32_t* active_rows,
                                        const int32_t* n_active, int max_active,
                                        const void* h_cur, const void* h_prev, float* inertia,
                                        const int32_t* force_layer, uint8_t* exit_flag,
                                        double* sim_out, void* stream) {
  ADEPT_REQUIRE(cfg != nullptr, "exit_test: cfg is NULL");
  ADEPT_REQUIRE(dt == ADEPT_F32 || dt == ADEPT_BF16, "exit_test: bad dtype %d", (int)dt);
  ADEPT_REQUIRE(cfg->metric == ADEPT_SIM_GLOBAL || cfg->metric == ADEPT_SIM_LOCAL ||
                    cfg->metric == ADEPT_SIM_BOTH,
                "exit_test: bad metric %d", cfg->metric);
  ADEPT_REQUIRE(cfg->n_layers >= 1 && layer >= 1 && layer <= cfg->n_layers,
                "exit_test: layer %d outside 1..%d", layer, cfg->n_layers);
  ADEPT_REQUIRE(max_active >= 0, "exit_test: max_active < 0");
  ADEPT_REQUIRE(!std::isnan(cfg->delta), "exit_test: delta is NaN");
  ADEPT_REQUIRE(cfg->prompt_level == 0 || cfg->prompt_level == 1,
                "exit_test: prompt_level %d is not 0 or 1", cfg->prompt_level);
  const bool global = cfg->metric != ADEPT_SIM_LOCAL;   // GLOBAL or BOTH: inertia
  const bool both = cfg->metric == ADEPT_SIM_BOTH;
  // elements per lane and chunk (kernel's E)
  const int V = global ? 4 : (dt == ADEPT_BF16 ? 8 : 4);
  ADEPT_REQUIRE(d_model > 0 && d_model % V == 0, "exit_test: d_model %d not a multiple of %d",
                d_model, V);
  ADEPT_REQUIRE(active_rows && n_active && h_cur && exit_flag, "exit_test: NULL tensor");
  ADEPT_REQUIRE(!global || inertia != nullptr, "exit_test: GLOBAL/BOTH need inertia");
  ADEPT_REQUIRE((global && !both) || h_prev != nullptr, "exit_test: LOCAL/BOTH need h_prev");
  ADEPT_REQUIRE(aligned16(h_cur) && (!h_prev || aligned16(h_prev)) &&
                    (!inertia || aligned16(inertia)),
                "exit_test: tensors must be 16-byte aligned");
  if (max_active == 0) return ADEPT_OK;
  const int nvec = d_model / V;
  int ch = (nvec + 63) / 64;
  int chp = 1;
  while (chp < ch) chp <<= 1;
  const int max_ch = both ? kMaxChunksBoth : kMaxChunks;
  if (chp > max_ch) {
    set_error("exit_test: d_model %d too large (max %d)", d_model, max_ch * 64 * V);
    return ADEPT_E_UNSUPPORTED;
  }
  ExitParams p{cfg->delta, cfg->min_exit_layer, cfg->n_layers, layer, d_model};
  hipStream_t s = as_stream(stream);
#define ADEPT_EXIT_MODE(T)                                                                   \
  switch (cfg->metric) {                                                                     \
    case ADEPT_SIM_GLOBAL:                                                                   \
      return launch_exit<T, kGlobal>(chp, p, max_active, active_rows, n_active, h_cur, h_prev, \
                                     inertia, force_layer, exit_flag, sim_out, s);           \
    case ADEPT_SIM_LOCAL:                                                                    \
      return launch_exit<T, kLocal>(chp, p, max_active, active_rows, n_active, h_cur, h_prev,  \
                                    inertia, force_layer, exit_flag, sim_out, s);            \
    default:                                                                                 \
      return launch_exit<T, kBoth>(chp, p, max_active, active_rows, n_active, h_cur, h_prev,   \
                                   inertia, force_layer, exit_flag, sim_out, s);             \
  }
  if (dt == ADEPT_BF16) {
    ADEPT_EXIT_MODE(bf16)
  }
  ADEPT_EXIT_MODE(float)
#undef ADEPT_EXIT_MODE
}

namespace adept {

bool exit_compact_fits(const adept_exit_cfg& cfg, int d, int max_active, bool ln) {
  return cfg.metric == ADEPT_SIM_GLOBAL && max_active > 0 && max_active <= 64 &&
         d <= (ln ? 4 : 8) * 4 * kSmallThreads;
}

adept_status exit_compact(const ExitCompact& x, hipStream_t s) {
  // the argument checks of the exit test and of the compaction, with no rows
  ADEPT_TRY(adept_exit_test(ADEPT_BF16, x.d, x.layer, x.cfg, x.rows, x.n_active, 0, x.h, nullptr,
                            x.inertia, x.force_layer, x.exit_flag, x.sim_out, (void*)s));
  ADEPT_TRY(compact_check(x.layer, x.cfg->n_layers, x.exit_flag, x.rows, x.n_active, x.next,
                          x.n_next, x.exited, x.n_exited, x.exit_layer));
  const ExitParams p{x.cfg->delta, x.cfg->min_exit_layer, x.cfg->n_layers, x.layer, x.d};
  const SmallExit a{x.rows, x.n_active, x.max_active, (bf16*)x.h, x.inertia, x.force_layer,
                    x.exit_flag, x.sim_out, x.next, x.n_next, x.exited, x.n_exited, x.exit_layer,
                    x.ticket, (const bf16*)x.ln_g, (const bf16*)x.ln_b, x.ln_eps, x.cls_seq_len,
                    x.key_live};
  const dim3 grid(x.max_active), block(kSmallThreads);
  const int ch = ceil_div(x.d / 4, kSmallThreads);
#define ADEPT_SMALL_CASE(C)                                                             \
  do {                                                                                  \
    if (x.ln_g)                                                                         \
      ADEPT_LAUNCH((exit_compact_kernel<C, true>), grid, block, 0, s, p, a);            \
    else                                                                                \
      ADEPT_LAUNCH((exit_compact_kernel<C, false>), grid, block, 0, s, p, a);           \
  } while (0)
  if (ch <= 1) ADEPT_SMALL_CASE(1);
  else if (ch <= 2) ADEPT_SMALL_CASE(2);
  else if (ch <= 4) ADEPT_SMALL_CASE(4);
  else ADEPT_LAUNCH((exit_compact_kernel<8, false>), grid, block, 0, s, p, a);   // no LN: _fits
#undef ADEPT_SMALL_CASE
  return launch_status("exit_compact");
}

}  // namespace adept
