// The output tile of the bf16 GEMMs, C[m][n] = sum_k A[m][k] B[n][k] (B in
// nn.Linear [out][in] order, so both operands are K-contiguous), and its
// epilogues.  Three sizes, all by 256 threads: 256x256 (gemm.hip: many rows),
// 128x256 and 128x128 (gemm_mid.h, and the K/V generation of few tiles).
//
// v_mfma_f32_32x32x16_bf16; each of the four waves owns 128 rows x 128
// columns (4x4 MFMA blocks, 256 accumulators per lane held in AGPRs), 64 x 128
// (2x4 blocks) or 32 x 128 (1x4).  K advances 64 at a time.  Operands reach LDS by direct global->LDS loads
// (global_load_lds_dwordx4: lane l of an instruction lands 16 bytes at base
// + 16 l), eight lanes per 128-byte row, so every row of a stage is one whole
// cache line: the load path sustains about 1.5x the bytes per cycle it does
// with half-line requests.  The LDS is a ring of about two and a
// half stages (160 KiB, 256x256; 80 KiB, 128x128) or three (144 KiB); while stage k is
// consumed, stage k+1 and (parts of) stage k+2 are in flight, so the loads
// that miss L2 have one to two stages of MFMA work to land.  Within a row the
// eight 16-byte chunks are permuted, chunk c of row r at position
// c ^ ((r >> 1) & 7): LDS serves a 16-byte read for 16 lanes per cycle
// (64 banks), the 16 rows of such a read fall into the two bank halves by
// r mod 2, and the permutation gives the 8 rows of a half 8 distinct chunk
// positions, so the operand reads are free of bank conflicts.  The operand
// fragments of the next k step are read while the current step's MFMAs run,
// and the loads of later stages are issued between MFMAs; one vmcnt wait and
// one barrier per stage order the ring.
//
// Row gathers (active-row lists) are folded into the per-lane load
// addresses.  The epilogue stages the accumulators through LDS, 32 rows of a
// wave at a time, so that its global loads and stores cover whole rows; a
// per-row scale (1/rms of the row, with the norm gain folded into B
// beforehand) is applied first, then RoPE + cache store (the wave's 128
// columns cover whole heads of 64 or 128, so a column's rotary partner is in
// the same staged row), residual add, SwiGLU (B tile = 64 gate rows + 64 up
// rows per wave), or plain store.
#pragma once

#include <algorithm>
#include <type_traits>

#include "common.h"

namespace adept {

constexpr int BK = 64;                                          // k columns per stage: 128-byte rows
constexpr int kEpiStride = 136;                                 // floats per staged epilogue row
constexpr int kEpiWaveBytes = 32 * kEpiStride * 4;              // one wave's 32 staged rows
constexpr int kEpiMetaBytes = 128 * 3 * 4;                      // per-row scale, row/slot, position

// Geometry of a TM x TN output tile: waves of 32 MB rows x 128 columns, the
// LDS ring and the issue plan of the K loop.  The 256 x 256 tile's ring has
// five one-operand slots (A of stage k in slot 2k mod 5, B in 2k+1 mod 5: all
// of a CU's LDS); the smaller tiles keep whole stages, kPeriod of them.
//
// Plan: 2-bit counts over the 4 MB MFMAs of a k step (field n: how many
// follow MFMA n): kRead, the fragment reads of the next k step (MB of A, 4 of
// B); kDma[ks], the direct loads of the stage two ahead (A's first, then
// B's), over the four k steps.  A wave stalls when the load path's queue is
// full and the waves issue in step, so the loads are spread out.
template <int TM_, int TN_, int MB_> struct GeoBase {
  static constexpr int kTM = TM_, kTN = TN_, kMB = MB_;
  static constexpr int kWM = TM_ / (32 * MB_), kWN = TN_ / 128;  // waves down, across
  static constexpr int kWaves = kWM * kWN, kThreads = 64 * kWaves;
  static constexpr int kABytes = TM_ * BK * 2, kBBytes = TN_ * BK * 2;   // one stage
  static constexpr int kLoadsA = TM_ / 8 / kWaves, kLoadsB = TN_ / 8 / kWaves;  // per wave and stage
};
template <int TM, int TN> struct Geo;
template <> struct Geo<256, 256> : GeoBase<256, 256, 4> {
  static constexpr int kPeriod = 5, kLds = 5 * 32768;
  // LDS offset of operand o (0 = A, 1 = B) of a stage of phase P = stage mod kPeriod
  __host__ __device__ static constexpr int base(int o, int P) { return ((2 * P + o) % 5) * 32768; }
  static constexpr uint32_t kRead = 0x00005555;
  // B's slot is freed by the barrier before the last k step
  static constexpr uint32_t kDma[4] = {0x40400000, 0x40404040, 0x40400000, 0x55550000};
};
template <> struct Geo<128, 256> : GeoBase<128, 256, 2> {
  static constexpr int kPeriod = 3, kLds = 3 * (kABytes + kBBytes);
  __host__ __device__ static constexpr int base(int o, int P) {
    return (P % 3) * (kABytes + kBBytes) + o * kABytes;
  }
  static constexpr uint32_t kRead = 0x0555;
  static constexpr uint32_t kDma[4] = {0x4440, 0x4440, 0x4440, 0x4440};
};
template <> struct Geo<128, 128> : GeoBase<128, 128, 1> {
  static constexpr int kPeriod = 5, kLds = 5 * 16384;
  __host__ __device__ static constexpr int base(int o, int P) { return ((2 * P + o) % 5) * 16384; }
  static constexpr uint32_t kRead = 0x56;
  static constexpr uint32_t kDma[4] = {0x40, 0x44, 0x40, 0x55};
};
// the first n fields' sum
constexpr int plan_sum(uint32_t f, int n) {
  int s = 0;
  for (int i = 0; i < n; ++i) s += (f >> (2 * i)) & 3;
  return s;
}
// loads issued before k step ks
template <class GT> constexpr int plan_before(int ks) {
  int s = 0;
  for (int i = 0; i < ks; ++i) s += plan_sum(GT::kDma[i], 16);
  return s;
}
template <class GT> constexpr bool geo_ok() {
  return plan_before<GT>(4) == GT::kLoadsA + GT::kLoadsB && plan_sum(GT::kRead, 16) == GT::kMB + 4 &&
         GT::kWaves * (kEpiWaveBytes + kEpiMetaBytes) <= GT::kLds && GT::kLds <= 160 * 1024;
}
static_assert(geo_ok<Geo<256, 256>>() && geo_ok<Geo<128, 256>>() && geo_ok<Geo<128, 128>>(),
              "every load and fragment read is issued; the epilogue staging fits in the ring");

typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(3))) char lds_char_t;
typedef __attribute__((address_space(3))) const bf16x8_t lds_bf16x8_t;
typedef __attribute__((address_space(1))) void glb_void_t;

struct GP {
  int M_max;
  const int32_t* M_dev;
  int N, K;
  const bf16* A;
  const int32_t* a_rows;
  int64_t lda;
  const bf16* B;
  const bf16* B2;
  int64_t ldb;
  void* C;
  int64_t ldc;
  int c_f32;
  const float* row_scale;   // [compact m] or nullptr
  const int32_t* rows;
  const bf16* resid;
  const bf16* bias;         // [N] or nullptr
  const int32_t* pos;
  const int32_t* slot;
  const float* rope_cos;
  const float* rope_sin;
  int head_dim, d_q;
  bf16* q_out;
  bf16* k_cache;
  bf16* v_cache;
  int tiles_m, tiles_n;
  // grouped (KV generation)
  const int32_t* work;      // packed (layer << 16) | m_tile
  const int32_t* n_work;
  const int32_t* grp_m;     // [N+2]: rows with exit layer < r
  const int32_t* srows;     // exited rows sorted by exit layer
  int64_t b_layer_stride;
  int64_t cache_layer_stride;
  int64_t bias_layer_stride; // grouped: layer r's bias at bias + (r-1) * stride
  int a_sorted;             // grouped: A holds the rows in sorted order (row m), not by token
  // per-row second A buffer: token row r reads A2 when a_sel[r] & 1 (nullable)
  const bf16* A2;
  const int32_t* a_sel;
  float* rinv_out;          // skinny RESID: 1/rms of each result row (nullable)
  bf16* ln_out;             // skinny RESID: LayerNorm of each result row (nullable)
  float row_eps;
  RowExit ex;               // skinny RESID: the exit test of each result row (has_exit)
  int has_exit;
};

// x * sigmoid(x) with the hardware reciprocal (about 1 ulp in f32, far below
// the bf16 rounding of the output)
__device__ __forceinline__ float silu(float g) {
  return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g));
}

// x * Phi(x) rounded to bf16, where Phi is formed by 1 + erff: the same bits for
// every x, mostly without erff.  The normal CDF from Phi(-a) = t P(t) exp(-a^2/2),
// a = |x|, t = 1/(1 + 0.21213203f a), where P fits exp(a^2/2) Phi(-a) / t over
// a = 0..13.5 to 4.5e-8 relative (least squares weighted towards the largest
// error), is within kGeluErr a of the form with erff, so where both ends of that
// interval round to the same bf16 that is the result; erff decides the others
// (6e-4 of the values in (-1, 0), 3e-3 in (-2, -1), 4e-2 in (-3, -2)).  A 32768 x
// 3072 x 768 GELU projection takes 196 us; 185 with the polynomial alone, whose f32
// results are off by up to 7e-6 (near -12.6) and whose bf16 ones differ now and then.
constexpr float kGeluErr = 4.5e-7f;   // the largest over all floats: 2.98e-7
__device__ __forceinline__ uint32_t gelu_ends(float x) {   // low and high end, rounded
  const float a = fabsf(x);
  const float t = __builtin_amdgcn_rcpf(fmaf(0.2121320366859436f, a, 1.0f));
  float q = -0.06472896039485931f;
  q = fmaf(q, t, 0.242610901594162f);
  q = fmaf(q, t, -0.2557545602321625f);
  q = fmaf(q, t, 0.2733757495880127f);
  q = fmaf(q, t, -0.04695289954543114f);
  q = fmaf(q, t, 0.10728416591882706f);
  q = fmaf(q, t, 0.07422187924385071f);
  q = fmaf(q, t, 0.08534912019968033f);
  q = fmaf(q, t, 0.08459459245204926f);
  const float h = t * q * __expf(-0.5f * a * a);   // Phi(-a)
  const float y = x * (x < 0.0f ? h : 1.0f - h), e = kGeluErr * a;
  return pack_bf16x2(y - e, y + e);
}
// N values in place; the few that need erff are one branch for all of them
template <int N> __device__ __forceinline__ void gelu_erf(float (&x)[N]) {
  uint32_t w[N], open = 0;
#pragma unroll
  for (int n = 0; n < N; ++n) {
    w[n] = gelu_ends(x[n]);
    open |= (w[n] ^ (w[n] << 16)) >> 16;   // the ends differ (or NaN and not)
  }
  if (open) {
#pragma unroll
    for (int n = 0; n < N; ++n)
      if ((w[n] ^ (w[n] << 16)) >> 16)
        w[n] = f2bf(0.5f * x[n] * (1.0f + erff(x[n] * 0.7071067811865476f)));
  }
#pragma unroll
  for (int n = 0; n < N; ++n) x[n] = __uint_as_float(w[n] << 16);
}

// x * Phi(x) with the tanh approximation of the normal CDF (GPT-2's MLP):
// (1 + tanh u) / 2 = 1 / (1 + exp(-2u)), u = sqrt(2/pi) (x + 0.044715 x^3)
__device__ __forceinline__ float gelu_tanh(float x) {
  const float u2 = 1.5957691216057308f * fmaf(0.044715f * x, x * x, x);
  return x * __builtin_amdgcn_rcpf(1.0f + __expf(-u2));
}

// Four bias values of columns c..c+3 (zeros when there is no bias).
__device__ __forceinline__ float4 bias4(const bf16* b, int64_t c) {
  if (!b) return make_float4(0.f, 0.f, 0.f, 0.f);
  const bf16x4_t v = *reinterpret_cast<const bf16x4_t*>(b + c);
  return make_float4(bf2f(v[0]), bf2f(v[1]), bf2f(v[2]), bf2f(v[3]));
}

// Four values of a rotary table, which callers need not align past its floats
// (passes above 64 rows read single ones): the unaligned load is one instruction.
__device__ __forceinline__ float4 rope4(const float* t) {
  typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
  const f32x4_any v = *reinterpret_cast<const f32x4_any*>(t);
  return make_float4(v[0], v[1], v[2], v[3]);
}

__device__ __forceinline__ void dma16(const bf16* g, char* l) {
  __builtin_amdgcn_global_load_lds((glb_void_t*)g, (lds_void_t*)l, 16, 0, 0);
}

// s_waitcnt immediate (gfx9 encoding) that waits for all LDS operations and
// leaves the vector-memory and export counters free: vmcnt 63, expcnt 7,
// lgkmcnt 0.
constexpr int kWaitLgkm0 = 0xC07F;

// s_waitcnt for at most N outstanding vector-memory operations (6-bit
// vmcnt: low bits 3:0, high bits 15:14), leaving the export and LDS
// counters free.
template <int N> __device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt field");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

__device__ __forceinline__ void wait_dma() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Workgroup barrier of the K loop.  __syncthreads() would also wait for every
// outstanding vector-memory operation, i.e. drain the direct-to-LDS loads of
// the later stages and leave no load in flight across the barrier; here the
// caller waits for exactly the stage it needs (vmcnt) and the memory clobber
// keeps the compiler from moving LDS accesses across the barrier.  The
// operand reads of the previous stage have completed by then: the MFMAs that
// consume them were issued before it.
__device__ __forceinline__ void stage_barrier() { asm volatile("s_barrier" ::: "memory"); }

// One output tile of geometry GT: rows [mt*TM, M) against column tile nt of Bm,
// over the k stages [k0, k0 + KT).  part != NULL (a tile split over K): the
// f32 sums go to part [TM][TN] instead of the epilogue.
// HD (64 or 128) is the head size of the rotary epilogues (0 otherwise).
// EXT: the shapes and inputs beyond the plain case -- a ragged last column
// tile (N not a multiple of TN), cache sections that do not align with the
// 128-column waves (H*hd not a multiple of 128), a per-row second A buffer;
// the plain instantiation carries none of their per-lane tests (registers).
template <int EPI, bool GROUPED, int HD, bool EXT, class GT, bool SPLIT>
__device__ __forceinline__ void gemm_tile(const GP& p, char* smem, int layer, int mt, int nt,
                                          int M, const bf16* Bm, int k0, int KT, float* part) {
  constexpr int BM = GT::kTM, BN = GT::kTN, MB = GT::kMB;
  constexpr int kWaveRows = 32 * MB, NA = GT::kLoadsA, NB = GT::kLoadsB;
  // the wave index in a scalar register: LDS destinations of the direct
  // loads (M0) then need no read-back from a vector register
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / GT::kWN, wn = wave % GT::kWN;
  const int m0 = mt * BM;

  // ---- load assignment: DMA instruction j of wave w fills the 1 KiB of
  // stage rows 8q .. 8q+7 of A (q = w*NA + j) or of B (q = w*NB + j); lane l
  // -> row 8q + l/8, stored position l%8, logical chunk (l%8) ^ ((row >> 1) & 7)
  // = (l%8) ^ ((4q + (l >> 4)) & 7).  A row's 128 bytes are one cache line.
  const int lrow = lane >> 3;
  const bf16* a_src[NA];
  const bf16* b_src[NB];
#pragma unroll
  for (int j = 0; j < NA; ++j) {
    const int q = wave * NA + j;
    const int lchunk = (lane & 7) ^ ((4 * q + (lane >> 4)) & 7);
    int m = m0 + 8 * q + lrow;
    if (m >= M) m = m0;  // clamp: loaded, never stored
    const int arow = GROUPED ? (p.a_sorted ? m : p.srows[m]) : (p.a_rows ? p.a_rows[m] : m);
    const bf16* abase = (EXT && !GROUPED && p.a_sel && (p.a_sel[arow] & 1)) ? p.A2 : p.A;
    a_src[j] = abase + (int64_t)arow * p.lda + lchunk * 8 + k0 * BK;
  }
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int q = wave * NB + j;
    const int r = 8 * q + lrow;
    const int lchunk = (lane & 7) ^ ((4 * q + (lane >> 4)) & 7);
    const bf16* bbase = Bm;
    int64_t brow;
    if (EPI == EPI_SWIGLU) {
      const int half = r >> 7, within = r & 127;
      bbase = within < 64 ? p.B : p.B2;
      brow = (int64_t)nt * (BN / 2) + half * 64 + (within & 63);
    } else {
      // a ragged last column tile re-reads the last row: computed, never stored
      brow = EXT ? min((int64_t)nt * BN + r, (int64_t)p.N - 1) : (int64_t)nt * BN + r;
    }
    b_src[j] = bbase + brow * p.ldb + lchunk * 8 + k0 * BK;
  }
  // Per-row inputs of the epilogue (row scale, residual row or cache slot,
  // rotary position) for the wave's rows, one per lane and 64 rows: loaded here so
  // that their latency (two dependent loads for a cache slot) passes during
  // the K loop.
  constexpr int NPRE = (kWaveRows + 63) / 64;
  float pre_sc[NPRE];
  int pre_row[NPRE], pre_pos[NPRE];
  {
    constexpr bool kC = EPI == EPI_QKV || EPI == EPI_KV;
    const int secp = kC ? (nt * BN + wn * 128) / p.d_q : 0;
    const bool q_sec = EPI == EPI_QKV && secp == 0;
    const bool v_sec = EPI == EPI_QKV ? secp == 2 : (EPI == EPI_KV && secp == 1);
#pragma unroll
    for (int h = 0; h < NPRE; ++h) {
      const int mc = min(m0 + wm * kWaveRows + lane + 64 * h, M - 1);   // clamped: never stored
      pre_sc[h] = p.row_scale ? p.row_scale[mc] : 1.0f;
      pre_row[h] = 0;
      pre_pos[h] = 0;
      if (EPI == EPI_RESID) {
        pre_row[h] = p.rows[mc];
      } else if (kC) {
        const int row = GROUPED ? p.srows[mc] : p.rows[mc];
        pre_row[h] = (q_sec && p.d_q % 128 == 0) ? 0 : (p.slot ? p.slot[row] : row);
        pre_pos[h] = (v_sec || !p.rope_cos) ? 0 : p.pos[row];
      }
    }
  }
  // Direct load u of stage k (in ring phase P, any int): A's NA, then B's NB.
  auto issue = [&](int k, int P, int u) {
    P %= GT::kPeriod;
    if (u < NA)
      dma16(a_src[u < NA ? u : 0] + k * BK, smem + GT::base(0, P) + (wave * NA + u) * 1024);
    else
      dma16(b_src[u < NA ? 0 : u - NA] + k * BK,
            smem + GT::base(1, P) + (wave * NB + u - NA) * 1024);
  };

  f32x16_t acc[MB][4];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

  // MFMA operand addresses: block i row R = (wave's first row) + i*32 + lane%32; logical
  // chunk 2*ks + lane/32 (k step ks = 0..3) stored at chunk ^ ((R >> 1) & 7),
  // and the block offsets are multiples of 32, so the position is
  // chunk ^ ((lane >> 1) & 7).
  const int rA = wm * kWaveRows + (lane & 31);
  const int rB = wn * 128 + (lane & 31);
  const int swz = (lane >> 1) & 7;
  // Fragment reads of a phase known at compile time: win[o][w][ks] + a
  // constant, with window w (64 KiB of the ring) plus the lane's offset of k
  // step ks in block 0 of operand o (0 = A, 1 = B); the operand's place in the
  // window and the block (i * 4 KiB) fit the 16-bit offset of ds_read, so a
  // read takes no address arithmetic.
  constexpr int kWin = (GT::kLds + 65535) / 65536;
  lds_char_t* win[2][kWin][4];
#pragma unroll
  for (int o = 0; o < 2; ++o)
#pragma unroll
    for (int w = 0; w < kWin; ++w)
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
        win[o][w][ks] = (lds_char_t*)smem + w * 65536 +
                        ((o ? rB : rA) * 8 + ((2 * ks + (lane >> 5)) ^ swz)) * 16;
  // Re-defines the bases (no instruction): otherwise the compiler hoists
  // the addresses derived for every phase, operand and k step out of the
  // loop, into registers of their own.
  auto refresh = [&]() {
#pragma unroll
    for (int o = 0; o < 2; ++o)
#pragma unroll
      for (int w = 0; w < kWin; ++w)
        asm volatile("" : "+v"(win[o][w][0]), "+v"(win[o][w][1]), "+v"(win[o][w][2]),
                     "+v"(win[o][w][3]));
  };
  // Fragment n of k step ks of phase P: A and B blocks in turn as far as A's
  // go, then the other B blocks.  Compile-time phase (fixed) or any phase
  // (run-time address arithmetic).
  auto is_b = [](int n) { return n < 2 * MB ? (n & 1) != 0 : true; };
  auto blk = [](int n) { return n < 2 * MB ? n >> 1 : n - MB; };
  auto frag_fixed = [&](int P, int ks, int n, bf16x8_t (&a)[MB], bf16x8_t (&b)[4]) {
    const int i = blk(n), o = is_b(n) ? 1 : 0;
    const int at = GT::base(o, P % GT::kPeriod);
    const bf16x8_t f = *reinterpret_cast<const lds_bf16x8_t*>(win[o][at / 65536][ks] +
                                                              at % 65536 + i * 4096);
    if (o) b[i] = f;
    else a[i < MB ? i : 0] = f;
  };
  auto frag_any = [&](int P, int ks, int n, bf16x8_t (&a)[MB], bf16x8_t (&b)[4]) {
    const int ch = (2 * ks + (lane >> 5)) ^ swz;
    const int i = blk(n), o = is_b(n) ? 1 : 0;
    const bf16x8_t f = *reinterpret_cast<const lds_bf16x8_t*>(
        (lds_char_t*)smem + GT::base(o, P % GT::kPeriod) +
        (((o ? rB : rA) + i * 32) * 8 + ch) * 16);
    if (o) b[i] = f;
    else a[i < MB ? i : 0] = f;
  };
  // One k step: 4 MB MFMAs on (a, b), with read(u) and dma(d0 + u) issued
  // between them as the plan's fields say, so that every non-MFMA instruction
  // issues while the matrix core has work queued.  The plan is a compile-time
  // constant: a branch between MFMAs costs an instruction-fetch bubble.
  auto kstep = [&](const bf16x8_t (&a)[MB], const bf16x8_t (&b)[4], auto&& read, auto&& dma,
                   auto rmask, auto dmask, int d0) {
    constexpr uint32_t RM = decltype(rmask)::value, DM = decltype(dmask)::value;
#pragma unroll
    for (int n = 0; n < 4 * MB; ++n) {
      const int i = n >> 2, j = n & 3;
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
#pragma unroll
      for (int u = plan_sum(RM, n); u < plan_sum(RM, n + 1); ++u) read(u);
#pragma unroll
      for (int u = plan_sum(DM, n); u < plan_sum(DM, n + 1); ++u) dma(d0 + u);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  using Reads = std::integral_constant<uint32_t, GT::kRead>;
  using D0 = std::integral_constant<uint32_t, GT::kDma[0]>;
  using D1 = std::integral_constant<uint32_t, GT::kDma[1]>;
  using D2 = std::integral_constant<uint32_t, GT::kDma[2]>;
  using D3 = std::integral_constant<uint32_t, GT::kDma[3]>;
  constexpr int kD1 = plan_before<GT>(1), kD2 = plan_before<GT>(2), kD3 = plan_before<GT>(3);

  // K loop over the ring.  At the top of iteration kt stage kt has landed and
  // is visible to every wave, stage kt+1 is in flight, and the fragments of
  // stage kt's first k step were read just before.  Stage kt+2 is loaded
  // during the iteration into room that a barrier has freed: five one-operand
  // slots, A_kt+2 into the slot of B_kt-1 during k steps 0..2, and B_kt+2
  // into the slot of A_kt right after this iteration's barrier; three whole
  // stages, stage kt+2 into the place of stage kt-1.  So each stage has one to
  // two iterations of MFMA work to land.  Before each k step, the reads issued
  // during the previous one are waited for; at most 8 LDS reads are ever
  // outstanding (the 4-bit lgkm counter cannot express more).  The wait for
  // stage kt+1 (only the loads of stage kt+2 issued so far may stay
  // outstanding) and the barrier, which publishes stage kt+1 and retires every
  // read of stage kt, come before the last k step, whose MFMAs then cover the
  // reads of stage kt+1's first fragments.
  //
  // Every iteration issues the same loads: past the last stage the stage
  // index is clamped, so the last two iterations refill free room with
  // data that is never read (two stages of extra L2 traffic per tile) and
  // the body has no conditional code.  The loop runs in groups of the ring's
  // period, in which every phase is a compile-time constant; the leading
  // iterations before them take the same body with run-time phases.
  const int kLast = KT - 1;
  // stage k's phase is shifted by sh so that the groups start at phase 0
  constexpr int PD = GT::kPeriod;
  const int sh = (PD - KT % PD) % PD;
#pragma unroll
  for (int u = 0; u < NA + NB; ++u) issue(0, sh, u);
#pragma unroll
  for (int u = 0; u < NA + NB; ++u) issue(min(1, kLast), sh + 1, u);
  wait_vm<NA + NB>();
  stage_barrier();
  bf16x8_t fa[MB], fb[4], ga[MB], gb[4];
#pragma unroll
  for (int n = 0; n < MB + 4; ++n) frag_any(sh, 0, n, fa, fb);
  // iteration kt, with P = (kt + sh) mod PD (a compile-time constant when FIXED)
  auto iteration = [&](int kt, int P, auto fixed) {
    constexpr bool kFixed = decltype(fixed)::value;
    auto frag = [&](int ph, int ks, int n, bf16x8_t (&a)[MB], bf16x8_t (&b)[4]) {
      if constexpr (kFixed) frag_fixed(ph, ks, n, a, b);
      else frag_any(ph, ks, n, a, b);
    };
    const int kd = min(kt + 2, kLast);
    auto dma = [&](int u) { issue(kd, P + 2, u); };
    if constexpr (kFixed) refresh();
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
    __builtin_amdgcn_sched_barrier(0);
    kstep(fa, fb, [&](int n) { frag(P, 1, n, ga, gb); }, dma, Reads{}, D0{}, 0);
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
    __builtin_amdgcn_sched_barrier(0);
    kstep(ga, gb, [&](int n) { frag(P, 2, n, fa, fb); }, dma, Reads{}, D1{}, kD1);
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
    __builtin_amdgcn_sched_barrier(0);
    kstep(fa, fb, [&](int n) { frag(P, 3, n, ga, gb); }, dma, Reads{}, D2{}, kD2);
    // every read of stage kt has completed: wait for stage kt+1 (the loads of
    // stage kt+2 so far may stay outstanding), publish it, retire stage kt
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
    __builtin_amdgcn_sched_barrier(0);
    wait_vm<kD3>();
    stage_barrier();
    // after the last stage this reads stale but valid LDS
    kstep(ga, gb, [&](int n) { frag(P + 1, 0, n, fa, fb); }, dma, Reads{}, D3{}, kD3);
  };
  using Fixed = std::true_type;
  using Any = std::false_type;
  const int r = KT % PD;
  int kt = 0;
  for (; kt < r; ++kt) iteration(kt, (kt + sh) % PD, Any{});
  for (; kt < KT; kt += PD) {
    iteration(kt, 0, Fixed{});
    iteration(kt + 1, 1, Fixed{});
    iteration(kt + 2, 2, Fixed{});
    if constexpr (PD == 5) {
      iteration(kt + 3, 3, Fixed{});
      iteration(kt + 4, 4, Fixed{});
    }
  }
  wait_dma();   // the clamped loads of the last iterations land before LDS is reused
  __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
  stage_barrier();   // every wave is done with the ring; LDS is reused below
  if (SPLIT && part) {
    // value v of a block is row 8*(v/4) + 4*(lane/32) + v%4, column lane%32
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int r = wm * kWaveRows + i * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
        if (m0 + r < M) {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            part[r * BN + wn * 128 + j * 32 + (lane & 31)] = acc[i][j][v];
        }
      }
    return;
  }

  // ---- epilogue, staged through LDS 32 rows at a time.  Lane holds column
  // (lane & 31) of each 32x32 block and rows 8*(v/4) + 4*(lane/32) + v%4,
  // v = 0..15.  Block i of the wave (32 rows x its 128 columns, f32) is
  // written to the wave's LDS area with a row stride of kEpiStride floats
  // (the two row groups of a write then fall on disjoint banks), then read
  // back as 4 consecutive columns per lane, so every global load and store
  // of the epilogue covers whole rows: 32 lanes x 8 bytes = one 256-byte row
  // of 128 bf16 columns.  The per-row inputs (scale, residual row or cache
  // slot and position) of the wave's 128 rows are gathered into LDS first,
  // two memory latencies per tile instead of one per store round.
  float* stg = reinterpret_cast<float*>(smem + wave * kEpiWaveBytes);
  float* msc = reinterpret_cast<float*>(smem + GT::kWaves * kEpiWaveBytes + wave * kEpiMetaBytes);
  int* mrow = reinterpret_cast<int*>(msc + 128);   // residual row / cache slot
  int* mpos = mrow + 128;                          // rotary position
  const int col_l = lane & 31;
  const int row_q = 4 * (lane >> 5);
  const int c4 = (lane & 31) * 4;         // first of the lane's 4 columns (wave space)
  const int nw = nt * BN + wn * 128;      // first output column of this wave
  // grouped: layer r's bias; a ragged column tile's waves past N store
  // nothing (SwiGLU tiles are never ragged: 128 outputs of N per tile)
  const bf16* bias = GROUPED && EXT && p.bias ? p.bias + (int64_t)(layer - 1) * p.bias_layer_stride
                                       : p.bias;
  const bool wave_out = EXT && EPI != EPI_SWIGLU && nw >= p.N;
  constexpr bool kCache = EPI == EPI_QKV || EPI == EPI_KV;
  const int sec = kCache ? nw / p.d_q : 0;    // QKV: 0 q, 1 k, 2 v;  KV: 0 k, 1 v
  const bool is_q = EPI == EPI_QKV && sec == 0;
  const bool is_v = EPI == EPI_QKV ? sec == 2 : (EPI == EPI_KV && sec == 1);
  const int cbase = nw - sec * p.d_q;         // column within the section
  constexpr int hd = HD > 0 ? HD : 128, half = hd >> 1;
  // destination of the QKV / KV epilogues: Q rows by compact index, K and V
  // rows by cache slot (in layer r's cache for the grouped variant)
  bf16* sec_dst = nullptr;
  if (kCache) {
    if (is_q) {
      sec_dst = p.q_out;
    } else {
      sec_dst = is_v ? p.v_cache : p.k_cache;
      if (GROUPED) sec_dst += (int64_t)(layer - 1) * p.cache_layer_stride;
    }
    sec_dst += cbase;
  }
#pragma unroll
  for (int h = 0; h < NPRE; ++h) {
    const int lr = lane + 64 * h;
    msc[lr] = pre_sc[h];
    if (EPI == EPI_RESID || kCache) mrow[lr] = pre_row[h];
    if (kCache) mpos[lr] = pre_pos[h];
  }
  // one 32-row block; the block index is a compile-time constant (an
  // accumulator indexed at run time would move the whole tile to scratch)
  auto block = [&](auto ic) {
    constexpr int i = decltype(ic)::value;
    const int mb = m0 + wm * kWaveRows + i * 32;   // first row of the block
    if (mb >= M || wave_out) return;          // rows past M / columns past N
    if constexpr (EPI == EPI_SWIGLU) {
      // Gate (blocks j = 0, 1) and up (j = 2, 3) of an output column sit in
      // the same lane, so h = silu(g) * u is formed in registers; lanes 2k
      // and 2k+1 hold adjacent columns and swap one value (DPP), so the even
      // lane holds row v and the odd lane row v+1 of a pair of columns as
      // one 4-byte bf16 pair.  The pairs go to LDS (32 rows x 128 bytes; two
      // rows fill the 64 banks) and come back as 16-byte row segments: four
      // full-row stores per block instead of 32 narrow ones.
      float sc[16];
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const float4 t = *reinterpret_cast<const float4*>(msc + i * 32 + 8 * g4 + row_q);
        sc[4 * g4 + 0] = t.x; sc[4 * g4 + 1] = t.y; sc[4 * g4 + 2] = t.z; sc[4 * g4 + 3] = t.w;
      }
      const bool odd = lane & 1;
      char* sb = reinterpret_cast<char*>(stg);
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          const int v0 = 2 * t, v1 = 2 * t + 1;
          const float h0 = silu(acc[i][j][v0] * sc[v0]) * (acc[i][j + 2][v0] * sc[v0]);
          const float h1 = silu(acc[i][j][v1] * sc[v1]) * (acc[i][j + 2][v1] * sc[v1]);
          // quad_perm [1,0,3,2]: exchange with the neighbouring lane
          const float y = __int_as_float(__builtin_amdgcn_mov_dpp(
              __float_as_int(odd ? h0 : h1), 0xB1, 0xF, 0xF, false));
          const uint32_t w = odd ? pack_bf16x2(y, h1) : pack_bf16x2(h0, y);
          const int lr = 8 * (v0 >> 2) + row_q + (v0 & 3) + (odd ? 1 : 0);
          *reinterpret_cast<uint32_t*>(sb + lr * 128 + j * 64 + (col_l & ~1) * 2) = w;
        }
      __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
      __builtin_amdgcn_wave_barrier();
      const bool full = mb + 32 <= M;
      bf16* cb = reinterpret_cast<bf16*>(p.C) + nw / 2 + (lane & 7) * 8;
      uint4 seg[4];
#pragma unroll
      for (int q = 0; q < 4; ++q)
        seg[q] = *reinterpret_cast<const uint4*>(sb + (8 * q + (lane >> 3)) * 128 + (lane & 7) * 16);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int m = mb + 8 * q + (lane >> 3);
        if (full || m < M) *reinterpret_cast<uint4*>(cb + (int64_t)m * p.ldc) = seg[q];
      }
      __builtin_amdgcn_s_waitcnt(kWaitLgkm0);   // reads done before the next block's writes
      __builtin_amdgcn_wave_barrier();
      return;
    }
    if constexpr (kCache) {
      if (!p.bias) {   // wave-uniform: the decoder's QKV and the KV generation
        // The wave's 128 columns are whole heads, so the rotary partner of a
        // column (c ^ hd/2) sits in the same lane, hd/64 blocks away: RoPE
        // runs on the accumulators.  Positions come from the gathered
        // per-row inputs and the cos/sin values of the block's 16 rows per
        // lane are loaded at once (one memory latency per block).  Results
        // leave as in the SwiGLU path: bf16 pairs (DPP lane swap) to LDS,
        // 32 rows x 256 bytes, each row's four 64-byte segments permuted by
        // (row & 1) | ((row >> 2) & 1) << 1 so the four row groups of a
        // write fall on distinct banks, read back as 16-byte row segments
        // and stored as whole 256-byte rows of the destination.
        constexpr int kPair = hd / 64;          // block distance of rotary partners
        constexpr int kTab = hd == 128 ? 2 : 1; // table columns per lane and row
        const bool rope = !is_v && p.rope_cos;  // wave-uniform
        float sc[16];
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
          const float4 t = *reinterpret_cast<const float4*>(msc + i * 32 + 8 * g4 + row_q);
          sc[4 * g4 + 0] = t.x; sc[4 * g4 + 1] = t.y; sc[4 * g4 + 2] = t.z; sc[4 * g4 + 3] = t.w;
        }
        float cv[16][kTab], sv[16][kTab];
        if (rope) {
          int ps[16];
#pragma unroll
          for (int g4 = 0; g4 < 4; ++g4) {
            const int4 t = *reinterpret_cast<const int4*>(mpos + i * 32 + 8 * g4 + row_q);
            ps[4 * g4 + 0] = t.x; ps[4 * g4 + 1] = t.y; ps[4 * g4 + 2] = t.z; ps[4 * g4 + 3] = t.w;
          }
#pragma unroll
          for (int v = 0; v < 16; ++v)
#pragma unroll
            for (int u = 0; u < kTab; ++u) {
              const int64_t t = (int64_t)ps[v] * half + u * 32 + col_l;
              cv[v][u] = p.rope_cos[t];
              sv[v][u] = p.rope_sin[t];
            }
        }
        // output of column block j, row v of the lane
        auto out = [&](int j, int v) {
          const float x = acc[i][j][v] * sc[v];
          if (!rope) return x;
          const float y = acc[i][j ^ kPair][v] * sc[v];
          const int u = hd == 128 ? (j & 1) : 0;
          const bool first = hd == 128 ? j < 2 : (j & 1) == 0;   // column < hd/2
          return first ? x * cv[v][u] - y * sv[v][u] : x * cv[v][u] + y * sv[v][u];
        };
        // Lanes 2k, 2k+1 hold adjacent columns.  Each packs its rows v0, v1
        // as one bf16 pair, the pairs are swapped (DPP quad_perm [1,0,3,2])
        // and one byte permute forms row v0 (even lane) or row v1 (odd
        // lane) of the two columns.
        const bool odd = lane & 1;
        const uint32_t psel = odd ? 0x03020706u : 0x05040100u;
        char* sb = reinterpret_cast<char*>(stg);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int t = 0; t < 8; ++t) {
            const int v0 = 2 * t, v1 = 2 * t + 1;
            const uint32_t own = pack_bf16x2(out(j, v0), out(j, v1));
            const uint32_t nbr = (uint32_t)__builtin_amdgcn_mov_dpp((int)own, 0xB1, 0xF, 0xF, false);
            const uint32_t w = __builtin_amdgcn_perm(nbr, own, psel);
            const int lr = 8 * (v0 >> 2) + row_q + (v0 & 3) + (odd ? 1 : 0);
            const int g = (lr & 1) | (((lr >> 2) & 1) << 1);
            *reinterpret_cast<uint32_t*>(sb + lr * 256 + ((j ^ g) << 6) + (col_l & ~1) * 2) = w;
          }
        __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
        __builtin_amdgcn_wave_barrier();
        const bool full = mb + 32 <= M;
        const int sg = lane & 15;
        typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
        u32x4_t seg[8];
        int drow[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const int R = 4 * q + (lane >> 4);
          const int g = (R & 1) | (((R >> 2) & 1) << 1);
          seg[q] = *reinterpret_cast<const u32x4_t*>(sb + R * 256 + (((sg >> 2) ^ g) << 6) +
                                                     (sg & 3) * 16);
          drow[q] = is_q ? mb + R : mrow[i * 32 + R];
        }
        // cache rows are streamed out (not read again while cached); Q rows
        // are read by the attention that follows
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const int m = mb + 4 * q + (lane >> 4);
          u32x4_t* dst = reinterpret_cast<u32x4_t*>(sec_dst + (int64_t)drow[q] * p.d_q + sg * 8);
          if (full || m < M) {
            if (is_q) *dst = seg[q];
            else __builtin_nontemporal_store(seg[q], dst);
          }
        }
        __builtin_amdgcn_s_waitcnt(kWaitLgkm0);   // reads done before the next block's writes
        __builtin_amdgcn_wave_barrier();
        return;
      }
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int lr = 8 * (v >> 2) + row_q + (v & 3);
#pragma unroll
      for (int j = 0; j < 4; ++j) stg[lr * kEpiStride + j * 32 + col_l] = acc[i][j][v];
    }
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
    __builtin_amdgcn_wave_barrier();
    if constexpr (EPI == EPI_RESID || EPI == EPI_STORE || EPI == EPI_GELU ||
                  EPI == EPI_GELU_TANH) {
      if (EPI != EPI_STORE || !p.c_f32) {   // wave-uniform
        // Row-segment form: 16 lanes per row, 8 consecutive columns per lane
        // (two 16-byte LDS reads of the staged f32 row), so the residual
        // segment is one 16-byte load and the result one 16-byte store; the
        // 8 residual loads of a block are issued together (one memory
        // latency per block).  The sum is rounded to bf16 once.
        const bool full = mb + 32 <= M;
        const int sg = lane & 15;
        const int col = nw + 8 * sg;
        const bool col_in = !EXT || col < p.N;   // N is a multiple of 64: whole 8-column segments
        int drow[8];
        float scv[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const int R = 4 * q + (lane >> 4);
          drow[q] = EPI == EPI_RESID ? mrow[i * 32 + R] : mb + R;
          scv[q] = msc[i * 32 + R];
        }
        uint4 rres[8];
        if constexpr (EPI == EPI_RESID) {
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            const int m = mb + 4 * q + (lane >> 4);
            rres[q] = ((full || m < M) && col_in) ? *reinterpret_cast<const uint4*>(
                                            reinterpret_cast<const bf16*>(p.resid) +
                                            (int64_t)drow[q] * p.ldc + col)
                                      : make_uint4(0, 0, 0, 0);
          }
        }
        const float4 b0 = bias4(col_in ? bias : nullptr, col);
        const float4 b1 = bias4(col_in ? bias : nullptr, col + 4);
        const float bv[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const int R = 4 * q + (lane >> 4);
          const int m = mb + R;
          const float4 f0 = *reinterpret_cast<const float4*>(stg + R * kEpiStride + 8 * sg);
          const float4 f1 = *reinterpret_cast<const float4*>(stg + R * kEpiStride + 8 * sg + 4);
          const float f[8] = {f0.x, f0.y, f0.z, f0.w, f1.x, f1.y, f1.z, f1.w};
          float x[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            x[e] = f[e] * scv[q] + bv[e];
            if constexpr (EPI == EPI_GELU_TANH) x[e] = gelu_tanh(x[e]);
          }
          if constexpr (EPI == EPI_GELU) gelu_erf(x);
          if constexpr (EPI == EPI_RESID) {
            const uint32_t rw[4] = {rres[q].x, rres[q].y, rres[q].z, rres[q].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              x[2 * e] += __uint_as_float(rw[e] << 16);
              x[2 * e + 1] += __uint_as_float(rw[e] & 0xffff0000u);
            }
          }
          const uint4 o = make_uint4(pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]),
                                     pack_bf16x2(x[4], x[5]), pack_bf16x2(x[6], x[7]));
          if ((full || m < M) && col_in)
            *reinterpret_cast<uint4*>(reinterpret_cast<bf16*>(p.C) + (int64_t)drow[q] * p.ldc +
                                      col) = o;
        }
        __builtin_amdgcn_s_waitcnt(kWaitLgkm0);   // reads done before the next block's writes
        __builtin_amdgcn_wave_barrier();
        return;
      }
    }
    // Each block is emitted in phases: all LDS reads of a group of rounds
    // into registers, then the global loads they index, then arithmetic and
    // stores (the stores go through generic pointers, which the compiler
    // must otherwise keep ordered before later LDS reads).  Rows past M exist
    // only in the last block of a ragged tile; full blocks take the variant
    // without the per-row store check.
    auto emit = [&](auto check) {
      constexpr bool kCheck = decltype(check)::value;
      if (EPI == EPI_SWIGLU) {
        // 64 outputs per row (gate columns 0..63 of the wave, up columns
        // 64..127): 16 lanes per row, 4 rows per round, 8 rounds
        const int c = (lane & 15) * 4;
        float4 g[8], u[8];
        float sc[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          const int lr = 4 * r + (lane >> 4);
          g[r] = *reinterpret_cast<const float4*>(stg + lr * kEpiStride + c);
          u[r] = *reinterpret_cast<const float4*>(stg + lr * kEpiStride + 64 + c);
          sc[r] = msc[i * 32 + lr];
        }
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          const int m = mb + 4 * r + (lane >> 4);
          bf16x4_t o;
          o[0] = f2bf(silu(g[r].x * sc[r]) * (u[r].x * sc[r]));
          o[1] = f2bf(silu(g[r].y * sc[r]) * (u[r].y * sc[r]));
          o[2] = f2bf(silu(g[r].z * sc[r]) * (u[r].z * sc[r]));
          o[3] = f2bf(silu(g[r].w * sc[r]) * (u[r].w * sc[r]));
          if (!kCheck || m < M)
            *reinterpret_cast<bf16x4_t*>(reinterpret_cast<bf16*>(p.C) + (int64_t)m * p.ldc +
                                         nw / 2 + c) = o;
        }
      } else {
        // 2 rows per round (32 lanes x 4 columns each), 16 rounds in groups of
        // G (4 for the rotary epilogues, whose rounds hold 4 float4 each)
        constexpr bool kRope = EPI == EPI_QKV || EPI == EPI_KV;
        constexpr int G = kRope ? 4 : 8;
        const bool rope = kRope && !is_v && p.rope_cos;   // wave-uniform
        const bool col_in = !EXT || nw + c4 < p.N;        // N is a multiple of 4
        const float4 bx = bias4(col_in ? bias : nullptr, nw + c4);
        const float4 by = rope ? bias4(bias, nw + (c4 ^ half)) : bx;
        // a wave's 128 columns lie in one section (Q, K or V) when d_q is a
        // multiple of 128; otherwise (no RoPE then) each lane finds its own
        const bool sec_wave = !EXT || p.d_q % 128 == 0;     // wave-uniform
#pragma unroll
        for (int hh = 0; hh < 16 / G; ++hh) {
          float4 x4[G], y4[G], cs[G], sn[G];
          float sc[G];
          int mr[G], mp[G];
          bf16x4_t rv[G];
#pragma unroll
          for (int r = 0; r < G; ++r) {
            const int lr = 2 * (G * hh + r) + (lane >> 5);
            x4[r] = *reinterpret_cast<const float4*>(stg + lr * kEpiStride + c4);
            if (rope)
              y4[r] = *reinterpret_cast<const float4*>(stg + lr * kEpiStride + (c4 ^ half));
            sc[r] = msc[i * 32 + lr];
            mr[r] = mrow[i * 32 + lr];
            mp[r] = mpos[i * 32 + lr];
          }
#pragma unroll
          for (int r = 0; r < G; ++r) {
            if (EPI == EPI_RESID && col_in)
              rv[r] = *reinterpret_cast<const bf16x4_t*>(p.resid + (int64_t)mr[r] * p.ldc + nw + c4);
            if (rope) {
              const int c = (cbase + c4) & (hd - 1);
              const int64_t t = (int64_t)mp[r] * half + (c & (half - 1));
              cs[r] = *reinterpret_cast<const float4*>(p.rope_cos + t);
              sn[r] = *reinterpret_cast<const float4*>(p.rope_sin + t);
            }
          }
#pragma unroll
          for (int r = 0; r < G; ++r) {
            const int m = mb + 2 * (G * hh + r) + (lane >> 5);
            const float x[4] = {x4[r].x * sc[r] + bx.x, x4[r].y * sc[r] + bx.y,
                                x4[r].z * sc[r] + bx.z, x4[r].w * sc[r] + bx.w};
            bf16x4_t o;
            if (EPI == EPI_GELU_TANH) {
#pragma unroll
              for (int e = 0; e < 4; ++e) o[e] = f2bf(gelu_tanh(x[e]));
              if ((!kCheck || m < M) && col_in)
                *reinterpret_cast<bf16x4_t*>(reinterpret_cast<bf16*>(p.C) + (int64_t)m * p.ldc +
                                             nw + c4) = o;
            } else if (EPI == EPI_STORE) {
              const int64_t off = (int64_t)m * p.ldc + nw + c4;
              if ((!kCheck || m < M) && col_in) {
                if (p.c_f32) {
                  *reinterpret_cast<float4*>(reinterpret_cast<float*>(p.C) + off) =
                      make_float4(x[0], x[1], x[2], x[3]);
                } else {
#pragma unroll
                  for (int e = 0; e < 4; ++e) o[e] = f2bf(x[e]);
                  *reinterpret_cast<bf16x4_t*>(reinterpret_cast<bf16*>(p.C) + off) = o;
                }
              }
            } else if (EPI == EPI_RESID) {
#pragma unroll
              for (int e = 0; e < 4; ++e) o[e] = f2bf(x[e] + bf2f(rv[r][e]));
              if ((!kCheck || m < M) && col_in)
                *reinterpret_cast<bf16x4_t*>(reinterpret_cast<bf16*>(p.C) +
                                             (int64_t)mr[r] * p.ldc + nw + c4) = o;
            } else {  // EPI_QKV / EPI_KV
              if (!rope) {
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = f2bf(x[e]);
              } else {
                // rotate-half RoPE: column c pairs with c +- hd/2 of the same head
                const float y[4] = {y4[r].x * sc[r] + by.x, y4[r].y * sc[r] + by.y,
                                    y4[r].z * sc[r] + by.z, y4[r].w * sc[r] + by.w};
                const int c = (cbase + c4) & (hd - 1);   // column within the head
                const float cv[4] = {cs[r].x, cs[r].y, cs[r].z, cs[r].w};
                const float sv[4] = {sn[r].x, sn[r].y, sn[r].z, sn[r].w};
#pragma unroll
                for (int e = 0; e < 4; ++e)
                  o[e] = f2bf(c < half ? x[e] * cv[e] - y[e] * sv[e] : x[e] * cv[e] + y[e] * sv[e]);
              }
              if (rope || sec_wave) {
                const int64_t drow = is_q ? (int64_t)m : (int64_t)mr[r];
                if ((!kCheck || m < M) && col_in)
                  *reinterpret_cast<bf16x4_t*>(sec_dst + drow * p.d_q + c4) = o;
              } else {
                const int secl = (nw + c4) / p.d_q;
                const bool lq = EPI == EPI_QKV && secl == 0;
                const bool lv = EPI == EPI_QKV ? secl == 2 : (EPI == EPI_KV && secl == 1);
                bf16* ldst = lq ? p.q_out
                                : (lv ? p.v_cache : p.k_cache) +
                                      (GROUPED ? (int64_t)(layer - 1) * p.cache_layer_stride : 0);
                const int64_t drow = lq ? (int64_t)m : (int64_t)mr[r];
                if ((!kCheck || m < M) && col_in)
                  *reinterpret_cast<bf16x4_t*>(ldst + drow * p.d_q + nw + c4 - secl * p.d_q) = o;
              }
            }
          }
        }
      }
    };
    if (mb + 32 <= M) emit(std::false_type{});
    else emit(std::true_type{});
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);   // block reads done before the next block's writes
    __builtin_amdgcn_wave_barrier();
  };
  block(std::integral_constant<int, 0>{});
  if constexpr (MB >= 2) block(std::integral_constant<int, 1>{});
  if constexpr (MB == 4) {
    block(std::integral_constant<int, 2>{});
    block(std::integral_constant<int, 3>{});
  }
}

// Epilogue of 4 consecutive output columns n..n+3 of compact row m from
// their sums x4 (row scale sc): for the split GEMMs, whose sums come from
// partial tiles.  partner(dc): the sums dc columns further (the rotary
// partner); up(): SwiGLU's up sums of the same outputs.
template <int EPI, class Partner, class Up>
__device__ __forceinline__ void epilogue4(const GP& p, int m, int n, float sc, float4 x4,
                                          Partner&& partner, Up&& up) {
  const float4 bx = bias4(p.bias, n);
  float x[4] = {x4.x * sc + bx.x, x4.y * sc + bx.y, x4.z * sc + bx.z, x4.w * sc + bx.w};
  bf16x4_t o;
  if (EPI == EPI_GELU || EPI == EPI_GELU_TANH) {
    if constexpr (EPI == EPI_GELU) gelu_erf(x);
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = f2bf(EPI == EPI_GELU ? x[e] : gelu_tanh(x[e]));
    *reinterpret_cast<bf16x4_t*>(reinterpret_cast<bf16*>(p.C) + (int64_t)m * p.ldc + n) = o;
  } else if (EPI == EPI_STORE) {
    const int64_t off = (int64_t)m * p.ldc + n;
    if (p.c_f32) {
      *reinterpret_cast<float4*>(reinterpret_cast<float*>(p.C) + off) =
          make_float4(x[0], x[1], x[2], x[3]);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = f2bf(x[e]);
      *reinterpret_cast<bf16x4_t*>(reinterpret_cast<bf16*>(p.C) + off) = o;
    }
  } else if (EPI == EPI_RESID) {
    const int64_t off = (int64_t)p.rows[m] * p.ldc + n;
    const bf16x4_t r = *reinterpret_cast<const bf16x4_t*>(p.resid + off);
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = f2bf(x[e] + bf2f(r[e]));
    *reinterpret_cast<bf16x4_t*>(reinterpret_cast<bf16*>(p.C) + off) = o;
  } else if (EPI == EPI_SWIGLU) {
    const float4 u4 = up();
    const float u[4] = {u4.x * sc, u4.y * sc, u4.z * sc, u4.w * sc};
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = f2bf(silu(x[e]) * u[e]);
    *reinterpret_cast<bf16x4_t*>(reinterpret_cast<bf16*>(p.C) + (int64_t)m * p.ldc + n) = o;
  } else {  // EPI_QKV
    const int sec = n / p.d_q, cin = n - sec * p.d_q;
    const int row = p.rows[m];
    const bool is_v = sec == 2;
    bf16* dst = sec == 0 ? p.q_out + (int64_t)m * p.d_q
                         : (is_v ? p.v_cache : p.k_cache) +
                               (int64_t)(p.slot ? p.slot[row] : row) * p.d_q;
    if (is_v || !p.rope_cos) {
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = f2bf(x[e]);
    } else {
      // rotate-half RoPE: column c pairs with c +- hd/2 of the same head
      const int hd = p.head_dim, half = hd >> 1;
      const int c = cin & (hd - 1);
      const float4 y4 = partner((n ^ half) - n);
      const float4 by = bias4(p.bias, n ^ half);
      const float y[4] = {y4.x * sc + by.x, y4.y * sc + by.y, y4.z * sc + by.z, y4.w * sc + by.w};
      const int64_t t = (int64_t)p.pos[row] * half + (c & (half - 1));
      const float4 cs = rope4(p.rope_cos + t), sn = rope4(p.rope_sin + t);
      const float cv[4] = {cs.x, cs.y, cs.z, cs.w}, sv[4] = {sn.x, sn.y, sn.z, sn.w};
#pragma unroll
      for (int e = 0; e < 4; ++e)
        o[e] = f2bf(c < half ? x[e] * cv[e] - y[e] * sv[e] : x[e] * cv[e] + y[e] * sv[e]);
    }
    *reinterpret_cast<bf16x4_t*>(dst + cin) = o;
  }
}

// Row tiles per raster group: the tiles running together on an XCD cover a
// block of about kRasterRows row tiles by a few column tiles.
constexpr int kRasterRows = 8;

// Tile t of the raster: groups of kRasterRows row tiles, row tiles fastest.
__device__ __forceinline__ void raster_tile(int t, int tiles_m, int tiles_n, int* mt, int* nt) {
  const int gsz = kRasterRows * tiles_n;
  const int g = t / gsz, r = t - g * gsz;
  const int rows_in_g = min(kRasterRows, tiles_m - g * kRasterRows);
  *mt = g * kRasterRows + r % rows_in_g;
  *nt = r / rows_in_g;
}

inline GP to_gp(const GemmArgs& g) {
  GP p{};
  p.M_max = g.M_max; p.M_dev = g.M_dev; p.N = g.N; p.K = g.K;
  p.A = (const bf16*)g.A; p.a_rows = g.a_rows; p.lda = g.lda;
  p.B = (const bf16*)g.B; p.B2 = (const bf16*)g.B2; p.ldb = g.ldb;
  p.C = g.C; p.ldc = g.ldc; p.c_f32 = g.c_f32; p.row_scale = g.row_scale;
  p.rows = g.rows; p.resid = (const bf16*)g.resid; p.pos = g.pos; p.slot = g.slot;
  p.bias = (const bf16*)g.bias;
  p.rope_cos = g.rope_cos; p.rope_sin = g.rope_sin; p.head_dim = g.head_dim; p.d_q = g.d_q;
  p.q_out = (bf16*)g.q_out; p.k_cache = (bf16*)g.k_cache; p.v_cache = (bf16*)g.v_cache;
  p.bias_layer_stride = g.bias_layer_stride; p.a_sorted = g.a_sorted;
  p.A2 = (const bf16*)g.A2; p.a_sel = g.a_sel;
  p.rinv_out = g.rinv_out; p.ln_out = (bf16*)g.ln_out; p.row_eps = g.row_eps;
  p.has_exit = g.exit != nullptr;
  if (g.exit) p.ex = *g.exit;
  return p;
}

// The extended instantiation only where the shape or the inputs need it.
inline bool tile_needs_ext(const GP& p, int epi, int tile) {
  return (epi != EPI_SWIGLU && p.N % tile != 0) ||
         ((epi == EPI_QKV || epi == EPI_KV) && p.d_q % 128 != 0) || p.a_sel != nullptr;
}

// Sets a kernel's dynamic-LDS limit once per process.
inline adept_status lds_limit(const void* kernel, size_t bytes, bool* done, const char* what) {
  if (*done) return ADEPT_OK;
  if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) !=
      hipSuccess)
    return launch_status(what);
  *done = true;
  return ADEPT_OK;
}

// The skinny path's cut of the weights (gemm.hip): units of one 64-column tile
// times one 64-deep k step, in equal contiguous ranges, one per workgroup.
constexpr int kSkinnyBN = 64;     // output columns per tile
struct SkSplit {
  int G;        // workgroups
  int U;        // units per workgroup (the last one may hold fewer)
  int KT;       // k steps per tile
  int64_t total;
};
SkSplit skinny_split(int Nt, int K);

// The smaller tiles.  mid_choose: which tile the GEMM takes; gemm_mid_128x256
// and gemm_mid_128x128 run it, cutting tiles along K into the workspace when
// it has mid_ws_bytes.
enum MidTile { kTileLarge = 0, kTile128x256 = 1, kTile128x128 = 2 };
MidTile mid_choose(const GP& p, int epi, size_t ws_bytes);
adept_status gemm_mid_128x256(GP p, int epi, const char* name, float* ws, size_t ws_bytes,
                              hipStream_t s);
adept_status gemm_mid_128x128(GP p, int epi, const char* name, float* ws, size_t ws_bytes,
                              hipStream_t s);

}  // namespace adept
