// The 128x256 tiles of gemm_mid.h, and the choice of tile and plan.
#include "gemm_mid.h"

namespace adept {
namespace {

// Measured times (us, MI355X) of a 64-deep k stage of the workgroups of one
// round, by how many of them run (w <= slots): one per CU costs little more
// than one alone, two per CU (128x128) take turns on the CU's load path, and
// the 128x256 tile slows towards a full chip (loads through L2).  Weights that
// few row tiles share come from HBM: with u = w / tm streams of them a stage
// waits up to about 0.9 us for its loads.  `fixed`: the rest of a tile (first
// loads, epilogue).
struct Tile {
  int cols, slots;
  double fixed;
};
constexpr Tile kTileA{128, 512, 3.0}, kTileB{256, 256, 6.5};
constexpr double kLargeStage = 1.25, kLargeFixed = 18.0;   // 256x256, 256 slots
constexpr double kLargeGelu = 10.0;      // its GELU epilogues, over 4 blocks a wave
constexpr double kReduceUs = 4.0;        // the second kernel
constexpr double kPartBytesUs = 6.0e6;   // bytes per us the partial sums are written and read at

double stage_us(const Tile& c, int w, int tm) {
  const double f = w / 256.0;
  const double hbm = 0.5 + 0.4 * std::min(1.0, (double)w / tm * c.cols / 16384.0);
  const double t = c.cols == 256 ? 0.62 + 0.31 * f * f
                                 : (w <= 256 ? 0.50 + 0.04 * f : 0.88 + 0.18 * (f - 1.0));
  return std::max(t, hbm);
}

// w workgroups of `stages` k stages each, in rounds of the chip.
double rounds_us(const Tile& c, int64_t w, double stages, int tm) {
  const int64_t full = w / c.slots;
  const int rest = (int)(w % c.slots);
  double t = full * (c.fixed + stages * stage_us(c, c.slots, tm));
  if (rest) t += c.fixed + stages * stage_us(c, rest, tm);
  return t;
}

// The cheapest plan for tm x tn tiles: whole rounds in one piece, the tiles
// left over cut into as many pieces as one round holds, one or two per CU
// (S = 1: nothing cut).
double best_plan(const Tile& c, int tm, int tn, int KT, bool split, int* tail, int* S) {
  const int64_t T = (int64_t)tm * tn;
  double best = rounds_us(c, T, KT, tm);
  *tail = 0;
  *S = 1;
  if (!split || tm > kMidMaxTm) return best;
  for (int unit = 256; unit <= c.slots; unit *= 2) {
    const int rest = (int)(T % unit);
    if (rest == 0) continue;
    const double full = rounds_us(c, T - rest, KT, tm);
    for (int w = 256; w <= c.slots; w *= 2) {
      const int s = std::min({w / rest, KT / kMidMinStages, kMidMaxS});
      if (s < 2) continue;
      const double bytes = 2.0 * rest * s * kMidRows * c.cols * 4.0;
      const double t = full + rounds_us(c, (int64_t)rest * s, (double)((KT + s - 1) / s), tm) +
                       kReduceUs + bytes / kPartBytesUs;
      if (t < best) {
        best = t;
        *tail = rest;
        *S = s;
      }
    }
  }
  return best;
}

const Tile& tile_of(int cols) { return cols == 128 ? kTileA : kTileB; }

}  // namespace

MidBound mid_table(int cols, int M_max, int tiles_n, int KT, bool split, MidTable* out) {
  MidBound b{0, 0, 0};
  const int tm_max = ceil_div(M_max, kMidRows);
  for (int tm = 1; tm <= std::min(tm_max, kMidMaxTm); ++tm) {
    int tail, S;
    best_plan(tile_of(cols), tm, tiles_n, KT, split, &tail, &S);
    if (out) {
      out->tail[tm - 1] = (uint16_t)tail;
      out->S[tm - 1] = (uint8_t)S;
    }
    const MidPlan pl{tm * tiles_n - tail, tail, S};
    b.blocks = std::max(b.blocks, pl.full_blocks() + pl.tail_blocks());
    b.tail = std::max(b.tail, tail);
    b.pieces = std::max(b.pieces, tail * S);
  }
  if (tm_max > kMidMaxTm)
    b.blocks = std::max(b.blocks, MidPlan{tm_max * tiles_n, 0, 1}.full_blocks());
  return b;
}

// An upper bound over the plans (no plan is made): a round's pieces of either
// tile are 32 MiB, and there are no more than every tile cut kMidMaxS ways.
size_t mid_ws_bytes(int M_max, int N, int K, int epi) {
  if (!mid_cuts(epi) || M_max <= 0 || N <= 0 || K < BK) return 0;
  const int64_t most = std::min(K / BK / kMidMinStages, kMidMaxS);
  if (most < 2) return 0;
  // in 128x128 tiles, of which a 128x256 tile is two
  const int64_t tiles =
      (int64_t)std::min(ceil_div(M_max, kMidRows), kMidMaxTm) * 2 * mid_tiles_n(256, N, epi);
  return (size_t)std::min<int64_t>(tiles * most, 512) * kMidRows * 128 * sizeof(float);
}

MidTile mid_choose(const GP& p, int epi, size_t ws_bytes) {
  const int KT = p.K / BK, tm = ceil_div(p.M_max, kMidRows);
  int tail, S;
  const int tl = ceil_div(p.M_max, 256) * mid_tiles_n(256, p.N, epi);
  const bool gelu = epi == EPI_GELU || epi == EPI_GELU_TANH;
  double best = ceil_div(tl, 256) * (kLargeFixed + (gelu ? kLargeGelu : 0.0) + kLargeStage * KT);
  MidTile pick = kTileLarge;
  const bool split = mid_cuts(epi) && ws_bytes > 0 &&
                     ws_bytes >= mid_ws_bytes(p.M_max, p.N, p.K, epi);
  const double b = best_plan(kTileB, tm, mid_tiles_n(256, p.N, epi), KT, split, &tail, &S);
  if (b < best) { best = b; pick = kTile128x256; }
  const double a = best_plan(kTileA, tm, mid_tiles_n(128, p.N, epi), KT, split, &tail, &S);
  if (a < best) pick = kTile128x128;
  return pick;
}

adept_status gemm_mid_128x256(GP p, int epi, const char* name, float* ws, size_t ws_bytes,
                              hipStream_t s) {
  return gemm_mid<Geo<128, 256>>(p, epi, name, ws, ws_bytes, s);
}

}  // namespace adept
