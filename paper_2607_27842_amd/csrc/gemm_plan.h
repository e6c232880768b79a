// Host side of the bf16 GEMM launches: which output tile a problem (or two in one launch) takes.
// Plain arithmetic on the shapes, without HIP.
#pragma once
#include <stdint.h>

#include <algorithm>

namespace ff {

// M x N outputs over K; operand rows lda and ldw elements apart.  Row r of A is row
// r % seg of sample r / seg, samples `rows` rows apart (seg == rows: consecutive).
struct GemmShape { int M, N, K, lda, ldw, seg, rows; };

// Tile choice: the candidate with the least estimated time.  A round of workgroups takes
// lat + k * K us, bound by its own chain of stages.  A grid takes at least pow us per 256 tiles and unit
// of K: for the 256-row tiles the card's power limit (large grids: the clock falls to about 1.9 GHz, so
// that a grid that leaves CUs idle runs its tiles faster), for the others what the caches deliver at
// long K, about (BM + BN) bytes * 2 * K per tile at 8 to 14 TB/s.  Tiles that leave room for a second
// workgroup per CU take lat2 + k2 * K for a round of 257 to 512.
// Measured on MI355X with random bf16 data; 256-row tiles run k_gemm_pp (three stages or more), the
// others k_gemm_ks (four or more), the register-staged kernel k_gemm_bf16 (any K, and operand rows
// beyond 32-bit offsets of each other).
// In us at K = 1152 / 4608 for one round of few tiles: 256x256 31 / 85, 256x192 28 / 70, 256x128
// 21 / 57-69, 128x192 19 / 58, 128x128 15 / 33, 128x96 13.6 / 30, 128x64 9.3 / 22.5, 64x96 8.1 / 19,
// 64x64 7.0 / 15.6 (288 tiles: 10.3 / 26.7), 64x32 6.1 / 12.9 (288: 8.2 / 20.5), 64x96 with 384 tiles
// 14.5 / 37; a full round at K = 3072 (clock down): 77, 62, 47 us for the 256-row tiles.
// The pow of the smaller tiles and the k of three of them are fitted to the GEMMs of DiT blocks, each on
// every tile: widths 256 to 4096, 256 to 8192 rows, K up to 16384, 618 shapes; over those with K > 256
// the choice is 0.6 % above the best tile on average (with pow from K = 4608 alone: 2.6 %).  What that
// changed: M = 256, N = 16384, K = 4096 70 (64x96) -> 49 us (128x128); M = 768, N = 4096, K = 16384 194 (64x96) ->
// 138 (128x128); M = 3328, N = 1152, K = 4608 55 (64x96) -> 39 (128x128); M = 768, N = 2432, K = 9728 73 (128x96) ->
// 62 (128x64); M = 256, N = 3072, K = 12288 76 (64x96) -> 60 (64x64).
// What the 256-row tiles take against the kernels before them (256x256 and 256x192 of 32x32x16
// MFMAs with one wait and barrier per stage): M = 4608, N = 21504, K = 3072 545 -> 460 us
// (1324 TFLOP/s), 4096 x 3072 x 12288 263 -> 222 us, 14310 x 8192 x 2048 440 -> 370 us.
enum { kTile256, kTile256x192, kTile256x128, kTile128x192, kTile128, kTile128x96, kTile128x64, kTile64x96, kTile64,
       kTile64x32, kTileCount, kTileShort64 = kTileCount, kTileShort64x32, kTileReg };
constexpr int kShortStages = 3;   // most stages of the short tiles
struct TilePlan { int tile; double cost; };
struct TileCost { int bm, bn; double lat, k, pow, lat2, k2; };
constexpr TileCost kTileCost[kTileCount] = {
    {256, 256, 15.0, 0.0150, 0.0245, 0, 0},  {256, 192, 13.0, 0.0122, 0.0192, 0, 0},
    {256, 128, 7.5, 0.0118, 0.0145, 0, 0},   {128, 192, 8.0, 0.0108, 0.0112, 0, 0},
    {128, 128, 8.0, 0.0076, 0.0095, 0, 0},   {128, 96, 8.0, 0.0048, 0.0083, 0, 0},
    {128, 64, 4.8, 0.0042, 0.0049, 0, 0},    {64, 96, 4.6, 0.0035, 0.0045, 6.5, 0.0062},
    {64, 64, 4.2, 0.0025, 0.0034, 5.0, 0.0047}, {64, 32, 3.9, 0.0020, 0.0028, 4.0, 0.0036}};

constexpr double kNoCost = 1e300;   // no tile of the table fits: the register-staged kernel

// Short K: lat + k * K us for a small grid, base + tile_us + tile_k * K per 256 tiles for a larger one.
// Up to three stages the short tiles (every stage has a buffer, so nothing waits for a refill), up
// to kRegK the register-staged kernel, whose few large tiles store faster than the card runs many
// small ones.  Measured, us, in brackets in the kernel before all of these: K = 192, M = 512, N = 576
// 4.5 (64x32), 8.0 (256x128), [5.3]; K = 128, M = 4096, N = 128 gated 5.3 (64x32), 7.7 register-staged, [6.1];
// K = 128, M = 16384, N = 512 9.9 register-staged, 15.0 (64x64), [11.3]; K = 256, M = 4096, N = 1024 9.1
// register-staged, 11.7 (128x128), 12.2 (256x128), [10.4].  At K = 320 the other tiles are level with it.
constexpr int kRegK = 256;
struct ShortCost { int tile, bm, bn; double lat, k, base, tile_us, tile_k; };
constexpr ShortCost kShortCost[3] = {{kTileShort64, 64, 64, 4.2, 0.0058, 4.0, 0.80, 0.0035},
                                     {kTileShort64x32, 64, 32, 3.8, 0.0050, 4.0, 0.56, 0.0016},
                                     {kTileReg, 128, 128, 4.4, 0.0170, 4.4, 0.50, 0.0135}};

inline long tiles_of(const GemmShape* a, int n, unsigned bm, unsigned bn) {
  long t = 0;
  for (int i = 0; i < n; ++i) t += (long)(((unsigned)a[i].M + bm - 1) / bm) * (((unsigned)a[i].N + bn - 1) / bn);
  return t;
}

// The operand rows of every bm x bn tile lie within a 32-bit byte offset of its first row (bm
// consecutive rows of a row map span at most (bm - 1) / seg + 1 further samples, and no more than
// there are), with room left for the offset along K.
inline bool dma_ok(const GemmShape* a, int n, int bm, int bn) {
  for (int i = 0; i < n; ++i) {
    const int more = std::min((bm - 1) / a[i].seg + 1, (a[i].M - 1) / a[i].seg);
    const uint64_t span = a[i].seg == a[i].rows ? bm : (uint64_t)more * a[i].rows + bm;
    if (span * a[i].lda * 2 > 0xf0000000ull || (uint64_t)bn * a[i].ldw * 2 > 0xf0000000ull) return false;
  }
  return true;
}

// 64-wide K stages of the problem with the fewest
inline int min_stages(const GemmShape* a, int n) {
  int nk = (a[0].K + 63) / 64;
  for (int i = 1; i < n; ++i) nk = std::min(nk, (a[i].K + 63) / 64);
  return nk;
}

// n (1 or 2) problems in one launch, each with rows and columns
inline TilePlan plan_tiles(const GemmShape* a, int n) {
  TilePlan best{kTileReg, kNoCost};
  const int nk = min_stages(a, n);
  int K = 0;
  for (int i = 0; i < n; ++i) K = std::max(K, a[i].K);
  const bool near = dma_ok(a, n, 256, 256);   // then every tile's rows are
  for (int c = 0; c < kTileCount; ++c) {
    if (nk < (c <= kTile256x128 ? 3 : c == kTile128 ? 5 : 4)) continue;   // the stages that the kernel's prologue takes
    const TileCost& t = kTileCost[c];
    if (!near && !dma_ok(a, n, t.bm, t.bn)) continue;
    const long tiles = tiles_of(a, n, t.bm, t.bn), slots = t.lat2 > 0 ? 512 : 256, rest = tiles % slots;
    const double one = t.lat + t.k * K, full = t.lat2 > 0 ? t.lat2 + t.k2 * K : one;
    const double cost = std::max(tiles / slots * full + (rest == 0 ? 0 : rest <= 256 ? one : full), tiles / 256.0 * t.pow * K);
    if (cost < best.cost) best = TilePlan{c, cost};
  }
  if (K > kRegK) return best;
  for (const ShortCost& t : kShortCost) {
    if (t.tile != kTileReg && (K > 64 * kShortStages || !(near || dma_ok(a, n, t.bm, t.bn)))) continue;
    const double rounds = tiles_of(a, n, t.bm, t.bn) / 256.0;
    const double cost = std::max(t.lat + t.k * K, t.base + rounds * (t.tile_us + t.tile_k * K));
    if (cost < best.cost) best = TilePlan{t.tile, cost};
  }
  return best;
}

// Two problems share a launch when that is estimated to take no longer than two.  The margin on that
// is set by three near ties: proj of 512 + 1024 rows, N = K = 3072 (41.2 against 40.9 us in two), takes
// 45 us in one launch and about 50 in two; fc1 of 256 + 14310 rows, N = 8192, K = 2048 (365.8 against
// 364.6), is 24 us faster in one; fc1 of 512 + 1024 rows, N = 12288, K = 3072 (101.0 against 100.2), is 4 us
// faster in two.  Where one of the problems fits no tile, the other keeps its own.
inline bool plan_grouped(const GemmShape& a0, const GemmShape& a1) {
  const GemmShape both[2] = {a0, a1};
  const double b = plan_tiles(both, 2).cost, c0 = plan_tiles(&a0, 1).cost, c1 = plan_tiles(&a1, 1).cost;
  return b == kNoCost ? c0 == kNoCost && c1 == kNoCost : b <= 1.0035 * (c0 + c1) + 0.2;
}

}  // namespace ff
