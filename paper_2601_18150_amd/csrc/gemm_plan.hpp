// Which kernel and tile a dense blockwise-scaled FP8 product runs on: plain host
// arithmetic on (m, n, k), no HIP, so that the choices can be checked on the CPU.
#pragma once

#include <stdint.h>

namespace fp8rl {

constexpr int kCus = 256;     // MI355X

// Few tokens: dense products of at most kSmallTokens tokens, and grouped ones of
// at most kSmallRowsPerExpert rows per expert on average, stream the weights once
// (gemm_small.hpp) instead of running padded output tiles.
constexpr int64_t kSmallTokens = 64;
constexpr int64_t kSmallRowsPerExpert = 12;
constexpr int64_t kSmallMaxN = int64_t(1) << 24;     // one workgroup per 16-64 weight rows: grid limit

inline bool few_tokens(int64_t m, int64_t n) { return m <= kSmallTokens && n < kSmallMaxN; }

// Dense products are one round or several of tiles over the 256 CUs, and a tile's
// time is its K blocks times a step time that hardly depends on the shape; so the
// tile is the one with the smallest (rounds x step time).  Step times (us per
// 128-wide K block and round, Qwen3-8B linears, 80 .. 2000 tokens, weights from HBM;
// about 3 us per call besides):
//   64x64      0.32   gemm_pipe, two wave groups split K
//   64x128, 128x64  0.49   the same
//   128x128    0.66   gemm_pipe, eight waves, 4-slot ring
//   128x256, 256x128  1.2 (1.07 with few bytes of weights)  gemm_pipe, 3-slot ring
//   256x256    1.5 in one round, 1.75 a round in several (2.05 at 8192 tokens, where
//              the power limit lowers the clock)   gemm_tiles
//   128x128, two workgroups per CU walking their tiles as one pipeline (gemm_tiles):
//              1.25 per 512 tiles, 0.75 for a last half
// Against the three fixed ranges of rows that chose the tile before (us): M = 300
// qkv 32.2 -> 17.9, o_proj 31.4 -> 15.8, gate_up 68.9 -> 53.8, down 87 -> 38.8; M = 777
// o_proj 31.4 -> 23.2, down 86.3 -> 60.5; M = 2000 qkv 64.8 -> 53.4, gate_up 228.7 ->
// 183.8; M = 256 o_proj 15.9 -> 13.2, qkv 21.2 -> 18.6.
// Tiles are BN x BM, in the order that breaks ties.
enum class Tile { k64x64, k64x128, k128x64, k128x128, k128x256, k256x128, k256x256, kPersistent };

struct TileChoice {
  Tile tile;
  double step;      // rounds x step time, us per K block
};

struct TileCost {
  Tile tile;
  int bn, bm;
  double one, more;      // us per K block: a single round, each of several
};
constexpr TileCost kTileCosts[] = {
    {Tile::k64x64, 64, 64, 0.32, 0.32},     {Tile::k64x128, 64, 128, 0.49, 0.49},
    {Tile::k128x64, 128, 64, 0.49, 0.49},   {Tile::k128x128, 128, 128, 0.66, 0.66},
    {Tile::k128x256, 128, 256, 1.2, 1.2},   {Tile::k256x128, 256, 128, 1.2, 1.2},
    {Tile::k256x256, 256, 256, 1.5, 1.75},
};

// A launch of one workgroup of 512 threads per tile: HIP takes less than 2^32 threads
// in a grid dimension.  (The persistent grid has no such limit.)
constexpr int kTileThreads = 512;
constexpr int64_t kMaxTiles = ((int64_t(1) << 32) - 1) / kTileThreads;

inline int64_t tile_count(const TileCost& c, int64_t m, int64_t n) {
  return ((m + c.bm - 1) / c.bm) * ((n + c.bn - 1) / c.bn);
}

// The smallest rounds x step time.
inline TileChoice tile_for(int64_t m, int64_t n) {
  const int64_t tiles128 = ((m + 127) / 128) * (n / 128), pairs = tiles128 / 512, rest = tiles128 % 512;
  TileChoice best{Tile::kPersistent, 1.25 * (double)pairs + (rest == 0 ? 0.0 : rest <= 256 ? 0.9 : 1.25)};
  if (pairs > 0 && rest > 0 && rest <= 256) best.step -= 0.15;
  for (const TileCost& c : kTileCosts) {
    const int64_t tiles = tile_count(c, m, n);
    if (tiles > kMaxTiles) continue;
    const int64_t rounds = (tiles + kCus - 1) / kCus;
    const double step = rounds == 1 ? c.one : c.more * (double)rounds;
    if (step < best.step) best = {c.tile, step};
  }
  return best;
}

// A nearly empty last round costs almost as much as a full one.  Where that is dear,
// the first n1 output columns run as whole rounds of 256x256 tiles and the others as a
// product of their own with the tile that suits them (n1 = 0: one launch for all), if
// the table promises a tenth with the second launch's 3 us counted.  Qwen3-8B, one
// launch / two, us: gate_up M = 777 106.7 / 96.5, M = 1000 110.9 / 103.1, M = 1300 160.3 /
// 149.6; M = 3001 qkv 92.4 / 80.6; M = 5000 down 267 / 246.  Smaller promises are within
// the table's error (gate_up M = 1600, 5%: 169 / 170; M = 3001, 3%: 283 / 293), and so were
// those of the smaller tiles (M = 1300 down, 4%: 89.8 / 98.5).
struct ColumnSplit {
  int64_t n1;
  Tile first;
  Tile rest;             // (n1 = 0: the tile of the whole product)
};

inline ColumnSplit column_split(int64_t m, int64_t n, int64_t k) {
  const double kb = (double)(k / 128);
  const TileChoice whole = tile_for(m, n);
  constexpr TileCost c = kTileCosts[sizeof(kTileCosts) / sizeof(kTileCosts[0]) - 1];
  static_assert(c.tile == Tile::k256x256, "the last entry");
  const int64_t tiles_m = (m + c.bm - 1) / c.bm;
  if (tiles_m <= kCus) {
    const int64_t per_round = kCus / tiles_m, rounds = n / c.bn / per_round, n1 = rounds * per_round * c.bn;
    if (rounds >= 1 && n1 < n && tile_count(c, m, n1) <= kMaxTiles) {
      const TileChoice rest = tile_for(m, n - n1);
      const double both = ((rounds == 1 ? c.one : c.more * (double)rounds) + rest.step) * kb + 3.0;
      if (both < 0.9 * whole.step * kb) return {n1, c.tile, rest.tile};
    }
  }
  return {0, c.tile, whole.tile};
}

// K ranges of a split product (1: never split).
inline int splitk_ranges(int64_t m, int64_t n, int64_t k) {
  // Split K only when the 128x128 tiles cover less than half of MI355X's 256
  // CUs, into the largest power of two of ranges that keeps tiles x splits
  // within 256, each range at least 4 K blocks long.  (Measured on the decode
  // linears, M = 256: more ranges lose to the fp32 partial-sum traffic, which
  // grows with the split.)
  if (m <= 0 || n <= 0 || k <= 0 || (m >= 2048 && n >= 2048)) return 1;
  // decode batches run unsplit on 64x64 tiles when K is short enough for one
  // workgroup's K loop (Qwen3-8B qkv, o_proj: K = 4096; down, K = 12288, splits)
  if (m > 128 && m <= 256 && k <= 4096 && ((m + 63) / 64) * (n / 64) <= 512) return 1;
  const int64_t tiles = ((m + 127) / 128) * (n / 128);
  if (2 * tiles >= kCus) return 1;
  int64_t s = 1;
  while (2 * s * tiles <= kCus) s *= 2;
  const int64_t by_k = (k / 128) / 4;
  if (s > by_k) s = by_k;
  return s > 1 ? (int)s : 1;
}

// Whether the `splits` ranges of splitk_ranges are run, where there is room for their
// partial sums.  Few tokens need no K ranges across workgroups (measured at M = 64,
// down: 20.6 us against 20.2 us split with its reduction; every other shape faster), and
// others only where their ranges, the partial sums (16 MiB: 9 us) and the second launch
// beat the unsplit tile.  Split / unsplit us: M = 128 down 22.9 / 34, M = 256 down 29.6 /
// 34; M = 128 qkv 18.7 / 13.5, o_proj 20.5 / 13.1, M = 300 o_proj 23.1 / 15.8, down
// 42.4 / 38.8.
inline bool splitk_pays(int64_t m, int64_t n, int64_t k, int splits) {
  if (splits <= 1 || few_tokens(m, n)) return false;
  const double kb = (double)(k / 128), mib = (double)(splits * m * n) / (1 << 18);
  return tile_for(m, n).step * kb > 0.75 * kb / splits + 9.0 * mib / 16.0;
}

}  // namespace fp8rl
