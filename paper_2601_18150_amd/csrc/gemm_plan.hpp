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
// tile is the one with the smallest (rounds x step time), above kShortK K blocks.  Step times (us per
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
enum class Tile { k64x64, k64x128, k128x64, k128x128, k128x256, k256x128, k256x256, kPersistent, k64x64Short };

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

// Up to four K blocks a step time says little: a call is its launch, the tiles' prologues
// and ends, and the output.  Three kernels are left there: 64x64 tiles of one wave group and
// a 3-slot ring, three workgroups per CU, which the two groups' sums would only hold up; the
// persistent 128x128; and 256x256.  Their times in us, with KB K blocks, R rounds of 256
// tiles and the padded output in millions of elements, fitted to 226 shapes of 65 .. 8192
// tokens and N = 128 .. 24576 (within 2 to 3% at the median); the choice is on average 0.4%
// from the fastest of all nine kernels, at most 13%.  By rounds x step time / now, us: 148 x
// 2688 x 384 4.4 / 4.1, 222 x 5504 x 384 6.0 / 5.1, 1076 x 3840 x 256 8.8 / 6.9, 1382 x 5248
// x 512 9.9 / 8.9, 6355 x 5248 x 128 25.0 / 17.0.
constexpr int64_t kShortK = 4;

inline Tile short_tile(int64_t m, int64_t n, int64_t kb) {
  const auto padded = [&](int64_t bm, int64_t bn) {
    return (double)((m + bm - 1) / bm * bm) * (double)((n + bn - 1) / bn * bn) / 1e6;
  };
  const auto rounds = [&](int64_t bm, int64_t bn) {
    return (double)((((m + bm - 1) / bm) * ((n + bn - 1) / bn) + kCus - 1) / kCus);
  };
  const double k = (double)kb;
  const double small = 2.7 + 0.35 * k + (rounds(64, 64) - 1) * 0.16 * k + 0.46 * padded(64, 64);
  const double large = 4.8 + 1.3 * k + (rounds(256, 256) - 1) * (2.4 + 1.6 * k) + 0.26 * padded(256, 256);
  const double halves = rounds(128, 128);          // (512 workgroups are resident)
  const double persistent = 3.6 + 0.7 * k + (halves > 1 ? 0.2 + 0.25 * k : 0.0) +
                            (halves > 2 ? (halves - 2) * (0.6 + 0.55 * k) : 0.0) + 0.18 * padded(128, 128);
  if (small < large && small < persistent && ((m + 63) / 64) * (n / 64) <= kMaxTiles) return Tile::k64x64Short;
  return large < persistent && ((m + 255) / 256) * ((n + 255) / 256) <= kMaxTiles ? Tile::k256x256 : Tile::kPersistent;
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
  if (k / 128 <= kShortK) return {0, Tile::k256x256, short_tile(m, n, k / 128)};
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

// K ranges of a split product, with room for which a caller may lend a workspace (1:
// never split): only where the 128x128 tiles cover less than half of the CUs, the
// largest power of two of ranges that keeps tiles x ranges within the CUs (more ranges
// lose to the fp32 partial sums), each at least 4 K blocks long.
inline int splitk_ranges(int64_t m, int64_t n, int64_t k) {
  if (m <= 0 || n <= 0 || k <= 0 || (m >= 2048 && n >= 2048)) return 1;
  // (short K on up to two 64x64 tiles per CU: never faster split)
  if (m > 128 && m <= 256 && k <= 4096 && ((m + 63) / 64) * (n / 64) <= 512) return 1;
  const int64_t tiles = ((m + 127) / 128) * (n / 128);
  if (2 * tiles >= kCus) return 1;
  int64_t s = 1;
  while (2 * s * tiles <= kCus) s *= 2;
  const int64_t by_k = (k / 128) / 4;
  if (s > by_k) s = by_k;
  return s > 1 ? (int)s : 1;
}

// Whether those ranges are run, given the room: a cost in us for each side, fitted to the
// layers below and others, 65 .. 800 tokens, and to 8 .. 64 tokens with K = 4096 .. 24576,
// weights from HBM.  Split: 7.8 for the two launches with the pipelines' start and end,
// 0.65 per K block of a range, 0.5 per MiB of partial sums written and read, 0.2 per range
// that the reduction adds, and no less than 11 beside the weights at 5.5 TB/s.  Unsplit: 3
// and the tile's step times, or for few tokens 2.5 and a step that grows with the tokens
// and rows (never up to 16 tokens, where eight waves split K already, nor up to K = 12288,
// where the two are within 1.8 us of each other).  Split / unsplit:
//   M            65           100          128          200          256          300
//   qkv       16.2 / 12.7  17.5 / 12.7  18.7 / 13.9
//   o_proj    15.7 / 11.9  18.1 / 12.5  21.0 / 13.3                            22.2 / 15.9
//   down      20.4 / 27.1  21.5 / 30.5  22.9 / 34.1  26.9 / 27.3  28.6 / 32.9  36.8 / 37.8
//   8192x4096 17.4 / 19.1  18.4 / 20.4  20.1 / 22.4  21.3 / 19.4  22.3 / 22.4  28.2 / 26.3
//   4096x1024 10.7 / 10.6  11.7 / 10.8  12.3 / 10.8                            15.1 / 10.9
//   12288x1024 18.1 / 25.2 19.8 / 28.7  21.9 / 32.3  21.2 / 25.6  22.9 / 30.6  20.0 / 29.6
//   M            16           32           40           64
//   down      18.8 / 14.3  18.5 / 15.9  18.9 / 18.4  19.8 / 21.1   (always unsplit)
//   16384x2048 17.5 / 12.8 17.0 / 15.9  17.5 / 19.4  18.1 / 21.9
//   24576x1024 20.8 / 17.9 20.2 / 23.4  21.3 / 28.5  22.0 / 33.4
// (K x N).  Where the rule takes the slower side it loses at most 1.7 us or 10%, but for 2.4
// and 3 us (6144x2560, M = 129; 9728x5120, M = 300) and, with 200 MB of weights, 6 (24576x8192,
// M = 48).
inline double split_cost(int64_t m, int64_t n, int64_t k, int splits) {
  const double kb = (double)(k / 128), mib = (double)((int64_t)splits * m * n) / (1 << 18);
  const double ranges = 7.8 + 0.65 * kb / splits + 0.5 * mib + 0.2 * splits;
  const double stream = 11.0 + (double)n * (double)k / 5.5e6;
  return ranges > stream ? ranges : stream;
}

inline bool splitk_pays(int64_t m, int64_t n, int64_t k, int splits) {
  const double kb = (double)(k / 128);
  if (splits <= 1) return false;
  if (few_tokens(m, n))
    return m > 16 && kb > 96 && 2.5 + kb * (0.045 + 0.0017 * (double)m + 1.2e-5 * (double)n) > split_cost(m, n, k, splits);
  return 3.0 + tile_for(m, n).step * kb > split_cost(m, n, k, splits);
}

}  // namespace fp8rl
