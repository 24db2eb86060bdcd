// Prints what the dense GEMM's plan (csrc/gemm_plan.hpp) chooses for each "m n k" of
// standard input: few-token kernel or not, columns of a first launch, its tile and the
// (other) tile, the workgroups of both, K ranges, whether they are run.
#include <cstdio>

#include "gemm_plan.hpp"

using namespace fp8rl;

static const char* name(Tile t) {
  switch (t) {
    case Tile::k64x64: return "64x64";
    case Tile::k64x128: return "64x128";
    case Tile::k128x64: return "128x64";
    case Tile::k128x128: return "128x128";
    case Tile::k128x256: return "128x256";
    case Tile::k256x128: return "256x128";
    case Tile::k256x256: return "256x256";
    case Tile::kPersistent: return "persistent";
    case Tile::k64x64Short: return "64x64-short";
  }
  return "?";
}

static long long workgroups(Tile t, int64_t m, int64_t n) {
  for (const TileCost& c : kTileCosts)
    if (c.tile == t || (c.tile == Tile::k64x64 && t == Tile::k64x64Short)) return tile_count(c, m, n);
  return 0;   // persistent: the resident ones
}

int main() {
  long long m, n, k;
  while (std::scanf("%lld %lld %lld", &m, &n, &k) == 3) {
    const ColumnSplit c = column_split(m, n, k);
    const int splits = splitk_ranges(m, n, k);
    std::printf("%d %lld %s %s %lld %lld %d %d\n", few_tokens(m, n) ? 1 : 0, (long long)c.n1,
                c.n1 ? name(c.first) : "-", name(c.rest), c.n1 ? workgroups(c.first, m, c.n1) : 0,
                workgroups(c.rest, m, n - c.n1), splits, splitk_pays(m, n, k, splits) ? 1 : 0);
  }
  return 0;
}
