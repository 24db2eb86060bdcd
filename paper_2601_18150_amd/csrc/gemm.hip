// Dense and grouped (MoE) blockwise-scaled FP8 GEMM kernels and launchers.
// The tile computation lives in gemm_core.hpp; this file maps workgroups to
// tiles.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "gemm_core.hpp"
#include "gemm_pipe.hpp"
#include "launch.hpp"

namespace fp8rl {
namespace {

// Tile configurations: BN x BM, waves along n and m, LDS ring depth.
//
// Dense products are one round or several of tiles over the 256 CUs, and a tile's
// time is its K blocks times a step time that hardly depends on the shape; so the
// tile is the one with the smallest (rounds x step time), tile_for() below.  Step
// times (us per 128-wide K block and round, Qwen3-8B linears, 80 .. 2000 tokens,
// weights from HBM; about 3 us per call besides):
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
using CfgLarge = GemmCfg<256, 256, 2, 4, 2>;   // 512 threads, wave tile 128(n) x 64(m), 130 KiB LDS
using CfgSmall = GemmCfg<128, 128, 2, 2, 2>;   // 256 threads, wave tile 64 x 64, 65 KiB LDS
using Cfg64x64 = GemmCfg<64, 64, 2, 2, 4>;     // two groups: 512 threads, wave tile 32 x 32, 130 KiB LDS
using Cfg64x128 = GemmCfg<64, 128, 2, 2, 3>;   // two groups: 512 threads, wave tile 32 x 64, 147 KiB LDS
using Cfg128x64 = GemmCfg<128, 64, 2, 2, 3>;   // two groups: 512 threads, wave tile 64 x 32, 146 KiB LDS
using Cfg128x128 = GemmCfg<128, 128, 2, 4, 4>; // 512 threads, wave tile 64 x 32, 130 KiB LDS
using Cfg128x256 = GemmCfg<128, 256, 2, 4, 3>; // 512 threads, wave tile 64 x 64, 147 KiB LDS
using Cfg256x128 = GemmCfg<256, 128, 4, 2, 3>; // 512 threads, wave tile 64 x 64, 146 KiB LDS
// Split-K ranges: one 128x128 tile per workgroup with eight waves (gemm_pipe; down, K =
// 12288, with its reduction: M = 256 29.9 us on four waves and a 3-slot ring of
// gemm_tiles, 29.0 now; M = 300 44.4, 36.5 now).
using CfgSplitK = Cfg128x128;
// The grouped GEMM: 128x128, two persistent workgroups per CU (gate_up of the expert
// block, 4096 tokens: 177 us; 256n x 128m 197, 128n x 64m 216, gemm_pipe with one
// workgroup per CU walking 256n x 128m / 128x128 tiles 196 / 212; down, K = 768: 108
// us, 256n x 128m 117, 128n x 64m 133).
using CfgGrouped = CfgSmall;

constexpr int kXcds = 8;        // MI355X: workgroup i is dispatched to XCD i % 8
constexpr int kGroupM = 8;      // m tiles per band of the grouped raster order

// Workgroup id -> output tile (encoded tile_n * tiles_m + tile_m).
// 1. Renumber so that the workgroups one XCD receives (ids x, x+8, x+16, ...)
//    walk one contiguous range of tile numbers.
// 2. Walk tile numbers in bands of kGroupM m tiles, m fastest: the tiles an XCD
//    runs at the same time share a few A row blocks and W row blocks, which
//    then stay in that XCD's L2.
// Renumber workgroup ids so that the ids one XCD receives (x, x+8, x+16, ...)
// map to one contiguous range of [0, total).
__device__ __forceinline__ int xcd_contiguous(int id, int total) {
  const int q = total / kXcds, r = total % kXcds;
  const int x = id % kXcds, j = id / kXcds;
  return x * q + min(x, r) + j;
}

__device__ __forceinline__ int band_tile(int t, int tiles_m, int tiles_n, int group_m = kGroupM) {
  const int band = t / (group_m * tiles_n);
  const int first_m = band * group_m;
  const int gm = min(tiles_m - first_m, group_m);
  const int in_band = t - band * group_m * tiles_n;
  const int tile_m = first_m + in_band % gm;
  const int tile_n = in_band / gm;
  return tile_n * tiles_m + tile_m;
}

__device__ __forceinline__ int xcd_grouped_tile(int id, int tiles_m, int tiles_n) {
  return band_tile(xcd_contiguous(id, tiles_m * tiles_n), tiles_m, tiles_n);
}

// The cross-tile pipeline (next tile's first load during this tile's last
// step) for the 128x128 tiles; the 256x256 tile has no registers to spare for
// the next tile's load plan and runs one tile per workgroup.
template <class C>
constexpr bool kCrossTiles = C::BN * C::BM <= 128 * 128;

// Job providers for gemm_tiles (see gemm_core.hpp): wave-uniform, no LDS
// writes, no synchronisation.

// Dense: a persistent grid; workgroup b runs tiles v = b, b + gridDim.x, ... of
// the renumbered order above (with gridDim.x a multiple of 8 every tile a
// workgroup runs is in its own XCD's range).
template <class C>
struct DenseJobs {
  int v, stride, tiles_m, tiles_n, M;
  __device__ bool next(TileJob& j) {
    if (v >= tiles_m * tiles_n) return false;
    const int tile = xcd_grouped_tile(v, tiles_m, tiles_n);
    v += stride;
    const int tile_m = tile % tiles_m;
    j.row_lo = tile_m * C::BM;
    j.m_valid = min(C::BM, M - j.row_lo);
    j.n0 = (tile / tiles_m) * C::BN;
    j.qw_off = 0;
    j.sw_off = 0;
    return true;
  }
};

// kMx: power-of-two scales through the MX-scaled MFMA (gemm_core.hpp).
template <class C, bool kMx>
__global__ __launch_bounds__(kMfmaBounds) void gemm_w8a8_block_kernel(
    const uint8_t* __restrict__ qa, int64_t lda, const float* __restrict__ sa, int64_t ld_sa,
    const uint8_t* __restrict__ qw, int64_t ldw, const float* __restrict__ sw,
    uint16_t* __restrict__ y, int64_t ldy, int64_t M, int64_t N, int KB, int tiles_m, int tiles_n) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[C::kLdsBytes];
  DenseJobs<C> jobs{(int)blockIdx.x, (int)gridDim.x, tiles_m, tiles_n, (int)M};
  gemm_tiles<C, kCrossTiles<C>, DenseJobs<C>, kMx>(qa, lda, sa, ld_sa, qw, ldw, sw, KB, y, ldy, (int)N, KB, jobs, lds);
}

// One tile per workgroup of C::kThreads * WK threads (gemm_pipe.hpp).
template <class C, int WK, bool kMx>
__global__ __launch_bounds__(kMfmaBounds) void gemm_w8a8_block_pipe_kernel(
    const uint8_t* __restrict__ qa, int64_t lda, const float* __restrict__ sa, int64_t ld_sa,
    const uint8_t* __restrict__ qw, int64_t ldw, const float* __restrict__ sw,
    uint16_t* __restrict__ y, int64_t ldy, int64_t M, int64_t N, int KB, int tiles_m, int tiles_n) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[kPipeLds<C, WK>];
  DenseJobs<C> jobs{(int)blockIdx.x, (int)gridDim.x, tiles_m, tiles_n, (int)M};
  gemm_pipe<C, WK, false, DenseJobs<C>, kMx>(qa, lda, sa, ld_sa, qw, ldw, sw, KB, y, ldy, nullptr, (int)N, KB, jobs,
                                            lds);
}

// Split-K dense GEMM, for shapes whose tiles alone cannot fill the GPU (decode:
// M = 256 gives 64-96 tiles of 128x128 for the narrow layers).  Workgroup v
// runs K range `split` of one tile and writes its fp32 sums to
// part[split][M][N]; splitk_reduce_kernel adds the ranges in order.  Ids are
// renumbered as in the dense kernel, split slowest, so the tiles an XCD runs
// together share their weight rows.
template <class C>
__global__ __launch_bounds__(kMfmaBounds) void gemm_w8a8_block_splitk_kernel(
    const uint8_t* __restrict__ qa, int64_t lda, const float* __restrict__ sa, int64_t ld_sa,
    const uint8_t* __restrict__ qw, int64_t ldw, const float* __restrict__ sw,
    float* __restrict__ part, int64_t M, int64_t N, int KB, int tiles_m, int tiles_n, int splits) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[C::kLdsBytes];
  const int total = tiles_m * tiles_n;
  const int v = xcd_contiguous(blockIdx.x, total * splits);
  const int split = v / total;
  const int tile = band_tile(v - split * total, tiles_m, tiles_n);
  const int tile_m = tile % tiles_m;
  const int kb0 = (int)(((int64_t)split * KB) / splits);
  const int kb1 = (int)(((int64_t)(split + 1) * KB) / splits);
  OneJob jobs;
  jobs.done = false;
  jobs.job.row_lo = tile_m * C::BM;
  jobs.job.m_valid = (int)min((int64_t)C::BM, M - jobs.job.row_lo);
  jobs.job.n0 = (tile / tiles_m) * C::BN;
  jobs.job.qw_off = (int64_t)kb0 * 128;
  jobs.job.sw_off = kb0;
  gemm_pipe<C, 1, true, OneJob, false>(qa + (int64_t)kb0 * 128, lda, sa + (int64_t)kb0 * ld_sa, ld_sa, qw, ldw, sw, KB,
                                       nullptr, 0, part + (int64_t)split * M * N, (int)N, kb1 - kb0, jobs, lds);
}

// y[m][n] = bf16_rne(part[0][m][n] + part[1][m][n] + ... ), eight n per thread.
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* __restrict__ part, int64_t M, int64_t N,
                                                            int splits, uint16_t* __restrict__ y, int64_t ldy) {
  const int64_t chunks = N / 8;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= M * chunks) return;
  const int64_t m = i / chunks;
  const int64_t c = i - m * chunks;
  const float* p = part + m * N + c * 8;
  float4 a = *reinterpret_cast<const float4*>(p);
  float4 b = *reinterpret_cast<const float4*>(p + 4);
  for (int s = 1; s < splits; ++s) {
    const float4 u = *reinterpret_cast<const float4*>(p + (int64_t)s * M * N);
    const float4 w = *reinterpret_cast<const float4*>(p + (int64_t)s * M * N + 4);
    a.x += u.x; a.y += u.y; a.z += u.z; a.w += u.w;
    b.x += w.x; b.y += w.y; b.z += w.z; b.w += w.w;
  }
  uint4 o;
  o.x = f32_to_bf16_rne(a.x) | (f32_to_bf16_rne(a.y) << 16);
  o.y = f32_to_bf16_rne(a.z) | (f32_to_bf16_rne(a.w) << 16);
  o.z = f32_to_bf16_rne(b.x) | (f32_to_bf16_rne(b.y) << 16);
  o.w = f32_to_bf16_rne(b.z) | (f32_to_bf16_rne(b.w) << 16);
  *reinterpret_cast<uint4*>(y + m * ldy + c * 8) = o;
}

// Grouped GEMM: m tiles are numbered over all experts in order (expert e owns
// ceil(rows_e / BM) consecutive m tiles, empty experts none).  Each workgroup
// first builds, in LDS, the first m tile and the first row of every expert
// from the device offsets (one prefix scan by wave 0), then runs tiles
// v = b, b + gridDim.x, ... of the (m tile, n tile) grid, renumbered so that
// each XCD walks a contiguous range in bands of kGroupMoe m tiles (m fastest
// inside a band): an XCD's concurrent tiles share their activation rows across
// the n tiles and, within an expert, its weight slab, both from its L2.
constexpr int kMaxExperts = 1024;          // table capacity (LDS: 8 KiB)
constexpr int kGroupMoe = 2;               // m tiles per band (measured: 2-4 best, 6-10% over m-fastest)

template <class C>
struct GroupedJobs {
  int v, stride, real_m, tiles_n, G;
  const int* tstart;                       // LDS [G+1]: first m tile of expert e
  const int* rstart;                       // LDS [G+1]: first row of expert e
  int64_t N, K;
  __device__ bool next(TileJob& j) {
    if (v >= real_m * tiles_n) return false;
    const int bt = band_tile(xcd_contiguous(v, real_m * tiles_n), real_m, tiles_n, kGroupMoe);
    v += stride;
    const int target = bt % real_m;
    const int tile_n = bt / real_m;
    // e = (number of experts whose first m tile is <= target) - 1: the last
    // such expert owns the tile (empty experts share their start with the next)
    const int lane = threadIdx.x & 63;
    int cnt = 0;
    for (int e0 = 0; e0 <= G; e0 += 64) {
      const int e = e0 + lane;
      const bool le = e <= G && tstart[e] <= target;
      const unsigned long long mask = __ballot(le);
      cnt += __popcll(mask);
      if (~mask) break;
    }
    // (the table entries are wave-uniform: keep them in scalar registers)
    const int e = __builtin_amdgcn_readfirstlane(cnt - 1);
    const int mt = target - __builtin_amdgcn_readfirstlane(tstart[e]);
    j.row_lo = __builtin_amdgcn_readfirstlane(rstart[e]) + mt * C::BM;
    j.m_valid = min(C::BM, __builtin_amdgcn_readfirstlane(rstart[e + 1]) - j.row_lo);
    j.n0 = tile_n * C::BN;
    j.qw_off = (int64_t)e * N * K;
    j.sw_off = (int64_t)e * (N / 128) * (K / 128);
    return true;
  }
};

// kGather: output row r takes its activation row from source row gidx[r] of qa
// ([src_rows][lda]) and sa ([K/128][ld_sa]); otherwise qa is [rows][K].
template <class C, bool kMx, bool kGather>
__global__ __launch_bounds__(kMfmaBounds) void grouped_gemm_w8a8_block_kernel(
    const uint8_t* __restrict__ qa, const float* __restrict__ sa, int64_t ld_sa,
    const uint8_t* __restrict__ qw, const float* __restrict__ sw,
    const int32_t* __restrict__ offsets, int G, uint16_t* __restrict__ y, int64_t N, int64_t K, int tiles_n,
    const int32_t* __restrict__ gidx, int src_rows, int64_t lda) {
  // one LDS object: the ring, then the two expert tables
  __shared__ __attribute__((aligned(16))) uint8_t lds[C::kLdsBytes + 2 * 4 * (kMaxExperts + 1)];
  int* tstart = reinterpret_cast<int*>(lds + C::kLdsBytes);
  int* rstart = tstart + (kMaxExperts + 1);
  const int t = threadIdx.x;
  if (t < 64) {
    // wave 0: exclusive prefix sum of the experts' m-tile counts, 64 at a time
    int base = 0;
    for (int e0 = 0; e0 <= G; e0 += 64) {
      const int e = e0 + t;
      int cnt = 0, r0 = 0;
      if (e <= G) r0 = offsets[e];
      if (e < G) cnt = (offsets[e + 1] - r0 + C::BM - 1) / C::BM;
      int incl = cnt;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const int u = __shfl_up(incl, d, 64);
        if (t >= d) incl += u;
      }
      if (e <= G) {
        tstart[e] = base + incl - cnt;
        rstart[e] = r0;
      }
      base += __shfl(incl, 63, 64);
    }
  }
  __syncthreads();
  GroupedJobs<C> jobs{(int)blockIdx.x, (int)gridDim.x, __builtin_amdgcn_readfirstlane(tstart[G]), tiles_n, G,
                      tstart, rstart, N, K};
  const int KB = (int)(K / 128);
  gemm_tiles<C, kCrossTiles<C>, GroupedJobs<C>, kMx, kGather>(qa, kGather ? lda : K, sa, ld_sa, qw, K, sw, KB, y, N,
                                                              (int)N, KB, jobs, lds, gidx, src_rows);
}

// Workgroups that stay resident on one CU for a configuration (LDS-limited).
template <class C, int kExtraLds = 0>
constexpr int per_cu() { return (160 * 1024) / (C::kLdsBytes + kExtraLds); }

constexpr int kCus = 256;     // MI355X; grids of kCus * per_cu() are multiples of 8 (one per XCD)

template <class C, bool kMx>
hipError_t launch_dense(const uint8_t* qa, int64_t lda, const float* sa, int64_t ld_sa, const uint8_t* qw,
                        int64_t ldw, const float* sw, uint16_t* y, int64_t ldy, int64_t m, int64_t n,
                        int64_t k, hipStream_t stream) {
  const int tiles_m = (int)((m + C::BM - 1) / C::BM);
  const int tiles_n = (int)((n + C::BN - 1) / C::BN);
  const int64_t total = (int64_t)tiles_m * tiles_n;
  // persistent grid with the cross-tile pipeline, else one workgroup per tile
  // (a persistent grid without it measured no faster)
  const int64_t slots = kCrossTiles<C> ? (int64_t)kCus * per_cu<C>() : total;
  hipLaunchKernelGGL((gemm_w8a8_block_kernel<C, kMx>), dim3((unsigned)(total < slots ? total : slots)),
                     dim3(C::kThreads), 0, stream, qa, lda, sa, ld_sa, qw, ldw, sw, y, ldy, m, n,
                     (int)(k / 128), tiles_m, tiles_n);
  return hipGetLastError();
}

template <class C, bool kMx, bool kGather = false>
hipError_t launch_grouped(const uint8_t* qa, const float* sa, int64_t ld_sa, const uint8_t* qw,
                          const float* sw, const int32_t* offsets, int64_t g, int64_t rows, uint16_t* y,
                          int64_t n, int64_t k, hipStream_t stream, const int32_t* gidx = nullptr,
                          int64_t src_rows = 0, int64_t lda = 0) {
  const int64_t max_tiles_m = rows / C::BM + g;        // upper bound on the real m tiles
  const int64_t tiles_n = (n + C::BN - 1) / C::BN;
  const int64_t total = max_tiles_m * tiles_n;
  static_assert(kCrossTiles<C>, "the grouped grid is persistent");
  const int64_t slots = (int64_t)kCus * per_cu<C, 2 * 4 * (kMaxExperts + 1)>();
  hipLaunchKernelGGL((grouped_gemm_w8a8_block_kernel<C, kMx, kGather>),
                     dim3((unsigned)(total < slots ? total : slots)), dim3(C::kThreads), 0, stream, qa, sa, ld_sa, qw,
                     sw, offsets, (int)g, y, n, k, (int)tiles_n, gidx, (int)src_rows, lda);
  return hipGetLastError();
}

}  // namespace

namespace {

// Dense tile configurations in the order that breaks ties.
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

// The smallest rounds x step time (figures at the configurations above).
TileChoice tile_for(int64_t m, int64_t n) {
  const int64_t pairs = ((m + 127) / 128) * (n / 128) / 512, rest = ((m + 127) / 128) * (n / 128) % 512;
  TileChoice best{Tile::kPersistent, 1.25 * (double)pairs + (rest == 0 ? 0.0 : rest <= 256 ? 0.9 : 1.25)};
  if (pairs > 0 && rest > 0 && rest <= 256) best.step -= 0.15;
  for (const TileCost& c : kTileCosts) {
    const int64_t tiles = ((m + c.bm - 1) / c.bm) * ((n + c.bn - 1) / c.bn);
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

ColumnSplit column_split(int64_t m, int64_t n, int64_t k) {
  const double kb = (double)(k / 128);
  const TileChoice whole = tile_for(m, n);
  const TileCost& c = kTileCosts[sizeof(kTileCosts) / sizeof(kTileCosts[0]) - 1];
  static_assert(kTileCosts[sizeof(kTileCosts) / sizeof(kTileCosts[0]) - 1].tile == Tile::k256x256, "the last entry");
  const int64_t tiles_m = (m + c.bm - 1) / c.bm;
  if (tiles_m <= kCus) {
    const int64_t per_round = kCus / tiles_m, rounds = n / c.bn / per_round, n1 = rounds * per_round * c.bn;
    if (rounds >= 1 && n1 < n) {
      const TileChoice rest = tile_for(m, n - n1);
      const double both = ((rounds == 1 ? c.one : c.more * (double)rounds) + rest.step) * kb + 3.0;
      if (both < 0.9 * whole.step * kb) return {n1, c.tile, rest.tile};
    }
  }
  return {0, c.tile, whole.tile};
}

template <class C, int WK, bool kMx>
hipError_t launch_pipe(const uint8_t* qa, int64_t lda, const float* sa, int64_t ld_sa, const uint8_t* qw, int64_t ldw,
                       const float* sw, uint16_t* y, int64_t ldy, int64_t m, int64_t n, int64_t k,
                       hipStream_t stream) {
  const int tiles_m = (int)((m + C::BM - 1) / C::BM);
  const int tiles_n = (int)((n + C::BN - 1) / C::BN);
  hipLaunchKernelGGL((gemm_w8a8_block_pipe_kernel<C, WK, kMx>), dim3((unsigned)((int64_t)tiles_m * tiles_n)),
                     dim3(C::kThreads * WK), 0, stream, qa, lda, sa, ld_sa, qw, ldw, sw, y, ldy, m, n, (int)(k / 128),
                     tiles_m, tiles_n);
  return hipGetLastError();
}

template <bool kMx>
hipError_t launch_tile(Tile tile, const uint8_t* qa, int64_t lda, const float* sa, int64_t ld_sa, const uint8_t* qw,
                       int64_t ldw, const float* sw, uint16_t* y, int64_t ldy, int64_t m, int64_t n, int64_t k,
                       hipStream_t stream) {
#define FP8RL_PIPE(C, WK) return launch_pipe<C, WK, kMx>(qa, lda, sa, ld_sa, qw, ldw, sw, y, ldy, m, n, k, stream)
  switch (tile) {
    case Tile::k64x64: FP8RL_PIPE(Cfg64x64, 2);
    case Tile::k64x128: FP8RL_PIPE(Cfg64x128, 2);
    case Tile::k128x64: FP8RL_PIPE(Cfg128x64, 2);
    case Tile::k128x128: FP8RL_PIPE(Cfg128x128, 1);
    case Tile::k128x256: FP8RL_PIPE(Cfg128x256, 1);
    case Tile::k256x128: FP8RL_PIPE(Cfg256x128, 1);
    case Tile::k256x256: return launch_dense<CfgLarge, kMx>(qa, lda, sa, ld_sa, qw, ldw, sw, y, ldy, m, n, k, stream);
    case Tile::kPersistent: break;
  }
#undef FP8RL_PIPE
  return launch_dense<CfgSmall, kMx>(qa, lda, sa, ld_sa, qw, ldw, sw, y, ldy, m, n, k, stream);
}

}  // namespace

hipError_t launch_gemm_w8a8_block(const uint8_t* qa, int64_t lda, const float* sa, int64_t ld_sa,
                                  const uint8_t* qw, int64_t ldw, const float* sw, uint16_t* y, int64_t ldy,
                                  int64_t m, int64_t n, int64_t k, hipStream_t stream, bool pow2_scales) {
  if (m <= kSmallTokens && n < kSmallMaxN)
    return launch_gemm_small(qa, lda, sa, ld_sa, qw, ldw, sw, y, ldy, m, n, k, stream, pow2_scales);
  const auto columns = [&](Tile tile, int64_t n0, int64_t cols) {
    const uint8_t* w = qw + n0 * ldw;
    const float* s = sw + n0 / 128 * (k / 128);
    return pow2_scales ? launch_tile<true>(tile, qa, lda, sa, ld_sa, w, ldw, s, y + n0, ldy, m, cols, k, stream)
                       : launch_tile<false>(tile, qa, lda, sa, ld_sa, w, ldw, s, y + n0, ldy, m, cols, k, stream);
  };
  const ColumnSplit c = column_split(m, n, k);
  if (c.n1 > 0) {
    const hipError_t e = columns(c.first, 0, c.n1);
    if (e != hipSuccess) return e;
  }
  return columns(c.rest, c.n1, n - c.n1);
}

// Decode batches (128 < M <= 256) whose 64x64 tiles number at most 512 (two per CU).
static bool decode_narrow_tiles(int64_t m, int64_t n) { return ((m + 63) / 64) * (n / 64) <= 512; }

int splitk_factor(int64_t m, int64_t n, int64_t k) {
  // Split K only when the 128x128 tiles cover less than half of MI355X's 256
  // CUs, into the largest power of two of ranges that keeps tiles x splits
  // within 256, each range at least 4 K blocks long.  (Measured on the decode
  // linears, M = 256: more ranges lose to the fp32 partial-sum traffic, which
  // grows with the split.)
  constexpr int64_t kCus = 256;
  if (m <= 0 || n <= 0 || k <= 0 || (m >= 2048 && n >= 2048)) return 1;
  // decode batches run unsplit on 64x64 tiles when K is short enough for one
  // workgroup's K loop (Qwen3-8B qkv, o_proj: K = 4096; down, K = 12288, splits)
  if (m > 128 && m <= 256 && k <= 4096 && decode_narrow_tiles(m, n)) return 1;
  const int64_t tiles = ((m + 127) / 128) * (n / 128);
  if (2 * tiles >= kCus) return 1;
  int64_t s = 1;
  while (2 * s * tiles <= kCus) s *= 2;
  const int64_t by_k = (k / 128) / 4;
  if (s > by_k) s = by_k;
  return s > 1 ? (int)s : 1;
}

hipError_t launch_gemm_w8a8_block_splitk(const uint8_t* qa, int64_t lda, const float* sa, int64_t ld_sa,
                                         const uint8_t* qw, int64_t ldw, const float* sw, uint16_t* y,
                                         int64_t ldy, int64_t m, int64_t n, int64_t k, float* part, int splits,
                                         hipStream_t stream) {
  // Few tokens need no K ranges across workgroups (measured at M = 64, down: 20.6 us
  // against 20.2 us split with its reduction; every other shape faster), and others
  // only where their ranges, the partial sums (16 MiB: 9 us) and the second launch beat
  // the unsplit tile.  Split / unsplit us: M = 128 down 22.9 / 34, M = 256 down 29.6 /
  // 34; M = 128 qkv 18.7 / 13.5, o_proj 20.5 / 13.1, M = 300 o_proj 23.1 / 15.8, down
  // 42.4 / 38.8.
  const double kb = (double)(k / 128), mib = (double)(splits * m * n) / (1 << 18);
  if ((m <= kSmallTokens && n < kSmallMaxN) || tile_for(m, n).step * kb <= 0.75 * kb / splits + 9.0 * mib / 16.0)
    return launch_gemm_w8a8_block(qa, lda, sa, ld_sa, qw, ldw, sw, y, ldy, m, n, k, stream, false);
  using C = CfgSplitK;
  const int tiles_m = (int)((m + C::BM - 1) / C::BM);
  const int tiles_n = (int)(n / C::BN);
  hipLaunchKernelGGL(gemm_w8a8_block_splitk_kernel<C>, dim3((unsigned)(tiles_m * tiles_n * splits)),
                     dim3(C::kThreads), 0, stream, qa, lda, sa, ld_sa, qw, ldw, sw, part, m, n, (int)(k / 128),
                     tiles_m, tiles_n, splits);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int64_t chunks = m * (n / 8);
  hipLaunchKernelGGL(splitk_reduce_kernel, dim3((unsigned)((chunks + 255) / 256)), dim3(256), 0, stream, part, m,
                     n, splits, y, ldy);
  return hipGetLastError();
}

// Split-K partial sums for callers that cannot allocate: a file-scope device
// array (each GPU the library runs on holds its own copy until the process
// ends).  In host code `scratch` only names the symbol; its device address on
// the current device comes from hipGetSymbolAddress, fetched once per device.
static __device__ __align__(256) float scratch[kSplitKScratchBytes / 4];

namespace {
constexpr int kMaxDevices = 64;
std::atomic<float*> scratch_ptr[kMaxDevices];
}  // namespace

hipError_t splitk_scratch(float** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  float* p = scratch_ptr[dev].load(std::memory_order_acquire);
  if (!p) {
    void* q = nullptr;
    e = hipGetSymbolAddress(&q, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    p = static_cast<float*>(q);
    scratch_ptr[dev].store(p, std::memory_order_release);   // racing first calls store the same address
  }
  *out = p;
  return hipSuccess;
}

hipError_t launch_grouped_gemm_w8a8_block(const uint8_t* qa, const float* sa, int64_t ld_sa,
                                          const uint8_t* qw, const float* sw, const int32_t* group_offsets,
                                          int64_t num_groups, int64_t total_rows, uint16_t* y, int64_t n,
                                          int64_t k, hipStream_t stream, bool pow2_scales) {
  if (total_rows <= kSmallRowsPerExpert * num_groups && n < kSmallMaxN)
    return launch_grouped_small(qa, k, sa, ld_sa, qw, sw, group_offsets, num_groups, total_rows, y, n, k, nullptr, 0,
                                stream, pow2_scales);
  if (pow2_scales)
    return launch_grouped<CfgGrouped, true>(qa, sa, ld_sa, qw, sw, group_offsets, num_groups, total_rows, y, n, k,
                                            stream);
  return launch_grouped<CfgGrouped, false>(qa, sa, ld_sa, qw, sw, group_offsets, num_groups, total_rows, y, n, k,
                                           stream);
}

hipError_t launch_grouped_gemm_w8a8_block_gathered(const uint8_t* qa, int64_t lda, const float* sa, int64_t ld_sa,
                                                   int64_t src_rows, const int32_t* row_index, const uint8_t* qw,
                                                   const float* sw, const int32_t* group_offsets, int64_t num_groups,
                                                   int64_t total_rows, uint16_t* y, int64_t n, int64_t k,
                                                   hipStream_t stream) {
  if (total_rows <= kSmallRowsPerExpert * num_groups && n < kSmallMaxN)
    return launch_grouped_small(qa, lda, sa, ld_sa, qw, sw, group_offsets, num_groups, total_rows, y, n, k, row_index,
                                src_rows, stream, false);
  return launch_grouped<CfgGrouped, false, true>(qa, sa, ld_sa, qw, sw, group_offsets, num_groups, total_rows, y,
                                                 n, k, stream, row_index, src_rows, lda);
}

}  // namespace fp8rl
