// Dense and grouped (MoE) blockwise-scaled FP8 GEMM kernels and launchers.
// The tile computation lives in gemm_core.hpp; this file maps workgroups to
// tiles.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "gemm_core.hpp"
#include "gemm_pipe.hpp"
#include "gemm_plan.hpp"
#include "launch.hpp"

namespace fp8rl {
namespace {

// Tile configurations: BN x BM, waves along n and m, LDS ring depth.
//
// The dense tile is chosen by the plan's table of step times (gemm_plan.hpp).
using CfgLarge = GemmCfg<256, 256, 2, 4, 2>;   // 512 threads, wave tile 128(n) x 64(m), 130 KiB LDS
using CfgSmall = GemmCfg<128, 128, 2, 2, 2>;   // 256 threads, wave tile 64 x 64, 65 KiB LDS
using Cfg64x64 = GemmCfg<64, 64, 2, 2, 4>;     // two groups: 512 threads, wave tile 32 x 32, 130 KiB LDS
using Cfg64x64Short = GemmCfg<64, 64, 2, 2, 3>; // one group: 256 threads, wave tile 32 x 32, 50 KiB LDS
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

// Workgroups that stay resident on one CU for a configuration (LDS-limited); grids of
// kCus * per_cu() are multiples of 8 (one per XCD).
template <class C, int kExtraLds = 0>
constexpr int per_cu() { return (160 * 1024) / (C::kLdsBytes + kExtraLds); }

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
  static_assert(kCrossTiles<C> || C::kThreads <= kTileThreads, "the plan's grid limit");
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

template <class C, int WK, bool kMx>
hipError_t launch_pipe(const uint8_t* qa, int64_t lda, const float* sa, int64_t ld_sa, const uint8_t* qw, int64_t ldw,
                       const float* sw, uint16_t* y, int64_t ldy, int64_t m, int64_t n, int64_t k,
                       hipStream_t stream) {
  const int tiles_m = (int)((m + C::BM - 1) / C::BM);
  const int tiles_n = (int)((n + C::BN - 1) / C::BN);
  static_assert(C::kThreads * WK <= kTileThreads, "the plan's grid limit");
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
    case Tile::k64x64Short: FP8RL_PIPE(Cfg64x64Short, 1);
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
  if (few_tokens(m, n))
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

int splitk_factor(int64_t m, int64_t n, int64_t k) { return splitk_ranges(m, n, k); }

hipError_t launch_gemm_w8a8_block_splitk(const uint8_t* qa, int64_t lda, const float* sa, int64_t ld_sa,
                                         const uint8_t* qw, int64_t ldw, const float* sw, uint16_t* y,
                                         int64_t ldy, int64_t m, int64_t n, int64_t k, float* part, int splits,
                                         hipStream_t stream) {
  if (!splitk_pays(m, n, k, splits))
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
