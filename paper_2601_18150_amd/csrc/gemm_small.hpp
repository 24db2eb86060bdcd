// Blockwise-scaled FP8 GEMM for few tokens (decode batches, experts with a few
// rows): one pass over the weights, bound by the HBM stream of the weight codes,
// the matrix cores nearly idle.
//
// A wave owns 16 * TN weight rows and some of the K blocks, and streams its
// operands through a ring of D K blocks in LDS that no other wave touches: the
// K loop has no barrier, each wave waits for its own DMA only, and a slot is
// refilled as soon as its fragments are in registers.  (Fragments loaded straight
// from global memory need no LDS, but adjacent lanes then hold different rows:
// four cache lines per quad of lanes, 38 bytes per ns and CU from the L2 where whole
// 128-byte lines, eight lanes a row as the DMA reads them, reach 130.)
// The WK waves of a workgroup split the K blocks of the same rows (wave w takes
// blocks w, w + WK, ...: together they read whole runs of each weight row) and
// add their fp32 sums through LDS in a fixed order, so that even a narrow layer
// puts a thousand waves on the weight stream.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.hpp"
#include "gemm_core.hpp"

namespace fp8rl {

template <int AO_, int TN_, int D_, int WK_, int WAVES_>
struct SmallCfg {
  static constexpr int AO = AO_;               // activation octets: 8 * AO tokens
  static constexpr int TM = (AO_ + 1) / 2;     // 16-token sub-tiles (AO = 1: half of one, its rows twice)
  static constexpr int TN = TN_;               // 16-row weight sub-tiles per wave
  static constexpr int D = D_;                 // ring depth in K blocks
  static constexpr int WK = WK_;               // waves that split the K blocks
  static constexpr int kWaves = WAVES_;
  static constexpr int kThreads = 64 * WAVES_;
  static constexpr int WN = WAVES_ / WK_;      // waves along n
  static constexpr int kRows = 16 * TN_ * WN;  // weight rows per workgroup
  static constexpr int kOctets = 2 * TN_ + AO_;
  static constexpr int kPer = kOctets + 1;     // DMA instructions per K block (one for the scales)
  static constexpr int kSlot = kOctets * 1024 + 256;
  static constexpr int kRing = D_ * kSlot;     // per wave
  static constexpr int kRed = WK_ > 1 ? WAVES_ * TN_ * TM * 1024 : 0;
  static constexpr int kLds = WAVES_ * kRing > kRed ? WAVES_ * kRing : kRed;
  static_assert(AO_ == 1 || AO_ % 2 == 0, "whole sub-tiles");
  static_assert(AO_ <= 8, "one scale DMA instruction covers 64 tokens");
  static_assert(WAVES_ % WK_ == 0 && 128 % kRows == 0, "a workgroup's rows sit inside one 128-row scale block");
  static_assert(kLds <= 160 * 1024 && (D_ - 1) * kPer < 64, "LDS is 160 KiB, vmcnt 6 bits");
};

// kRows weight rows from wbase (swrow: their block's scales per K block) times
// `m` tokens: this lane moves row arow[o] (a byte offset from qa) of activation
// octet o and the scale of token srow (an index into each row of sa); output
// row i at y + i * ldy.
template <class C, bool kMx>
__device__ __forceinline__ void small_tile(const uint8_t* __restrict__ wbase, uint32_t ldw,
                                           const float* __restrict__ swrow, const uint8_t* __restrict__ qa,
                                           const uint32_t (&arow)[C::AO], const float* __restrict__ sa, int64_t ld_sa,
                                           uint32_t srow, uint16_t* __restrict__ y, int64_t ldy, int m, int KB,
                                           uint8_t* lds) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wk = wave % C::WK, wn = wave / C::WK;
  const int frow = lane & 15, fg = lane >> 4;
  const __amdgpu_buffer_rsrc_t rw = buffer_rsrc(wbase + (int64_t)wn * (16 * C::TN) * ldw), ra = buffer_rsrc(qa);
  uint8_t* ring = lds + wave * C::kRing;
  // DMA: lane L of an octet's instruction moves physical chunk L & 7 of its row L >> 3
  const int lrow = lane >> 3;
  uint32_t goff[C::kOctets];
#pragma unroll
  for (int o = 0; o < C::kOctets; ++o) {
    const int r = (o < 2 * C::TN ? o : o - 2 * C::TN) * 8 + lrow;
    const uint32_t c = (uint32_t)(((lane & 7) ^ swz_key(r)) * 16);
    goff[o] = c + (o < 2 * C::TN ? (uint32_t)r * ldw : arow[o < 2 * C::TN ? 0 : o - 2 * C::TN]);
  }
  // fragments: chunks 2 fg, 2 fg + 1 of row frow of a sub-tile
  const int f0 = swz(frow, 2 * fg), f1 = swz(frow, 2 * fg + 1);
  const int a0 = C::AO == 1 ? swz(frow & 7, 2 * fg) : f0, a1 = C::AO == 1 ? swz(frow & 7, 2 * fg + 1) : f1;

  const int nb = (KB - wk + C::WK - 1) / C::WK;          // this wave's K blocks: wk, wk + WK, ...
  auto fetch = [&](int i, int slot) {
    const int kb = wk + i * C::WK;
    uint8_t* dst = ring + slot * C::kSlot;
#pragma unroll
    for (int o = 0; o < C::kOctets; ++o)
      lds_dma16(o < 2 * C::TN ? rw : ra, goff[o], (uint32_t)kb * 128u, dst + o * 1024);
    lds_dma4(sa + (int64_t)kb * ld_sa + srow, dst + C::kOctets * 1024);
  };

  v4f32 acc[C::TN][C::TM];
#pragma unroll
  for (int tn = 0; tn < C::TN; ++tn)
#pragma unroll
    for (int tm = 0; tm < C::TM; ++tm) acc[tn][tm] = (v4f32){0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int d = 0; d < C::D; ++d)
    if (d < nb) fetch(d, d);
  int slot = 0;
  for (int i = 0; i < nb; ++i) {
    const float swv = swrow[wk + i * C::WK];
    wait_own_ring<C::kPer, C::D>(nb - 1 - i);
    asm volatile("" ::: "memory");
    const uint8_t* st = ring + slot * C::kSlot;
    const uint8_t* sta = st + 2 * C::TN * 1024;
    const float* sts = reinterpret_cast<const float*>(st + C::kOctets * 1024);
    v8i32 w[C::TN], a[C::TM];
    float sc[C::TM];
#pragma unroll
    for (int tn = 0; tn < C::TN; ++tn) w[tn] = lds_frag2(st + tn * 2048, f0, f1);
#pragma unroll
    for (int tm = 0; tm < C::TM; ++tm) {
      a[tm] = lds_frag2(sta + tm * 2048, a0, a1);
      sc[tm] = sts[tm * 16 + frow];
    }
    // the slot's fragments are in registers before its refill is issued
    __builtin_amdgcn_s_waitcnt(0xF | (0x7 << 4) | (0x3 << 14));   // lgkmcnt(0)
    asm volatile("" ::: "memory");
    if (i + C::D < nb) fetch(i + C::D, slot);
    slot = slot + 1 == C::D ? 0 : slot + 1;
#pragma unroll
    for (int tm = 0; tm < C::TM; ++tm)
#pragma unroll
      for (int tn = 0; tn < C::TN; ++tn) {
        if constexpr (kMx) {
          acc[tn][tm] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
              w[tn], a[tm], acc[tn][tm], 0, 0, 0, (int)(__float_as_uint(swv) >> 23), 0,
              (int)(__float_as_uint(sc[tm]) >> 23));
        } else {
          const v4f32 p = mfma_fp8_16x16x128(w[tn], a[tm]);
          const float s = sc[tm] * swv;
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[tn][tm][r] = __builtin_fmaf(p[r], s, acc[tn][tm][r]);
        }
      }
  }

  // lane: four consecutive n (4 fg ..) of token frow of each sub-tile
  auto store = [&](const v4f32& v, int tn, int tm) {
    const int t = tm * 16 + frow;
    if (t < m) {
      uint2 o;
      o.x = f32_to_bf16_rne(v[0]) | (f32_to_bf16_rne(v[1]) << 16);
      o.y = f32_to_bf16_rne(v[2]) | (f32_to_bf16_rne(v[3]) << 16);
      *reinterpret_cast<uint2*>(y + (int64_t)t * ldy + (wn * C::TN + tn) * 16 + 4 * fg) = o;
    }
  };
  if constexpr (C::WK == 1) {
#pragma unroll
    for (int tn = 0; tn < C::TN; ++tn)
#pragma unroll
      for (int tm = 0; tm < C::TM; ++tm) store(acc[tn][tm], tn, tm);
  } else {
    constexpr int kSub = C::TN * C::TM;
    v4f32* red = reinterpret_cast<v4f32*>(lds);
    __syncthreads();                                     // every wave's ring is idle (its last DMA was waited for)
#pragma unroll
    for (int tn = 0; tn < C::TN; ++tn)
#pragma unroll
      for (int tm = 0; tm < C::TM; ++tm) red[(wave * kSub + tn * C::TM + tm) * 64 + lane] = acc[tn][tm];
    __syncthreads();
    // sub-tile s of these rows is added up by wave s % WK of the WK that share them
#pragma unroll
    for (int s0 = 0; s0 < kSub; s0 += C::WK) {
      const int s = s0 + wk;
      if (s < kSub) {
        v4f32 v = red[((wn * C::WK) * kSub + s) * 64 + lane];
#pragma unroll
        for (int k = 1; k < C::WK; ++k) v += red[((wn * C::WK + k) * kSub + s) * 64 + lane];
        store(v, s / C::TM, s % C::TM);
      }
    }
  }
}

// Dense, m <= 8 * AO: workgroup b owns weight rows b * kRows ..
template <class C, bool kMx>
__global__ __launch_bounds__(kMfmaBounds) void gemm_small_kernel(
    const uint8_t* __restrict__ qa, int64_t lda, const float* __restrict__ sa, int64_t ld_sa,
    const uint8_t* __restrict__ qw, int64_t ldw, const float* __restrict__ sw, uint16_t* __restrict__ y, int64_t ldy,
    int m, int KB) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[C::kLds];
  const int n0 = blockIdx.x * C::kRows;
  const int lane = threadIdx.x & 63;
  uint32_t arow[C::AO];                          // rows past the end re-read the last
#pragma unroll
  for (int o = 0; o < C::AO; ++o) arow[o] = (uint32_t)min(o * 8 + (lane >> 3), m - 1) * (uint32_t)lda;
  small_tile<C, kMx>(qw + (int64_t)n0 * ldw, (uint32_t)ldw, sw + (int64_t)(n0 >> 7) * KB, qa, arow, sa, ld_sa,
                     (uint32_t)min(lane, m - 1), y + n0, ldy, m, KB, lds);
}

// Grouped, for experts with a few rows each on average.  An expert's rows are cut into
// chunks: of 32 rows, each with the narrowest of three tiles that holds it (their rings
// take about the same LDS); past kWideFrom rows of 128, on a 64x128 tile of the common K
// loop in the same LDS, because every chunk streams the expert's weights again.
// Workgroup (x, `extra` + e) owns weight rows x * kRows .. of expert e's first chunk (an
// expert without rows costs one scalar load); the further chunks of popular experts are
// numbered over all experts in order and workgroup (x, c < extra) takes number c, so
// that they run side by side, first, and are no serial chain however the rows fall.
template <int WK>
struct GroupedSmall {
  using R8 = SmallCfg<1, 1, 4, WK, 4>;
  using R16 = SmallCfg<2, 1, 3, WK, 4>;
  using R32 = SmallCfg<4, 1, 2, WK, 4>;
  using Wide = GemmCfg<64, 128, 2, 2, 2>;
  static constexpr int kRows = R8::kRows;
  static constexpr int kMaxOf(int a, int b) { return a > b ? a : b; }
  static constexpr int kLds = kMaxOf(kMaxOf(R8::kLds, Wide::kLdsBytes), kMaxOf(R16::kLds, R32::kLds));
  static_assert(R8::kThreads == 256 && Wide::kThreads == 256 && Wide::BN % kRows == 0, "one workgroup for all");
};
constexpr int kChunkRows = 32;
// (one expert alone, gate_up: of 128 rows four chunks of 32 take 10.6 us, one wide chunk
// 12.5; of 256 rows 19.9 and 18.9.  Beside others a wide chunk is a long chain: expert
// block, 190 tokens x 8 by Zipf's law with up to 190 rows in an expert, 126.5 us with wide
// chunks there, 124.2 without)
constexpr int kWideFrom = 256;
constexpr int kWideRows = 128;

// The rows of a chunk: r0 .. r1 - 1, of expert e.
struct RowChunk {
  int e, r0, r1;
};

__device__ __forceinline__ int chunk_size(int rows) { return rows > kWideFrom ? kWideRows : kChunkRows; }

// Chunk number c of those behind each expert's first, false past the last (uniform over
// the workgroup of four waves).  Four experts a lane and one prefix sum for 256 experts:
// up to that many, every wave looks for itself; more of them (at most 1024) are shared by
// the four waves.
constexpr int kFindLds = 8 * 4;
__device__ __forceinline__ bool find_chunk(const int32_t* __restrict__ offsets, int G, int c, int* lds, RowChunk& out) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool shared = G > 256;
  const int e = (shared ? 256 * wave : 0) + 4 * lane;
  int o[5], n[4];
#pragma unroll
  for (int i = 0; i < 5; ++i) o[i] = offsets[min(e + i, G)];
#pragma unroll
  for (int i = 0; i < 4; ++i) n[i] = max(o[i + 1] - o[i] - 1, 0) / chunk_size(o[i + 1] - o[i]);
  const int mine = n[0] + n[1] + n[2] + n[3];
  int upto = wave_inclusive_sum(mine);
  if (shared) {
    if (lane == 63) lds[wave] = upto;
    __syncthreads();
    int before = 0;
    for (int w = 0; w < 4; ++w) {
      const int t = __builtin_amdgcn_readfirstlane(lds[w]);
      if (w < wave) before += t;
    }
    upto += before;
  }
  const unsigned long long has = __ballot(upto > c && upto - mine <= c);   // the lane whose four experts hold it
  if (has) {
    const int l = __builtin_ctzll(has);
    int at = c - (upto - mine), i = 0;           // (meaningful in lane l only)
#pragma unroll
    for (int k = 0; k < 3; ++k)
      if (i == k && at >= n[k]) {
        at -= n[k];
        i = k + 1;
      }
    const int lo = i == 0 ? o[0] : i == 1 ? o[1] : i == 2 ? o[2] : o[3];
    const int hi = i == 0 ? o[1] : i == 1 ? o[2] : i == 2 ? o[3] : o[4];
    const int size = chunk_size(hi - lo);
    out.e = __builtin_amdgcn_readlane(e + i, l);
    out.r0 = __builtin_amdgcn_readlane(lo + (at + 1) * size, l);
    out.r1 = __builtin_amdgcn_readlane(min(hi, lo + (at + 2) * size), l);
  }
  if (!shared) return has != 0;
  if (has && lane == 0) {
    lds[4] = out.e;
    lds[5] = out.r0;
    lds[6] = out.r1;
  }
  const int total = __builtin_amdgcn_readfirstlane(lds[0]) + __builtin_amdgcn_readfirstlane(lds[1]) +
                    __builtin_amdgcn_readfirstlane(lds[2]) + __builtin_amdgcn_readfirstlane(lds[3]);
  if (c >= total) return false;
  __syncthreads();
  out.e = __builtin_amdgcn_readfirstlane(lds[4]);
  out.r0 = __builtin_amdgcn_readfirstlane(lds[5]);
  out.r1 = __builtin_amdgcn_readfirstlane(lds[6]);
  return true;
}

template <int WK, bool kMx, bool kGather>
__global__ __launch_bounds__(kMfmaBounds) void grouped_gemm_small_kernel(
    const uint8_t* __restrict__ qa, int64_t lda, const float* __restrict__ sa, int64_t ld_sa,
    const uint8_t* __restrict__ qw, const float* __restrict__ sw, const int32_t* __restrict__ offsets, int G,
    int extra, uint16_t* __restrict__ y, int64_t N, int64_t K, const int32_t* __restrict__ gidx, int src_rows) {
  using S = GroupedSmall<WK>;
  __shared__ __attribute__((aligned(16))) uint8_t lds[S::kLds + kFindLds];
  RowChunk rc;
  if ((int)blockIdx.y < extra) {
    if (!find_chunk(offsets, G, (int)blockIdx.y, reinterpret_cast<int*>(lds + S::kLds), rc)) return;
  } else {
    rc.e = (int)blockIdx.y - extra;
    rc.r0 = offsets[rc.e];
    rc.r1 = offsets[rc.e + 1];
    if (rc.r0 >= rc.r1) return;
    rc.r1 = min(rc.r1, rc.r0 + chunk_size(rc.r1 - rc.r0));
  }
  const int n0 = blockIdx.x * S::kRows;
  const int KB = (int)(K / 128);
  const int m = rc.r1 - rc.r0;
  const int64_t qw_off = (int64_t)rc.e * N * K, sw_off = (int64_t)rc.e * (N / 128) * KB;
  if (m > kChunkRows) {
    if (n0 % S::Wide::BN) return;                  // (its neighbour's tile covers these weight rows)
    OneJob jobs{TileJob{rc.r0, m, n0, qw_off, sw_off}, false};
    gemm_tiles<typename S::Wide, true, OneJob, kMx, kGather>(qa, lda, sa, ld_sa, qw, K, sw, KB, y, N, (int)N, KB, jobs,
                                                             lds, gidx, src_rows);
    return;
  }
  auto chunk = [&](auto cfg) {
    using C = decltype(cfg);
    const int lane = threadIdx.x & 63;
    uint32_t arow[C::AO];                        // rows past the end re-read the last
#pragma unroll
    for (int o = 0; o < C::AO; ++o) {
      const int i = min(o * 8 + (lane >> 3), m - 1);
      arow[o] = (uint32_t)(kGather ? min(max(gidx[rc.r0 + i], 0), src_rows - 1) : i) * (uint32_t)lda;
    }
    const int i = min(lane, m - 1);
    const uint32_t srow = (uint32_t)(kGather ? min(max(gidx[rc.r0 + i], 0), src_rows - 1) : i);
    small_tile<C, kMx>(qw + qw_off + (int64_t)n0 * K, (uint32_t)K, sw + sw_off + (int64_t)(n0 >> 7) * KB,
                       kGather ? qa : qa + (int64_t)rc.r0 * lda, arow, kGather ? sa : sa + rc.r0, ld_sa, srow,
                       y + (int64_t)rc.r0 * N + n0, N, m, KB, lds);
  };
  if (m <= 8) chunk(typename S::R8{});
  else if (m <= 16) chunk(typename S::R16{});
  else chunk(typename S::R32{});
}

}  // namespace fp8rl
