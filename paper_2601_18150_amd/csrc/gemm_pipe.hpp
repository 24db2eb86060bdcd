// One output tile per workgroup of the blockwise-scaled FP8 GEMM, with a fragment
// pipeline, for wave tiles of at most 64 x 64 (the same product, operand layout and
// scale application as gemm_core.hpp's gemm_tiles, whose 128 x 64 wave tile has no
// registers for it).
//
// A K step of a small wave tile is a chain of latencies: barrier, LDS reads,
// MFMA, scale FMA.  Here a wave reads the fragments of step s + 1 while it
// multiplies those of step s: activation fragments into a second register set, each
// weight fragment over the one whose MFMAs have just been issued (a second set of
// those too would spill at 64 x 64).  So the LDS latency runs under the MFMAs; and
// since every wave holds its fragments of step s when that step begins, its slot is
// refilled with step s + S, a step earlier than a ring that is read while it is
// multiplied.
//   step s: wait for this wave's DMA of step s + 1; barrier (everyone's DMA of
//           step s + 1 landed, everyone's reads of step s are in registers);
//           DMA of s + S into the slot of s; multiply s and read s + 1.
// WK groups of waves may split the K blocks of one tile (group g takes blocks g,
// g + WK, ...), each with a ring of its own, so that a small tile has two waves per
// SIMD; their sums are added in LDS in order.
// What is left is mostly the DMA with weights from HBM, alone (no MFMA) 40 to 47 bytes
// per ns and busy CU: 12.6 of the 13.9 us of a 64x64 call (M = 256, o_proj), 16.8 of 19.6
// (64x128, qkv), 39.9 of 45.5 (128x256, gate_up); on 128x128 tiles (M = 777, o_proj) 17.6
// of 26.2, and the loop without DMA takes 20.2.
#pragma once

#include "gemm_core.hpp"

namespace fp8rl {

template <class C, int WK>
constexpr int kPipeLds = WK * C::kLdsBytes;

// kPartial: the fp32 sums of a K range to part (rows of N floats) instead of bf16 to y.
template <class C, int WK, bool kPartial, class Jobs, bool kMx>
__device__ __forceinline__ void gemm_pipe(const uint8_t* __restrict__ qa, int64_t lda, const float* __restrict__ sa,
                                          int64_t ld_sa, const uint8_t* __restrict__ qw, int64_t ldw,
                                          const float* __restrict__ sw, int sw_ld, uint16_t* __restrict__ y,
                                          int64_t ldy, float* __restrict__ part, int N, int KB, Jobs& jobs,
                                          uint8_t* lds) {
  constexpr int S = C::STAGES;
  static_assert(C::WTN <= 64 && C::WTM <= 64, "two fragment sets fit the registers");
  constexpr int kPer = C::kLoadsPerWave;
  const int t = threadIdx.x;
  const int lane = t & 63;
  const int gwave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int grp = WK > 1 ? gwave / C::kWaves : 0;
  const int wave = WK > 1 ? gwave % C::kWaves : gwave;
  const int wn = wave % C::WN, wm = wave / C::WN;
  const int frow = lane & 15, fg = lane >> 4;
  const int f0 = swz(frow, 2 * fg), f1 = swz(frow, 2 * fg + 1);
  uint8_t* ring = lds + grp * C::kLdsBytes;
  const int lrow = lane >> 3;
  const int swave = wave % C::kScaleLoads;                 // (every wave moves scales, some of them twice: one wait count)
  const int steps = (KB + WK - 1) / WK;                    // of the longest group
  const int mine = (KB - grp + WK - 1) / WK;               // of this one

  TileJob job;
  if (!jobs.next(job)) return;
  const int n_valid = min(C::BN, N - job.n0);
  // DMA plan as in gemm_tiles: wave w moves row octets w, w + kWaves, ...
  uint32_t goff[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int o = wave + i * C::kWaves;
    const bool w = o < C::BN / 8;
    const int r = (w ? o : o - C::BN / 8) * 8 + lrow;
    const int c = ((lane & 7) ^ swz_key(r)) * 16;
    goff[i] = w ? (uint32_t)(min(r, n_valid - 1) * ldw + c) : (uint32_t)(min(r, job.m_valid - 1) * lda + c);
  }
  const __amdgpu_buffer_rsrc_t rw = buffer_rsrc(qw + job.qw_off + (int64_t)job.n0 * ldw);
  const __amdgpu_buffer_rsrc_t ra = buffer_rsrc(qa + (int64_t)job.row_lo * lda);
  const float* sa_lane = sa + job.row_lo + min(swave * 64 + lane, job.m_valid - 1);
  auto fetch = [&](int s, int slot) {
    const int kb = s * WK + grp;
    uint8_t* dst = ring + slot * C::kStageBytes;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int o = wave + i * C::kWaves;
      lds_dma16(o < C::BN / 8 ? rw : ra, goff[i], (uint32_t)kb * 128u, dst + o * 1024);
    }
    lds_dma4(sa_lane + (int64_t)kb * ld_sa, dst + C::kWBytes + C::kABytes + swave * 256);
  };
  auto wait = [&](int later) { wait_own_ring<kPer + 1, S>(later); };

  // one step's activation fragments and scales (two sets); the weight fragments are
  // replaced row by row, each right behind the MFMAs that read it
  struct Acts {
    v8i32 a[C::TM];
    float sa[C::TM], sw;
  };
  auto slot_w = [&](int slot) { return ring + slot * C::kStageBytes + wn * C::WTN * 128; };
  auto slot_a = [&](int slot) { return ring + slot * C::kStageBytes + C::kWBytes + wm * C::WTM * 128; };
  auto read_scales = [&](Acts& f, int slot, const float* swrow, int kb) {
    const float* sts = reinterpret_cast<const float*>(ring + slot * C::kStageBytes + C::kWBytes + C::kABytes) +
                       wm * C::WTM + frow;
    f.sw = swrow[kb];
#pragma unroll
    for (int tm = 0; tm < C::TM; ++tm) f.sa[tm] = sts[tm * 16];
  };

  // (a wave past N reads the last block and stores nothing)
  const float* swrow = sw + job.sw_off + (int64_t)(min(job.n0 + wn * C::WTN, N - 1) >> 7) * sw_ld;

#pragma unroll
  for (int p = 0; p < S; ++p)
    if (p < mine) fetch(p, p);
  Acts f_a, f_b;
  v8i32 w[C::TN];
  wait(min(S, mine) - 1);
  lds_barrier();
  read_scales(f_a, 0, swrow, min(grp, KB - 1));
#pragma unroll
  for (int tm = 0; tm < C::TM; ++tm) f_a.a[tm] = lds_frag2(slot_a(0) + tm * 2048, f0, f1);
#pragma unroll
  for (int tn = 0; tn < C::TN; ++tn) w[tn] = lds_frag2(slot_w(0) + tn * 2048, f0, f1);

  int slot = 0;
  v4f32 acc[C::TN][C::TM];
#pragma unroll
  for (int i = 0; i < C::TN; ++i)
#pragma unroll
    for (int j = 0; j < C::TM; ++j) acc[i][j] = (v4f32){0.f, 0.f, 0.f, 0.f};

  auto step = [&](int s, Acts& now, Acts& then) {
    const int nslot = slot + 1 == S ? 0 : slot + 1;
    if (s + 1 < mine) wait(min(S - 2, mine - 2 - s));
    lds_barrier();
    // (past the end the next fragments are stale bytes of the ring, never multiplied)
    read_scales(then, nslot, swrow, min((s + 1) * WK + grp, KB - 1));
    if (s + S < mine) fetch(s + S, slot);
    slot = nslot;
    if (WK > 1 && s >= mine) return;
    const uint8_t* nw = slot_w(nslot);
    const uint8_t* na = slot_a(nslot);
    float sc[C::TM];
#pragma unroll
    for (int tm = 0; tm < C::TM; ++tm) sc[tm] = now.sa[tm] * now.sw;
#pragma unroll
    for (int tn = 0; tn < C::TN; ++tn) {
      v4f32 p[C::TM];
#pragma unroll
      for (int tm = 0; tm < C::TM; ++tm) {
        if constexpr (kMx)
          acc[tn][tm] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
              w[tn], now.a[tm], acc[tn][tm], 0, 0, 0, (int)(__float_as_uint(now.sw) >> 23), 0,
              (int)(__float_as_uint(now.sa[tm]) >> 23));
        else
          p[tm] = mfma_fp8_16x16x128(w[tn], now.a[tm]);
      }
      w[tn] = lds_frag2(nw + tn * 2048, f0, f1);
#pragma unroll
      for (int tm = tn; tm < C::TM; tm += C::TN) then.a[tm] = lds_frag2(na + tm * 2048, f0, f1);
      if constexpr (!kMx) {
#pragma unroll
        for (int tm = 0; tm < C::TM; ++tm)
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[tn][tm][r] = __builtin_fmaf(p[tm][r], sc[tm], acc[tn][tm][r]);
      }
      // (rows of MFMA results do not pile up: there are no registers for them)
      if (C::TN * C::TM >= 16) __builtin_amdgcn_sched_barrier(0);
    }
  };
  int s = 0;
  for (; s + 1 < steps; s += 2) {
    step(s, f_a, f_b);
    step(s + 1, f_b, f_a);
  }
  if (s < steps) step(s, f_a, f_b);

  // ---- the rings are idle (every fetch was waited for)
  if constexpr (WK > 1) {
    constexpr int kSub = C::TN * C::TM;
    static_assert(kSub * C::kWaves * 1024 <= C::kLdsBytes, "a group's sums fit its ring");
    lds_barrier();
    if (grp > 0) {
      v4f32* red = reinterpret_cast<v4f32*>(ring);
#pragma unroll
      for (int i = 0; i < kSub; ++i) red[(i * C::kWaves + wave) * 64 + lane] = acc[i / C::TM][i % C::TM];
    }
    lds_barrier();
    if (grp == 0) {
#pragma unroll
      for (int g = 1; g < WK; ++g) {
        const v4f32* red = reinterpret_cast<const v4f32*>(lds + g * C::kLdsBytes);
#pragma unroll
        for (int i = 0; i < kSub; ++i) acc[i / C::TM][i % C::TM] += red[(i * C::kWaves + wave) * 64 + lane];
      }
    }
  }
  if constexpr (kPartial) {
    static_assert(WK == 1, "the groups' sums are not split further");
#pragma unroll
    for (int tn = 0; tn < C::TN; ++tn) {
      const int nl = wn * C::WTN + tn * 16 + 4 * fg;
#pragma unroll
      for (int tm = 0; tm < C::TM; ++tm) {
        const int ml = wm * C::WTM + tm * 16 + frow;
        if (ml < job.m_valid && nl < n_valid)
          *reinterpret_cast<v4f32*>(part + (int64_t)(job.row_lo + ml) * N + job.n0 + nl) = acc[tn][tm];
      }
    }
    return;
  }
  // bf16 through LDS, whole 16-byte chunks of output rows with streaming stores
  // (layout as in gemm_tiles)
  constexpr int kRowBytes = C::BN * 2;
  constexpr int kChunks = kRowBytes / 16;
  constexpr int kRowsFit = C::kLdsBytes / kRowBytes;
  constexpr int kRows = kRowsFit >= C::BM ? C::BM : (kRowsFit / C::WTM) * C::WTM;
  static_assert(kChunks % 8 == 0 && kRows >= C::WTM && C::BM % kRows == 0, "bf16 staging must fit");
  constexpr int kSwz = kChunks % 16 == 0 ? 15 : 7;
  constexpr int kThreads = C::kThreads * WK;
#pragma unroll
  for (int g0 = 0; g0 < C::BM; g0 += kRows) {
    lds_barrier();
    if (grp == 0 && wm * C::WTM >= g0 && wm * C::WTM < g0 + kRows) {
#pragma unroll
      for (int tn = 0; tn < C::TN; ++tn) {
        const int nl = wn * C::WTN + tn * 16 + 4 * fg;
#pragma unroll
        for (int tm = 0; tm < C::TM; ++tm) {
          const int ml = wm * C::WTM + tm * 16 + frow - g0;
          uint2 o;
          o.x = f32_to_bf16_rne(acc[tn][tm][0]) | (f32_to_bf16_rne(acc[tn][tm][1]) << 16);
          o.y = f32_to_bf16_rne(acc[tn][tm][2]) | (f32_to_bf16_rne(acc[tn][tm][3]) << 16);
          *reinterpret_cast<uint2*>(lds + ml * kRowBytes + (((nl >> 3) ^ (ml & kSwz)) << 4) + ((nl >> 2) & 1) * 8) = o;
        }
      }
    }
    lds_barrier();
    const int c = t % kChunks;
#pragma unroll 4
    for (int r = t / kChunks; r < kRows; r += kThreads / kChunks) {
      if (g0 + r < job.m_valid && c * 8 < n_valid) {
        const uint4 v = *reinterpret_cast<const uint4*>(lds + r * kRowBytes + ((c ^ (r & kSwz)) << 4));
        store_stream16(y + (int64_t)(job.row_lo + g0 + r) * ldy + job.n0 + c * 8, v);
      }
    }
  }
}

}  // namespace fp8rl
