// Launchers of the few-token GEMMs (kernels in gemm_small.hpp).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gemm_small.hpp"
#include "launch.hpp"

namespace fp8rl {
namespace {

struct SmallArgs {
  const uint8_t* qa;
  int64_t lda;
  const float* sa;
  int64_t ld_sa;
  const uint8_t* qw;
  int64_t ldw;
  const float* sw;
  uint16_t* y;
  int64_t ldy, m, n, k;
};

template <class C, bool kMx>
hipError_t launch_small(const SmallArgs& a, hipStream_t stream) {
  hipLaunchKernelGGL((gemm_small_kernel<C, kMx>), dim3((unsigned)(a.n / C::kRows)), dim3(C::kThreads), 0, stream, a.qa,
                     a.lda, a.sa, a.ld_sa, a.qw, a.ldw, a.sw, a.y, a.ldy, (int)a.m, (int)(a.k / 128));
  return hipGetLastError();
}

// The tile: as many activation octets as the tokens need, and 32 instead of 16
// weight rows per wave (which halves the activation reads per weight byte) where
// that still leaves 160 workgroups; up to 8 tokens always 16.  Measured on the
// Qwen3-8B linears, weights from HBM, us per call of a graph replay, 16 / 32
// rows: M = 8 qkv 7.5 / 7.1, o_proj 5.6 / 6.4, gate_up 19.9 / 22.1, down 11.3 /
// 13.9; M = 16 qkv 8.4 / 7.5, o_proj 6.1 / 6.8, gate_up 22.6 / 22.1, down 12.5 /
// 15.8; M = 32 qkv 9.9 / 8.6, o_proj 6.7 / 7.9, gate_up 27.4 / 24.1, down 15.2 /
// 19.0; M = 64 qkv 14.5 / 11.0, o_proj 8.6 / 10.2, gate_up 41.9 / 31.9, down
// 20.6 / 25.7.
template <bool kMx>
hipError_t small_by_shape(const SmallArgs& a, hipStream_t stream) {
  const bool wide = a.n / 32 >= 160;
  if (a.m <= 8) return launch_small<SmallCfg<1, 1, 3, 8, 8>, kMx>(a, stream);
  if (a.m <= 16)
    return wide ? launch_small<SmallCfg<2, 2, 2, 4, 4>, kMx>(a, stream)
                : launch_small<SmallCfg<2, 1, 2, 8, 8>, kMx>(a, stream);
  if (a.m <= 32)
    return wide ? launch_small<SmallCfg<4, 2, 2, 4, 4>, kMx>(a, stream)
                : launch_small<SmallCfg<4, 1, 3, 4, 4>, kMx>(a, stream);
  return wide ? launch_small<SmallCfg<8, 2, 2, 4, 4>, kMx>(a, stream)
              : launch_small<SmallCfg<8, 1, 2, 4, 4>, kMx>(a, stream);
}

template <int WK, bool kMx, bool kGather>
hipError_t launch_grouped_wk(const uint8_t* qa, int64_t lda, const float* sa, int64_t ld_sa, const uint8_t* qw,
                             const float* sw, const int32_t* offsets, int64_t g, int64_t rows, uint16_t* y, int64_t n,
                             int64_t k, const int32_t* gidx, int64_t src_rows, hipStream_t stream) {
  // (an expert of r > 0 rows has at most (r - 1) / 32 chunks behind its first)
  const int64_t extra = rows / kChunkRows;
  hipLaunchKernelGGL((grouped_gemm_small_kernel<WK, kMx, kGather>),
                     dim3((unsigned)(n / GroupedSmall<WK>::kRows), (unsigned)(extra + g)), dim3(256), 0, stream, qa, lda,
                     sa, ld_sa, qw, sw, offsets, (int)g, (int)extra, y, n, k, gidx, (int)src_rows);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm_small(const uint8_t* qa, int64_t lda, const float* sa, int64_t ld_sa, const uint8_t* qw,
                             int64_t ldw, const float* sw, uint16_t* y, int64_t ldy, int64_t m, int64_t n, int64_t k,
                             hipStream_t stream, bool pow2_scales) {
  const SmallArgs a{qa, lda, sa, ld_sa, qw, ldw, sw, y, ldy, m, n, k};
  return pow2_scales ? small_by_shape<true>(a, stream) : small_by_shape<false>(a, stream);
}

hipError_t launch_grouped_small(const uint8_t* qa, int64_t lda, const float* sa, int64_t ld_sa, const uint8_t* qw,
                                const float* sw, const int32_t* offsets, int64_t g, int64_t rows, uint16_t* y,
                                int64_t n, int64_t k, const int32_t* gidx, int64_t src_rows, hipStream_t stream,
                                bool pow2_scales) {
  // short K: a wave runs all of it and four waves take 64 weight rows (96 tokens x
  // 8, down, K = 768: 32.8 us, 36.1 with K in two); longer K: pairs of waves split
  // it (gate_up, K = 2048: 61.6 us, 65.9 unsplit)
  const bool short_k = k <= 1024;
#define FP8RL_GROUPED_SMALL(WK, MX, G) \
  launch_grouped_wk<WK, MX, G>(qa, lda, sa, ld_sa, qw, sw, offsets, g, rows, y, n, k, gidx, src_rows, stream)
  if (gidx) return short_k ? FP8RL_GROUPED_SMALL(1, false, true) : FP8RL_GROUPED_SMALL(2, false, true);
  if (pow2_scales) return short_k ? FP8RL_GROUPED_SMALL(1, true, false) : FP8RL_GROUPED_SMALL(2, true, false);
  return short_k ? FP8RL_GROUPED_SMALL(1, false, false) : FP8RL_GROUPED_SMALL(2, false, false);
#undef FP8RL_GROUPED_SMALL
}

}  // namespace fp8rl
