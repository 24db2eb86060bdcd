// FP8 KV cache for long-context decode (paper section 2.3): per-tensor scale
// calibration at every RL step, quantised cache writes into a paged cache, and
// decode attention that reads the FP8 cache directly.
//
// Cache layout (one array each for K and V, one 2 KiB page per block and kv head):
//   K pages [num_blocks][kv_heads][16 tokens][128 dims] (token-major);
//   V pages [num_blocks][kv_heads][4][128 dims][4]: tokens 4a .. 4a+3 of each dim
//   are 4 adjacent bytes, so that the value product's MFMA operand (4 tokens of
//   8 dims per lane) is 32 contiguous bytes.
// token slot = block * 16 + offset; block_table [batch][max_blocks] int32.
//
// Decode attention ("KV cache FP8 only": the cache, not the arithmetic, is FP8):
//   scores:  E4M3 key codes widened exactly to bf16, times the bf16 query, by
//            v_mfma_f32_16x16x32_bf16 (16 tokens x 16 query-head columns, the
//            group's heads first), scaled by k_scale * sm_scale in fp32;
//   softmax: online per head in fp32;
//   values:  P (as a sum of two bf16 terms, 16 significant bits) x V (codes
//            widened exactly to bf16) by v_mfma_f32_16x16x16_bf16, 16 per page;
//            the score layout of the first product is already the P operand
//            layout of the second;
//   a workgroup covers one split of the sequence; a second kernel merges the
//   splits (log-sum-exp weights) and applies v_scale.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "common.hpp"
#include "gemm_core.hpp"
#include "launch.hpp"

namespace fp8rl {
namespace {

constexpr int kDim = 128;          // head dimension
constexpr int kPage = 16;          // tokens per cache block
constexpr float kE4M3Max = 448.0f;
// A running maximum before its first score: finite, so that scores of -inf (a query-key
// product past the range of fp32) weigh exp(-inf) = 0 also where they are the first ones
// seen, instead of exp(-inf + inf) = NaN; below or equal to every finite score.
constexpr float kNoScore = -3.4028234663852886e38f;

typedef __bf16 v8bf16_t __attribute__((ext_vector_type(8)));
typedef __bf16 v2bf16_t __attribute__((ext_vector_type(2)));
typedef __bf16 v4bf16_t __attribute__((ext_vector_type(4)));
typedef float v4f32_t __attribute__((ext_vector_type(4)));
typedef float v2f32_t __attribute__((ext_vector_type(2)));

// ---------------------------------------------------------------------------
// Calibration: amax over a bf16 tensor (15-bit magnitude patterns order like the
// magnitudes), per-workgroup maxima into the workspace, then scale = amax / 448.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void amax_partial_kernel(const uint16_t* __restrict__ x, int64_t n,
                                                          uint32_t* __restrict__ partial) {
  __shared__ uint32_t red[4];
  uint32_t m = 0;
  const int64_t n8 = n / 8;
  const uint4* x8 = reinterpret_cast<const uint4*>(x);
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n8; i += (int64_t)gridDim.x * 256)
    m = max(m, amax16_of(x8[i]));
  if (blockIdx.x == 0 && threadIdx.x < (n & 7)) m = max(m, (uint32_t)(x[n8 * 8 + threadIdx.x] & 0x7FFFu));
  m = wave_max(m);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) partial[blockIdx.x] = max(max(red[0], red[1]), max(red[2], red[3]));
}

// At most kMaxAmaxBlocks maxima, four loads in flight per thread (64 threads walking
// them sixteen deep took 4.6 us; a launch that does nothing takes about 2.5).
constexpr int kMaxAmaxBlocks = 1024;

__global__ __launch_bounds__(256) void scale_final_kernel(const uint32_t* __restrict__ partial, int blocks,
                                                        float* __restrict__ scale) {
  __shared__ uint32_t red[4];
  uint32_t v[kMaxAmaxBlocks / 256];
#pragma unroll
  for (int i = 0; i < kMaxAmaxBlocks / 256; ++i) v[i] = partial[min((int)threadIdx.x + 256 * i, blocks - 1)];
  uint32_t m = v[0];
#pragma unroll
  for (int i = 1; i < kMaxAmaxBlocks / 256; ++i) m = max(m, v[i]);
  m = wave_max(m);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  m = max(max(red[0], red[1]), max(red[2], red[3]));
  if (threadIdx.x == 0) scale[0] = m == 0u ? 1.0f : __uint_as_float(m << 16) / kE4M3Max;   // IEEE division
}

// ---------------------------------------------------------------------------
// Cache write: code = E4M3(fl32(x / s)) saturated at +-448 (the sign of x is OR-ed
// back so that -0 gives 0x80).  Slots outside [0, num_blocks * 16) are skipped
// (negative slots mark padding tokens).  A thread handles 8 dims of one kv head's
// keys and values.
// The value page holds four slots 4a .. 4a+3 of a dim in one dword, so a group is up
// to four tokens in a row whose slots follow each other inside one such dword: four of
// them are stored as 32 contiguous bytes, fewer byte by byte.  kv_write_kernel: a
// thread looks at the groups that start inside four consecutive tokens, one of them
// where a prompt's tokens lie in order, wherever in the batch the prompt starts.
// kv_write_token_kernel: one token per thread, for small calls (decode steps), which
// are one chain of latencies.  Graph replay, us, at first (four tokens per thread and
// position in the call, an IEEE division per element, loads behind the slots) / now: 64
// scattered tokens x 8 heads 8.7 / 3.6, 500 in order 5.5 / 4.1, 13500 in order 20.0 / 16.5,
// the same from slot 3 on (no four tokens of one dword at a multiple of four) 46.7 / 16.8.
// ---------------------------------------------------------------------------
// fl32(x / s) to within what decides its E4M3 code: Markstein's correction of
// x * fl32(1 / s) is the correctly rounded quotient while no intermediate leaves the
// normal range (quant_math.hpp).  For s in [2^-91, 2^110] that holds from quotients
// of 2^-11 (the smaller ones all give code 0) up to the clamp of the first estimate
// at 1024, beyond which the result stays above 448 and saturates.  Any other s
// divides.
struct StaticScale {
  float s, r;
  bool fast;
};

__device__ __forceinline__ StaticScale static_scale(float s) {
  return StaticScale{s, 1.0f / s, s >= 0x1p-91f && s <= 0x1p110f};
}

template <bool kFast>
__device__ __forceinline__ float static_quotient(float x, const StaticScale& sc) {
  if (!kFast) return x / sc.s;
  const float q0 = fminf(fmaxf(x * sc.r, -1024.0f), 1024.0f);
  return __builtin_fmaf(__builtin_fmaf(-q0, sc.s, x), sc.r, q0);
}

template <bool kFast>
__device__ __forceinline__ uint32_t quant4_static(uint32_t w0, uint32_t w1, const StaticScale& sc) {
  float q[4] = {__uint_as_float(w0 << 16), __uint_as_float(w0 & 0xFFFF0000u), __uint_as_float(w1 << 16),
                __uint_as_float(w1 & 0xFFFF0000u)};
#pragma unroll
  for (int i = 0; i < 4; ++i) q[i] = fminf(fmaxf(static_quotient<kFast>(q[i], sc), -kE4M3Max), kE4M3Max);
  int c = __builtin_amdgcn_cvt_pk_fp8_f32(q[0], q[1], 0, false);
  c = __builtin_amdgcn_cvt_pk_fp8_f32(q[2], q[3], c, true);
  const uint32_t signs = __builtin_amdgcn_perm(w1, w0, 0x07050301u) & 0x80808080u;
  return (uint32_t)c | signs;
}

__device__ __forceinline__ uint2 quant8_static(const uint4& v, const StaticScale& sc) {
  return sc.fast ? make_uint2(quant4_static<true>(v.x, v.y, sc), quant4_static<true>(v.z, v.w, sc))
                 : make_uint2(quant4_static<false>(v.x, v.y, sc), quant4_static<false>(v.z, v.w, sc));
}

// byte j of the result = byte `b` of word j (4x4 byte transpose, one output word)
__device__ __forceinline__ uint32_t gather_byte(const uint32_t (&w)[4], int b) {
  const uint32_t pick = 0x0C0C0400u + 0x0101u * (uint32_t)b;          // (0x0C: a zero byte)
  return __builtin_amdgcn_perm(w[1], w[0], pick) | __builtin_amdgcn_perm(w[3], w[2], pick) << 16;
}

struct KvWrite {
  const uint16_t* k;
  const uint16_t* v;
  uint8_t* kc;
  uint8_t* vc;
  int kv_heads;
};

// One token's value codes (dims c * 8 ..) to its slot, byte by byte.
__device__ __forceinline__ void kv_store_value_bytes(const KvWrite& p, int64_t slot, int h, int c, const uint2& codes) {
  const int off = (int)(slot % kPage);
  uint8_t* vd = p.vc + (slot / kPage * p.kv_heads + h) * (kPage * kDim) + ((off >> 2) * kDim + c * 8) * 4 + (off & 3);
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    vd[4 * d] = (uint8_t)(codes.x >> (8 * d));
    vd[4 * (d + 4)] = (uint8_t)(codes.y >> (8 * d));
  }
}

__device__ __forceinline__ void kv_store_key(const KvWrite& p, int64_t slot, int h, int c, const uint2& codes) {
  *reinterpret_cast<uint2*>(p.kc + (slot / kPage * p.kv_heads + h) * (kPage * kDim) + (slot % kPage) * kDim + c * 8) =
      codes;
}

// kTok tokens from t, kv head h, dims c * 8 .., to slot[0 ..] (kRun: the first nt of
// them, to consecutive slots inside one dword of the value page).
template <int kTok, bool kRun>
__device__ __forceinline__ void kv_write_tokens(const KvWrite& p, int64_t t, int nt, const int64_t (&slot)[kTok], int h,
                                                int c, const StaticScale& sk, const StaticScale& sv) {
  uint4 xk[kTok], xv[kTok];                                // every load in flight before any is used
#pragma unroll
  for (int r = 0; r < kTok; ++r) {
    const int64_t src = ((t + (kRun ? min(r, nt - 1) : r)) * p.kv_heads + h) * kDim + c * 8;
    xk[r] = *reinterpret_cast<const uint4*>(p.k + src);
    xv[r] = *reinterpret_cast<const uint4*>(p.v + src);
  }
  uint32_t vlo[kTok], vhi[kTok];                           // value codes of dims c*8 .. +3, +4 .. +7
#pragma unroll
  for (int r = 0; r < kTok; ++r) {
    const uint2 cv = quant8_static(xv[r], sv);
    vlo[r] = cv.x;
    vhi[r] = cv.y;
    if (!kRun || r < nt) kv_store_key(p, kRun ? slot[0] + r : slot[r], h, c, quant8_static(xk[r], sk));
  }
  if (kRun && nt == kTok) {
    // dword of dim d = the four tokens' codes of d, dims c*8 .. c*8+7 contiguous
    if constexpr (kTok == 4) {
      const int off = (int)(slot[0] % kPage);
      uint4* vq = reinterpret_cast<uint4*>(p.vc + (slot[0] / kPage * p.kv_heads + h) * (kPage * kDim) +
                                           ((off >> 2) * kDim + c * 8) * 4);
      vq[0] = make_uint4(gather_byte(vlo, 0), gather_byte(vlo, 1), gather_byte(vlo, 2), gather_byte(vlo, 3));
      vq[1] = make_uint4(gather_byte(vhi, 0), gather_byte(vhi, 1), gather_byte(vhi, 2), gather_byte(vhi, 3));
    }
    return;
  }
#pragma unroll
  for (int r = 0; r < kTok; ++r)
    if (!kRun || r < nt) kv_store_value_bytes(p, kRun ? slot[0] + r : slot[r], h, c, make_uint2(vlo[r], vhi[r]));
}

__global__ __launch_bounds__(256) void kv_write_kernel(const KvWrite p, int64_t tokens,
                                                      const int64_t* __restrict__ slots, int64_t num_blocks,
                                                      const float* __restrict__ k_scale,
                                                      const float* __restrict__ v_scale) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;      // below 2^31 (checked by the caller)
  const uint32_t per = (uint32_t)p.kv_heads * (kDim / 8);
  const uint32_t tq = i / per, rem = i - tq * per;
  const int h = (int)(rem / (kDim / 8)), c = (int)(rem % (kDim / 8));
  const int64_t t0 = (int64_t)tq * 4;
  if (t0 >= tokens) return;
  const int64_t limit = num_blocks * kPage;
  const StaticScale sk = static_scale(k_scale[0]), sv = static_scale(v_scale[0]);
  // slots of tokens t0 - 1 .. t0 + 6 (outside the call: -2, which follows nothing)
  int64_t s[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int64_t t = t0 - 1 + j;
    s[j] = t >= 0 && t < tokens ? slots[t] : -2;
  }
  // groups that start at t0 .. t0 + 3: their lengths, 4 bits each (0: none)
  uint32_t lens = 0;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int64_t a = s[r + 1];
    if (a < 0 || a >= limit || ((a & 3) != 0 && s[r] == a - 1 && s[r] >= 0)) continue;
    int n = 1;
#pragma unroll
    for (int j = 1; j < 4; ++j)
      if (n == j && ((a + j) & 3) != 0 && r + 1 + j < 8 && s[r + 1 + j < 8 ? r + 1 + j : 7] == a + j) n = j + 1;
    lens |= (uint32_t)n << (4 * r);
  }
  if (lens == 0x1111u) {                                   // four tokens of four places (a large decode step)
    const int64_t own[4] = {s[1], s[2], s[3], s[4]};
    kv_write_tokens<4, false>(p, t0, 4, own, h, c, sk, sv);
    return;
  }
#pragma unroll 1
  for (int r = 0; r < 4; ++r) {
    const int n = (int)(lens >> (4 * r)) & 15;
    const int64_t own[4] = {slots[min(t0 + r, tokens - 1)], 0, 0, 0};
    if (n > 0) kv_write_tokens<4, true>(p, t0 + r, n, own, h, c, sk, sv);
  }
}

__global__ __launch_bounds__(256) void kv_write_token_kernel(const KvWrite p, int64_t tokens,
                                                            const int64_t* __restrict__ slots, int64_t num_blocks,
                                                            const float* __restrict__ k_scale,
                                                            const float* __restrict__ v_scale) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  const uint32_t per = (uint32_t)p.kv_heads * (kDim / 8);
  const uint32_t t = i / per, rem = i - t * per;
  if (t >= tokens) return;
  const int64_t slot = slots[t];
  const StaticScale sk = static_scale(k_scale[0]), sv = static_scale(v_scale[0]);
  if (slot >= 0 && slot < num_blocks * kPage)
    kv_write_tokens<1, false>(p, t, 1, {slot}, (int)(rem / (kDim / 8)), (int)(rem % (kDim / 8)), sk, sv);
}

// ---------------------------------------------------------------------------
// Decode attention.
// ---------------------------------------------------------------------------
template <bool kFp8>
struct CacheElem;
template <>
struct CacheElem<true> { typedef uint8_t T; };
template <>
struct CacheElem<false> { typedef uint16_t T; };

typedef short v4i16_t __attribute__((ext_vector_type(4)));

// 8 consecutive cache values -> 8 bf16 (exact: every E4M3 value is a bf16 value)
__device__ __forceinline__ v8bf16_t to_bf16x8(const uint2& c) {
  const v2bf16_t a = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)c.x, 1.0f, false);
  const v2bf16_t b = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)c.x, 1.0f, true);
  const v2bf16_t d = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)c.y, 1.0f, false);
  const v2bf16_t e = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)c.y, 1.0f, true);
  return (v8bf16_t){a[0], a[1], b[0], b[1], d[0], d[1], e[0], e[1]};
}
__device__ __forceinline__ v8bf16_t to_bf16x8(const uint4& c) { return __builtin_bit_cast(v8bf16_t, c); }

// 4 consecutive cache values -> 4 bf16 as the 16x16x16 MFMA operand
__device__ __forceinline__ v4i16_t to_bf16x4(uint32_t c) {
  const v2bf16_t a = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)c, 1.0f, false);
  const v2bf16_t b = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)c, 1.0f, true);
  return __builtin_bit_cast(v4i16_t, (v4bf16_t){a[0], a[1], b[0], b[1]});
}
__device__ __forceinline__ v4i16_t to_bf16x4(const uint2& c) { return __builtin_bit_cast(v4i16_t, c); }

__device__ __forceinline__ float shfl_xor_f(float v, int m) { return __shfl_xor(v, m, 64); }

// The value that lane kLane of this lane's four neighbours (0-3, 4-7, ..) holds.
template <int kLane>
__device__ __forceinline__ float quad_lane(uint32_t v) {
  return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x55 * kLane, 0xF, 0xF, false));
}

// Max over the four lanes with the same L % 16 (lane-row swaps, no LDS traffic).
__device__ __forceinline__ float max_over_rows(float v) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// Partial record per (sequence, kv head, split): o[G][128], then m[G], l[G],
// padded to a multiple of 4 floats (16-byte aligned records).
template <int kG>
constexpr int partial_floats() { return kG * kDim + (2 * kG + 3) / 4 * 4; }
template <int kG>
constexpr int rec_m() { return kG * kDim; }
template <int kG>
constexpr int rec_l() { return kG * kDim + kG; }

// Workgroup = 4 waves on one split of one (sequence, kv head): wave w attends over
// pages w, w + 4, ... of the split's split_pages pages, and the four results are
// combined in LDS at the end, so a split leaves one record (or, when the whole
// sequence is one split, the output itself).
//
// Pages go from the cache to LDS by DMA, whole 1 KiB runs per instruction, into a
// ring of kDepth pages that only this wave touches: no barrier in the loop, each
// wave waits for its own DMA by count, and a page's slot is refilled as soon as
// its fragments are in registers.  Loaded straight into the MFMA's register
// layout, adjacent lanes hold different tokens, a cache line each, and a CU gets
// 38 bytes per ns from the L2, 130 in whole 1 KiB runs.  Qwen3-8B layer, 64 sequences of
// 4096 .. 20480 tokens, merge included: 331 us (4.74 TB/s of cache) with register
// loads and a split per wave, 305 us (5.15 TB/s) now; a probe of 2 KiB page reads
// alone reaches 5.5-5.9 TB/s.
//
// Grid (kv head, sequence, split): the kv heads of a block (adjacent in memory) run
// together and spread over the XCDs; with the split fastest an even split count sent
// all of a sequence's first splits, the full ones, to half of the XCDs (250 sequences
// of up to 3000 tokens, two splits: 210 us, 188 us in this order).
//
// Per page, lane L, g = L / 16, j = L % 16:
//   score product (16x16x32, 4 per page): A = keys of token j, dims 32g + 8kk ..
//     (the same dim permutation for the query operand, column j = head j of the
//     group, zero past kG); the result holds S[token 4g + i][head j];
//   online softmax per head j (lanes j hold head j's running max and, each for its
//     own tokens, sum);
//   value product (16x16x16, 8 per page): A = P[head j][tokens 4g .. 4g+3] (exactly
//     the score layout), B = V[tokens 4g .. 4g+3][dim]; nb = 0..7 covers the dims of
//     the lane's 16-byte value chunks: value_dim(j, nb).  The result holds
//     O[head 4g + i][value_dim(j, nb)].
// LDS: key rows with their 16-byte chunks XOR-swizzled (by the DMA's source
// addresses) so that the 16 rows of a fragment read spread over all banks; value
// pages as they are, read 256 contiguous bytes per 16 lanes.
template <bool kFp8>
__device__ __forceinline__ constexpr int value_dim(int j, int nb) {
  return kFp8 ? (nb >> 2) * 64 + 4 * j + (nb & 3) : (nb >> 1) * 32 + 2 * j + (nb & 1);
}

template <bool kFp8>
__device__ __forceinline__ int key_swz(int row, int chunk) {
  return kFp8 ? swz(row, chunk) : row * 256 + ((chunk ^ (row & 15)) << 4);
}

// Pages in flight per wave.  Depth 2 leaves room for five FP8 workgroups per CU:
// 2 / 3 / 4 pages take 13.7 / 14.2 / 14.4 us on 20 short sequences, 24.6 / 26.0 /
// 30.0 us on 16 of up to 4096 tokens, 308 / 308 / 307 us on 64 of up to 20480.
constexpr int kRingDepth = 2;

template <int kG, bool kFp8>
struct AttnLds {
  static constexpr int kWaves = 4;
  static constexpr int kHalf = kPage * kDim * (kFp8 ? 1 : 2);   // bytes of one kv head's key (or value) page
  static constexpr int kComb = kG * kDim + 2 * kG;               // floats a wave leaves for the combination
  static constexpr int kBytes = kWaves * kRingDepth * 2 * kHalf;
  static_assert(kWaves * kComb * 4 <= kBytes, "the combination reuses the rings");
};

template <int kG, bool kFp8>
__device__ __forceinline__ void attn_decode_split_of(
    const uint16_t* __restrict__ q, const typename CacheElem<kFp8>::T* __restrict__ kcache,
    const typename CacheElem<kFp8>::T* __restrict__ vcache, int64_t num_blocks,
    const int32_t* __restrict__ block_table, int max_blocks, const int32_t* __restrict__ seq_lens, int max_seq_len,
    const float* __restrict__ k_scale, const float* __restrict__ v_scale, float sm_scale, int kv_heads,
    int split_pages, int max_splits, float* __restrict__ partial, uint16_t* __restrict__ out,
    uint8_t* lds) {
  constexpr int kElem = kFp8 ? 1 : 2;
  constexpr int kHalf = AttnLds<kG, kFp8>::kHalf;
  constexpr int kDepth = kRingDepth;
  constexpr int kOct = kHalf / 1024;                      // DMA instructions per page half
  constexpr int kWaves = AttnLds<kG, kFp8>::kWaves;
  constexpr int kComb = AttnLds<kG, kFp8>::kComb;

  const int lane = threadIdx.x & 63;
  // wave-uniform as far as the compiler knows too: page indices stay in scalar
  // registers and the block-table reads are scalar loads
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kvh = blockIdx.x, b = blockIdx.y, split = blockIdx.z;
  const int g = lane >> 4, j = lane & 15;
  const int p0 = split * split_pages;
  const int32_t* table = block_table + (int64_t)b * max_blocks;
  auto page_id = [&](int i) {                             // a bad entry reads a wrong page, never outside
    const int blk = table[min(p0 + wave + i * kWaves, max_blocks - 1)];
    return blk < 0 ? 0 : ((int64_t)blk >= num_blocks ? (int)(num_blocks - 1) : blk);
  };
  int first[kDepth + 1];                                  // (loaded beside the sequence length, not after it)
#pragma unroll
  for (int d = 0; d <= kDepth; ++d) first[d] = page_id(d);
  const int n = min(seq_lens[b], max_seq_len);
  const int p1 = min((n + kPage - 1) / kPage, p0 + split_pages);
  uint16_t* orow = out + ((int64_t)b * kv_heads + kvh) * kG * kDim;
  if (p0 >= p1) {                                         // (uniform over the workgroup)
    if (max_splits == 1)                                  // an empty sequence gives 0
      for (int i = threadIdx.x; i < kG * kDim / 2; i += 256) reinterpret_cast<uint32_t*>(orow)[i] = 0u;
    return;
  }
  const int np = (p1 - p0 - wave + kWaves - 1) / kWaves;  // this wave's pages: p0 + wave, + 4, ... (may be 0)

  // query operand: head j of the group (zero columns past kG), dims 32g + 8kk ..+7
  v8bf16_t qb[4];
  {
    const int head = kvh * kG + min(j, kG - 1);
    const uint16_t* qrow = q + ((int64_t)b * kv_heads * kG + head) * kDim + 32 * g;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const uint4 w = *reinterpret_cast<const uint4*>(qrow + 8 * kk);
      qb[kk] = __builtin_bit_cast(v8bf16_t, j < kG ? w : make_uint4(0u, 0u, 0u, 0u));
    }
  }
  const float sscale = (k_scale ? k_scale[0] : 1.0f) * sm_scale;     // bf16 cache: no scale

  uint8_t* ring = lds + wave * (kDepth * 2 * kHalf);
  // DMA source offsets inside a page half: keys row by row with swizzled chunks, values linear
  uint32_t koff[kOct];
#pragma unroll
  for (int o = 0; o < kOct; ++o) {
    const int at = o * 1024 + lane * 16, row = at / (kDim * kElem), c = (at % (kDim * kElem)) / 16;
    koff[o] = (uint32_t)key_swz<kFp8>(row, c);            // (an involution: physical chunk c holds logical c ^ key)
  }
  auto fetch = [&](int blk, int slot) {
    const int64_t base = ((int64_t)blk * kv_heads + kvh) * kHalf;
    const __amdgpu_buffer_rsrc_t rk = buffer_rsrc(reinterpret_cast<const uint8_t*>(kcache) + base);
    const __amdgpu_buffer_rsrc_t rv = buffer_rsrc(reinterpret_cast<const uint8_t*>(vcache) + base);
    uint8_t* dst = ring + slot * (2 * kHalf);
#pragma unroll
    for (int o = 0; o < kOct; ++o) lds_dma16(rk, koff[o], 0, dst + o * 1024);
#pragma unroll
    for (int o = 0; o < kOct; ++o) lds_dma16(rv, lane * 16, o * 1024, dst + kHalf + o * 1024);
  };

  float m = kNoScore, l = 0.0f;                  // head j: running max; sum over this lane's tokens
  v4f32_t o[8];
#pragma unroll
  for (int nb = 0; nb < 8; ++nb) o[nb] = (v4f32_t){0.f, 0.f, 0.f, 0.f};

#pragma unroll
  for (int d = 0; d < kDepth; ++d)
    if (d < np) fetch(first[d], d);
  int next = first[kDepth];                       // the entry of the next page to fetch, loaded a page ahead
  int slot = 0;
  for (int i = 0; i < np; ++i) {
    wait_own_ring<2 * kOct, kDepth>(np - 1 - i);
    asm volatile("" ::: "memory");
    const uint8_t* st = ring + slot * (2 * kHalf);
    uint4 kf[2 * kElem], vf[2 * kElem];
#pragma unroll
    for (int c = 0; c < 2 * kElem; ++c) {
      kf[c] = *reinterpret_cast<const uint4*>(st + key_swz<kFp8>(j, 2 * kElem * g + c));
      vf[c] = *reinterpret_cast<const uint4*>(st + kHalf + g * (kHalf / 4) + c * 256 + j * 16);
    }
    // the slot's fragments are in registers before its refill is issued
    __builtin_amdgcn_s_waitcnt(0xF | (0x7 << 4) | (0x3 << 14));   // lgkmcnt(0)
    asm volatile("" ::: "memory");
    if (i + kDepth < np) fetch(next, slot);
    next = page_id(i + kDepth + 1);
    slot = slot + 1 == kDepth ? 0 : slot + 1;
    const int valid = min(kPage, n - (p0 + wave + i * kWaves) * kPage);

    // ---- scores
    v4f32_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      v8bf16_t a;
      if constexpr (kFp8) {
        const uint4& w = kf[kk >> 1];
        a = to_bf16x8((kk & 1) ? make_uint2(w.z, w.w) : make_uint2(w.x, w.y));
      } else {
        a = to_bf16x8(kf[kk]);
      }
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, qb[kk], acc, 0, 0, 0);
    }
    // ---- online softmax for head j (tokens 4g + i of the page)
    float s[4], mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      s[r] = (4 * g + r < valid) ? acc[r] * sscale : -INFINITY;
      mx = fmaxf(mx, s[r]);
    }
    const float m_new = fmaxf(m, max_over_rows(mx));
    const float alpha = __expf(m - m_new);                  // (first page: whatever it is, o and l are 0)
    l *= alpha;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      s[r] = __expf(s[r] - m_new);                          // masked tokens: 0
      l += s[r];
    }
    m = m_new;
    // rows of o are heads 4g + i: rescale by their alphas (held by lanes 4g + i)
    if (__ballot(j < kG && alpha != 1.0f)) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float ar = __shfl(alpha, 4 * g + r, 64);
#pragma unroll
        for (int nb = 0; nb < 8; ++nb) o[nb][r] *= ar;
      }
    }
    // ---- values: P[head j][tokens 4g .. 4g+3] in bf16 (masked tokens are 0); the
    //      values of tokens past the sequence end are zeroed too (unwritten cache
    //      bytes may hold NaN codes, and 0 x NaN is NaN)
    // P as the sum of two bf16 terms (16 significant bits; one bf16 term alone
    // leaves errors of 2^-9 of each weight), two MFMAs per value tile
    const v4bf16_t p_hi = {(__bf16)s[0], (__bf16)s[1], (__bf16)s[2], (__bf16)s[3]};
    const v4bf16_t p_lo = {(__bf16)(s[0] - (float)p_hi[0]), (__bf16)(s[1] - (float)p_hi[1]),
                           (__bf16)(s[2] - (float)p_hi[2]), (__bf16)(s[3] - (float)p_hi[3])};
    const v4i16_t pa = __builtin_bit_cast(v4i16_t, p_hi), pb = __builtin_bit_cast(v4i16_t, p_lo);
    const int keep = min(max(valid - 4 * g, 0), 4);                  // tokens of this lane's four
#pragma unroll
    for (int nb = 0; nb < 8; ++nb) {
      v4i16_t vb;
      if constexpr (kFp8) {
        const uint4& w = vf[nb >> 2];
        uint32_t word = (nb & 3) == 0 ? w.x : (nb & 3) == 1 ? w.y : (nb & 3) == 2 ? w.z : w.w;
        word &= keep >= 4 ? 0xFFFFFFFFu : (1u << (8 * keep)) - 1u;
        vb = to_bf16x4(word);
      } else {
        const uint4& w = vf[nb >> 1];
        uint2 pr = (nb & 1) ? make_uint2(w.z, w.w) : make_uint2(w.x, w.y);
        pr.x &= keep >= 2 ? 0xFFFFFFFFu : (keep == 1 ? 0xFFFFu : 0u);
        pr.y &= keep >= 4 ? 0xFFFFFFFFu : (keep == 3 ? 0xFFFFu : 0u);
        vb = to_bf16x4(pr);
      }
      o[nb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(pa, vb, o[nb], 0, 0, 0);
      o[nb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(pb, vb, o[nb], 0, 0, 0);
    }
  }
  l += shfl_xor_f(l, 16);
  l += shfl_xor_f(l, 32);

  // ---- combine the four waves: each leaves o[G][128], m[G], l[G] in LDS (a wave
  //      without pages m = kNoScore, l = 0, o = 0), then every thread adds its outputs
  float* comb = reinterpret_cast<float*>(lds);
  __syncthreads();                               // the rings are idle (every wave waited for its last DMA)
  {
    float* mine = comb + wave * kComb;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int head = 4 * g + r;
      if (head < kG) {
#pragma unroll
        for (int nb = 0; nb < 8; ++nb) mine[head * kDim + value_dim<kFp8>(j, nb)] = o[nb][r];
      }
    }
    if (g == 0 && j < kG) {
      mine[kG * kDim + j] = m;
      mine[kG * kDim + kG + j] = l;
    }
  }
  __syncthreads();
  float* rec = partial + (((int64_t)b * kv_heads + kvh) * max_splits + split) * partial_floats<kG>();
  for (int e = threadIdx.x; e < kG * kDim / 2; e += 256) {
    const int head = e / (kDim / 2), d = 2 * (e % (kDim / 2));
    float mm = kNoScore;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) mm = fmaxf(mm, comb[w * kComb + kG * kDim + head]);
    // expf as in the merge (exact to an ulp far below the maximum too), one per thread: lane
    // w of each four weighs wave w, and every lane takes the four weights from there
    static_assert(kWaves == 4, "one lane of four for each wave");
    const uint32_t mine = __float_as_uint(expf(comb[(threadIdx.x & 3) * kComb + kG * kDim + head] - mm));
    const float f[kWaves] = {quad_lane<0>(mine), quad_lane<1>(mine), quad_lane<2>(mine), quad_lane<3>(mine)};
    float ls = 0.0f, a0 = 0.0f, a1 = 0.0f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const float* c = comb + w * kComb;
      ls += c[kG * kDim + kG + head] * f[w];
      a0 += c[head * kDim + d] * f[w];
      a1 += c[head * kDim + d + 1] * f[w];
    }
    if (max_splits == 1) {                       // the whole sequence: the output itself
      const float f = (v_scale ? v_scale[0] : 1.0f) / ls;
      reinterpret_cast<uint32_t*>(orow)[e] = f32_to_bf16_rne(a0 * f) | (f32_to_bf16_rne(a1 * f) << 16);
    } else {
      *reinterpret_cast<float2*>(rec + head * kDim + d) = make_float2(a0, a1);
      if (d == 0) {
        rec[rec_m<kG>() + head] = mm;
        rec[rec_l<kG>() + head] = ls;
      }
    }
  }
}

template <int kG, bool kFp8>
__global__ __launch_bounds__(kMfmaBounds) void attn_decode_kernel(
    const uint16_t* __restrict__ q, const typename CacheElem<kFp8>::T* __restrict__ kcache,
    const typename CacheElem<kFp8>::T* __restrict__ vcache, int64_t num_blocks,
    const int32_t* __restrict__ block_table, int max_blocks, const int32_t* __restrict__ seq_lens, int max_seq_len,
    const float* __restrict__ k_scale, const float* __restrict__ v_scale, float sm_scale, int kv_heads,
    int split_pages, int max_splits, float* __restrict__ partial, uint16_t* __restrict__ out) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[AttnLds<kG, kFp8>::kBytes];
  attn_decode_split_of<kG, kFp8>(q, kcache, vcache, num_blocks, block_table, max_blocks, seq_lens, max_seq_len, k_scale,
                                 v_scale, sm_scale, kv_heads, split_pages, max_splits, partial, out, lds);
}

// out[b][head][d] = bf16( v_scale * sum_s e^(m_s - M) o_s[d] / sum_s e^(m_s - M) l_s ),
// one workgroup per (head, sequence): 32 lanes hold the head's dims, kMergeSets such
// sets take the splits in turn (the records' loads are then independent of each other)
// and are combined in LDS.  Empty sequences give 0.
constexpr int kMergeSets = 4;

template <int kG>
__global__ __launch_bounds__(32 * kMergeSets) void attn_merge_kernel(
    const float* __restrict__ partial, const int32_t* __restrict__ seq_lens, int max_seq_len,
    const float* __restrict__ v_scale, int kv_heads, int split_pages, int max_splits, uint16_t* __restrict__ out) {
  __shared__ float red[kMergeSets][kDim + 2];
  const int head = blockIdx.x, b = blockIdx.y;
  const int kvh = head / kG, h = head % kG;
  const int set = threadIdx.x >> 5, d = 4 * (threadIdx.x & 31);
  const int n = min(seq_lens[b], max_seq_len);
  const int ns = min(max_splits, (max(n, 0) + split_pages * kPage - 1) / (split_pages * kPage));
  const float* base = partial + ((int64_t)b * kv_heads + kvh) * max_splits * partial_floats<kG>();
  float m = kNoScore, l = 0.0f;
  float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
  for (int s = set; s < ns; s += kMergeSets) {
    const float* r = base + (int64_t)s * partial_floats<kG>();
    const float ms = r[rec_m<kG>() + h], ls = r[rec_l<kG>() + h];
    const float4 o = *reinterpret_cast<const float4*>(r + h * kDim + d);
    const float mn = fmaxf(m, ms), f = expf(m - mn), w = expf(ms - mn);
    l = l * f + ls * w;
    a.x = a.x * f + o.x * w;
    a.y = a.y * f + o.y * w;
    a.z = a.z * f + o.z * w;
    a.w = a.w * f + o.w * w;
    m = mn;
  }
  *reinterpret_cast<float2*>(&red[set][d]) = make_float2(a.x, a.y);
  *reinterpret_cast<float2*>(&red[set][d + 2]) = make_float2(a.z, a.w);
  if (d == 0) {
    red[set][kDim] = m;
    red[set][kDim + 1] = l;
  }
  __syncthreads();
  if (set != 0) return;
  float mm = kNoScore, lsum = 0.0f;
#pragma unroll
  for (int s = 0; s < kMergeSets; ++s) mm = fmaxf(mm, red[s][kDim]);
  a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int s = 0; s < kMergeSets; ++s) {
    const float w = ns > 0 ? expf(red[s][kDim] - mm) : 0.0f;              // (a set without splits adds 0)
    lsum += red[s][kDim + 1] * w;
    a.x += red[s][d] * w;
    a.y += red[s][d + 1] * w;
    a.z += red[s][d + 2] * w;
    a.w += red[s][d + 3] * w;
  }
  const float f = ns > 0 ? (v_scale ? v_scale[0] : 1.0f) / lsum : 0.0f;
  uint2 o2;
  o2.x = f32_to_bf16_rne(a.x * f) | (f32_to_bf16_rne(a.y * f) << 16);
  o2.y = f32_to_bf16_rne(a.z * f) | (f32_to_bf16_rne(a.w * f) << 16);
  uint32_t* orow = reinterpret_cast<uint32_t*>(out + ((int64_t)b * kv_heads * kG + head) * kDim + d);
  orow[0] = o2.x;                                  // (out is 4-byte aligned)
  orow[1] = o2.y;
}

}  // namespace

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
int kv_amax_blocks(int64_t n) {
  const int64_t b = (n / 8 + 255) / 256;
  return (int)(b < 1 ? 1 : (b > kMaxAmaxBlocks ? kMaxAmaxBlocks : b));
}

hipError_t launch_kv_calibrate_scale(const uint16_t* x, int64_t n, float* scale, uint32_t* partial,
                                     hipStream_t stream) {
  const int blocks = kv_amax_blocks(n);
  hipLaunchKernelGGL(amax_partial_kernel, dim3(blocks), dim3(256), 0, stream, x, n, partial);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(scale_final_kernel, dim3(1), dim3(256), 0, stream, partial, blocks, scale);
  return hipGetLastError();
}

// (token, kv head) pairs up to which a cache write runs one token per thread (1000 x 8: 6.0
// us scattered, four per thread 8.3; 2000 x 8 in order 8.9, four per thread 5.0).
constexpr int64_t kSmallWrite = 8192;

hipError_t launch_kv_cache_write(const uint16_t* k, const uint16_t* v, int64_t tokens, int kv_heads,
                                 const int64_t* slots, int64_t num_blocks, const float* k_scale, const float* v_scale,
                                 uint8_t* k_cache, uint8_t* v_cache, hipStream_t stream) {
  const auto blocks = [&](int64_t per_thread) {
    return (unsigned)(((tokens + per_thread - 1) / per_thread * kv_heads * (kDim / 8) + 255) / 256);
  };
  const KvWrite p{k, v, k_cache, v_cache, kv_heads};
  if (tokens * kv_heads <= kSmallWrite)
    hipLaunchKernelGGL(kv_write_token_kernel, dim3(blocks(1)), dim3(256), 0, stream, p, tokens, slots, num_blocks,
                       k_scale, v_scale);
  else
    hipLaunchKernelGGL(kv_write_kernel, dim3(blocks(4)), dim3(256), 0, stream, p, tokens, slots, num_blocks, k_scale,
                       v_scale);
  return hipGetLastError();
}

AttnSplit attn_decode_split(int64_t batch, int64_t kv_heads, int64_t group, int64_t max_seq_len) {
  // records the workspace has room for: about 6144 over the whole batch, of at least
  // 256 tokens each (the launch takes as many of them as attn_plan below wants)
  constexpr int64_t kTargetWaves = 6144;
  const int64_t pairs = batch * kv_heads;
  int64_t splits = (kTargetWaves + pairs - 1) / (pairs > 0 ? pairs : 1);
  if (splits < 1) splits = 1;
  int64_t per = (max_seq_len + splits - 1) / splits;
  per = (per + kPage - 1) / kPage * kPage;
  if (per < 256) per = 256;
  AttnSplit s;
  s.split_tokens = (int)per;
  s.max_splits = (int)((max_seq_len + per - 1) / per);
  if (s.max_splits < 1) s.max_splits = 1;
  s.partial_floats = (int)(group * kDim + (2 * group + 3) / 4 * 4);   // as partial_floats<G>()
  return s;
}

// Splits of the longest sequence, one workgroup of four waves each: at least 16
// pages long (four per wave) and never more than the workspace has records for, as
// many as put the target number of workgroups on the batch.  A large cache wants
// several rounds of the 1280 resident workgroups, so that ragged sequences even out
// (64 sequences of up to 20480 tokens, 512 / 1024 / 2048 / 4608 workgroups: 365 / 336 /
// 316 / 305 us); a small one pays more for each record than it gains (8 sequences, 4 kv
// heads, up to 20000 tokens: 37 / 41 / 45 / 47 us; 16 x 8 of up to 4096: 26 / 25 / 26 /
// 26 us).
struct AttnPlan {
  int split_pages, splits;
};
static AttnPlan attn_plan(int64_t batch, int64_t kv_heads, int64_t group, int64_t max_seq_len) {
  constexpr int64_t kMinPages = 16;
  const int64_t pages = max_seq_len > 0 ? (max_seq_len + kPage - 1) / kPage : 1;
  const int64_t pairs = batch * kv_heads;
  const int64_t target = pairs * pages >= (int64_t(1) << 18) ? 4608 : 1024;
  const int64_t most = attn_decode_split(batch, kv_heads, group, max_seq_len).max_splits;
  int64_t splits = (target + pairs - 1) / pairs;
  splits = splits > most ? most : splits;
  int64_t per = (pages + splits - 1) / splits;
  per = per < kMinPages ? kMinPages : per;
  return AttnPlan{(int)per, (int)((pages + per - 1) / per)};
}

template <int kG, bool kFp8>
static hipError_t launch_attn(const uint16_t* q, const void* kc, const void* vc, int64_t num_blocks,
                              const int32_t* block_table, int64_t max_blocks, const int32_t* seq_lens, int64_t batch,
                              int64_t kv_heads, int64_t max_seq_len, const AttnPlan& pl, const float* k_scale,
                              const float* v_scale, float sm_scale, uint16_t* out, float* partial,
                              hipStream_t stream) {
  typedef typename CacheElem<kFp8>::T E;
  hipLaunchKernelGGL((attn_decode_kernel<kG, kFp8>), dim3((unsigned)kv_heads, (unsigned)batch, (unsigned)pl.splits),
                     dim3(256), 0, stream, q, static_cast<const E*>(kc), static_cast<const E*>(vc), num_blocks,
                     block_table, (int)max_blocks, seq_lens, (int)max_seq_len, k_scale, v_scale, sm_scale,
                     (int)kv_heads, pl.split_pages, pl.splits, partial, out);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || pl.splits == 1) return e;
  hipLaunchKernelGGL((attn_merge_kernel<kG>), dim3((unsigned)(kv_heads * kG), (unsigned)batch),
                     dim3(32 * kMergeSets), 0, stream, partial, seq_lens, (int)max_seq_len, v_scale, (int)kv_heads, pl.split_pages, pl.splits, out);
  return hipGetLastError();
}

hipError_t launch_attention_decode(const uint16_t* q, const void* k_cache, const void* v_cache, bool fp8_cache,
                                   int64_t num_blocks, const int32_t* block_table, int64_t max_blocks,
                                   const int32_t* seq_lens, int64_t batch, int64_t q_heads, int64_t kv_heads,
                                   int64_t max_seq_len, const float* k_scale, const float* v_scale, float sm_scale,
                                   uint16_t* out, float* partial, hipStream_t stream) {
  const int64_t group = q_heads / kv_heads;
  const AttnPlan pl = attn_plan(batch, kv_heads, group, max_seq_len);
#define FP8RL_ATTN(G)                                                                                            \
  if (group == G)                                                                                                \
    return fp8_cache ? launch_attn<G, true>(q, k_cache, v_cache, num_blocks, block_table, max_blocks, seq_lens,  \
                                            batch, kv_heads, max_seq_len, pl, k_scale, v_scale, sm_scale, out, partial, stream) \
                     : launch_attn<G, false>(q, k_cache, v_cache, num_blocks, block_table, max_blocks, seq_lens, \
                                             batch, kv_heads, max_seq_len, pl, k_scale, v_scale, sm_scale, out, partial, stream);
  FP8RL_ATTN(1)
  FP8RL_ATTN(2)
  FP8RL_ATTN(4)
  FP8RL_ATTN(8)
#undef FP8RL_ATTN
  return hipErrorInvalidValue;
}

}  // namespace fp8rl
