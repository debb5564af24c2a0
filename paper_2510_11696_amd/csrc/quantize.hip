// nvfp4_quantize / nvfp4_dequantize kernels for gfx950.
//
// Format: Section 3.3 "NVFP4 Quantization" (E2M1 codes, one E4M3 scale per 16
// weights, one FP32 tensor scale) and Eq. 6 for the inverse map.  The forward
// rule is the fp32 round-to-nearest chain stated in the header.  This file is
// compiled with -ffp-contract=off: every fp32 operation below is a single,
// correctly rounded IEEE operation, which is what makes the output bytes
// reproducible.
//
// Both kernels stream: 2 B read + 0.5625 B written per weight (x2 reads, the
// tensor maximum needs its own pass).
#include <type_traits>

#include "common.hpp"

namespace qerl {

constexpr int kAmaxThreads = 256;
constexpr int kAmaxMaxBlocks = 2048;
constexpr int kEncodeMaxBlocks = 2048;   // eight workgroups per compute unit: every one re-reads the partial maxima

typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t max_u16x2(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}

// Element `first` of chunk i, CH weights per chunk.  DENSE (ldw == K): the chunks of all rows are one array, which
// saves the 64-bit division that finds a chunk's row.
template <int CH, bool DENSE>
__device__ __forceinline__ const u32x4* chunk_of(const uint16_t* W, int64_t i, int64_t chunks_per_row, int64_t ldw) {
  if constexpr (DENSE) return reinterpret_cast<const u32x4*>(W + i * CH);
  const int64_t row = i / chunks_per_row;
  return reinterpret_cast<const u32x4*>(W + row * ldw + (i - row * chunks_per_row) * CH);
}

// Pass 1: maximum |w| as the bf16 bit pattern with the sign cleared (for
// finite values the integer order of those patterns is the order of the
// magnitudes).  One partial per workgroup, no atomics.  18944 x 3584: 25.5 us, 5.3 TB/s; four or eight loads of a thread in
// flight are slower (29.2, 31 us).
template <bool DENSE>
__global__ __launch_bounds__(kAmaxThreads) void amax_partial_kernel(
    const uint16_t* __restrict__ W, int64_t N, int64_t K, int64_t ldw, uint32_t* __restrict__ partial) {
  const int64_t chunks_per_row = K / 8;
  const int64_t total = N * chunks_per_row;
  const int64_t step = (int64_t)gridDim.x * kAmaxThreads;
  uint32_t m2 = 0;
  for (int64_t i = (int64_t)blockIdx.x * kAmaxThreads + threadIdx.x; i < total; i += step) {
    const u32x4 v = *chunk_of<8, DENSE>(W, i, chunks_per_row, ldw);
#pragma unroll
    for (int j = 0; j < 4; ++j) m2 = max_u16x2(m2, v[j] & 0x7fff7fffu);
  }
  uint32_t m = (m2 & 0xffffu) > (m2 >> 16) ? (m2 & 0xffffu) : (m2 >> 16);
  m = wave_max_u32(m);
  __shared__ uint32_t s[kAmaxThreads / kWave];
  if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kAmaxThreads / kWave; ++w) m = s[w] > m ? s[w] : m;
    partial[blockIdx.x] = m;
  }
}

// The sixteen codes of a block by the chain itself: one IEEE division per weight.
__device__ __forceinline__ u32x2 encode_block_divide(const uint32_t (&w)[8], float d) {
  u32x2 packed = {0u, 0u};
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    uint32_t byte = 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t bits = (w[t] >> (16 * h)) & 0xffffu;
      const float a = bf16_bits_to_f32(bits & 0x7fffu);
      const uint32_t mag = (d == 0.0f) ? 0u : e2m1_encode_rne_sat(a / d);
      byte |= (mag | ((bits >> 15) << 3)) << (4 * h);
    }
    packed[t >> 2] |= byte << (8 * (t & 3));
  }
  return packed;
}

// w / d rounded to nearest, from inv = 1 / d rounded to nearest: w * inv is within one and a half units in the last place;
// the first correction by the exactly computed remainder brings it within one, and from there the second one gives the
// correctly rounded quotient (P. Markstein, IBM J. Res. Dev. 34 (1990) 111, Theorem on division).  For
// 2^-100 <= d <= 2^100 nothing overflows (w / d <= 12), and a remainder is only inexact where the quotient is far
// below the smallest boundary of E2M1.
__device__ __forceinline__ float quotient(float w, float d, float inv) {
  float q = w * inv;
  q = __builtin_fmaf(__builtin_fmaf(-q, d, w), inv, q);
  q = __builtin_fmaf(__builtin_fmaf(-q, d, w), inv, q);
  return __builtin_copysignf(q, w);   // the corrections lose the sign of a zero
}

// Pass 2: one thread per 16-weight block.
// Sixteen IEEE divisions by the block's one divisor and a chain of comparisons per code made this pass issue-bound
// (18944 x 3584: 74 us); with quotient() above and v_cvt_scalef32_pk_fp4_f32 (nearest even, saturating, sign kept -- as
// e2m1_encode_rne_sat and the sign bit of w) it takes 33 us (5.2 TB/s).  Only a block whose scale lies outside
// quotient()'s range (zero, infinite or NaN ones among them) goes through the divisions.  Tried at this size: without the
// DENSE form 41 us; wave-contiguous loads whose halves the lanes of a pair exchange, or the next block requested ahead,
// 35..36; dividing only blocks with a quotient next to a rounding boundary, 74 (amax and w have eight significant bits
// each and the block scale four, so exact ties occur in nearly every wave).
template <bool DENSE>
__global__ __launch_bounds__(256) void encode_kernel(
    const uint16_t* __restrict__ W, int64_t N, int64_t K, int64_t ldw,
    const uint32_t* __restrict__ partial, int n_partial,
    uint8_t* __restrict__ codes, uint8_t* __restrict__ scales, float* __restrict__ tensor_scale) {
  const int64_t blocks_per_row = K / kBlock;
  const int64_t total = N * blocks_per_row;
  const int64_t step = (int64_t)gridDim.x * 256;
  __shared__ uint32_t s[4];
  uint32_t m = 0;
  for (int p = threadIdx.x; p < n_partial; p += 256) { const uint32_t q = partial[p]; m = q > m ? q : m; }
  m = wave_max_u32(m);
  if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = m;
  __syncthreads();
  m = s[0];
  for (int w = 1; w < 4; ++w) m = s[w] > m ? s[w] : m;
  const float amax = bf16_bits_to_f32(m);
  const float S32 = (amax == 0.0f) ? 1.0f : amax / 2688.0f;
  if (blockIdx.x == 0 && threadIdx.x == 0) *tensor_scale = S32;

  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += step) {
    const u32x4* src = chunk_of<kBlock, DENSE>(W, i, blocks_per_row, ldw);
    const u32x4 v0 = src[0], v1 = src[1];
    const uint32_t w[8] = {v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
    uint32_t bm2 = 0;
#pragma unroll
    for (int t = 0; t < 8; ++t) bm2 = max_u16x2(bm2, w[t] & 0x7fff7fffu);
    const uint32_t bm = (bm2 & 0xffffu) > (bm2 >> 16) ? (bm2 & 0xffffu) : (bm2 >> 16);
    const float bamax = bf16_bits_to_f32(bm);
    const float v = (bamax / 6.0f) / S32;
    const uint32_t s8 = e4m3_encode_rne_sat(v);
    const float d = S32 * e4m3_to_f32(s8);
    const float inv = 1.0f / d;
    u32x2 packed;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      uint32_t out = 0;
      auto two = [&](uint32_t pair, uint32_t old, auto sel) {
        const float q0 = quotient(__uint_as_float(pair << 16), d, inv), q1 = quotient(__uint_as_float(pair & 0xffff0000u), d, inv);
        return __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(old, q0, q1, 1.0f, decltype(sel)::value);
      };
      out = two(w[4 * half + 0], out, std::integral_constant<int, 0>{});
      out = two(w[4 * half + 1], out, std::integral_constant<int, 1>{});
      out = two(w[4 * half + 2], out, std::integral_constant<int, 2>{});
      out = two(w[4 * half + 3], out, std::integral_constant<int, 3>{});
      packed[half] = out;
    }
    if (!(d >= 0x1p-100f && d <= 0x1p100f)) packed = encode_block_divide(w, d);
    *reinterpret_cast<u32x2*>(codes + i * 8) = packed;   // rows of codes and scales follow one another without gaps
    scales[i] = (uint8_t)s8;
  }
}

__global__ void write_one_kernel(float* p) { *p = 1.0f; }

// Eq. 6, one thread per byte pair-of-codes group of 8 weights.
__global__ __launch_bounds__(256) void dequantize_kernel(
    const uint8_t* __restrict__ codes, const uint8_t* __restrict__ scales,
    const float* __restrict__ tensor_scale, int64_t N, int64_t K, float* __restrict__ out) {
  const float S32 = *tensor_scale;
  const int64_t total = N * K / 8;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
    const uint32_t c = *reinterpret_cast<const uint32_t*>(codes + i * 4);
    const float s = e4m3_to_f32(scales[i / 2]);
    float o[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) o[t] = S32 * (s * e2m1_to_f32((c >> (4 * t)) & 15u));
    f32x4* dst = reinterpret_cast<f32x4*>(out + i * 8);
    dst[0] = f32x4{o[0], o[1], o[2], o[3]};
    dst[1] = f32x4{o[4], o[5], o[6], o[7]};
  }
}

}  // namespace qerl

using namespace qerl;

extern "C" size_t nvfp4_quantize_workspace_bytes(int64_t, int64_t) {
  return (size_t)kAmaxMaxBlocks * sizeof(uint32_t);
}

extern "C" int nvfp4_quantize(const void* W, int64_t N, int64_t K, int64_t ldw, uint8_t* codes,
                              uint8_t* scales, float* tensor_scale, void* workspace,
                              size_t workspace_bytes, void* stream) {
  if (!tensor_scale) return QERL_ERR_NULL;
  if (N < 0 || K < 0 || K % kBlock != 0 || ldw < K) return QERL_ERR_SHAPE;
  hipStream_t st = (hipStream_t)stream;
  if (N == 0 || K == 0) {
    write_one_kernel<<<1, 1, 0, st>>>(tensor_scale);
    return launch_status();
  }
  if (!W || !codes || !scales) return QERL_ERR_NULL;
  if (!aligned(W, 16) || ldw % 8 != 0 || !aligned(codes, 8) || !aligned(tensor_scale, 4))
    return QERL_ERR_ALIGN;
  if (!workspace || !aligned(workspace, 4) || workspace_bytes < nvfp4_quantize_workspace_bytes(N, K))
    return QERL_ERR_WORKSPACE;
  const int64_t chunks = N * (K / 8);
  int64_t nb = ceil_div(chunks, kAmaxThreads * 4);
  if (nb > kAmaxMaxBlocks) nb = kAmaxMaxBlocks;
  uint32_t* partial = (uint32_t*)workspace;
  const uint16_t* w = (const uint16_t*)W;
  const bool dense = ldw == K;
  (dense ? amax_partial_kernel<true> : amax_partial_kernel<false>)<<<(int)nb, kAmaxThreads, 0, st>>>(w, N, K, ldw, partial);
  const int rc = launch_status();
  if (rc != QERL_OK) return rc;
  int64_t eb = ceil_div(N * (K / kBlock), 256);
  if (eb > kEncodeMaxBlocks) eb = kEncodeMaxBlocks;
  (dense ? encode_kernel<true> : encode_kernel<false>)<<<(int)eb, 256, 0, st>>>(w, N, K, ldw, partial, (int)nb, codes, scales, tensor_scale);
  return launch_status();
}

extern "C" int nvfp4_dequantize(const uint8_t* codes, const uint8_t* scales, const float* tensor_scale,
                                int64_t N, int64_t K, float* W_f32, void* stream) {
  if (N < 0 || K < 0 || K % kBlock != 0) return QERL_ERR_SHAPE;
  if (N == 0 || K == 0) return QERL_OK;
  if (!codes || !scales || !tensor_scale || !W_f32) return QERL_ERR_NULL;
  if (!aligned(codes, 4) || !aligned(W_f32, 16)) return QERL_ERR_ALIGN;
  int64_t nb = ceil_div(N * K / 8, 256);
  if (nb > 65536) nb = 65536;
  dequantize_kernel<<<(int)nb, 256, 0, (hipStream_t)stream>>>(codes, scales, tensor_scale, N, K, W_f32);
  return launch_status();
}
