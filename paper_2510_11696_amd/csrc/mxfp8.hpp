// MXFP8 (E4M3 elements, one E8M0 byte per 32) of bf16 values held by four consecutive lanes, eight each.
#pragma once
#include "common.hpp"

namespace qerl {

__device__ __forceinline__ uint32_t e4m3_pair(uint32_t bits, float inv) {   // two bf16 in one word -> two bytes, in software
  const uint32_t b0 = e4m3_encode_rne_sat(bf16_bits_to_f32(bits & 0x7fffu) * inv) | ((bits >> 8) & 0x80u);
  const uint32_t b1 = e4m3_encode_rne_sat(bf16_bits_to_f32((bits >> 16) & 0x7fffu) * inv) | ((bits >> 24) & 0x80u);
  return b0 | (b1 << 8);
}

// v: this lane's eight values; the aligned four lanes of a quad hold one block and all take part.  Scale byte: the exponent
// field of the largest magnitude less 8 (E4M3's largest exponent), at least 0.  v_cvt_pk_fp8_f32 rounds to nearest even and
// keeps subnormals; it does not saturate, hence the clamp, and treats infinities and NaNs in its own way, so that blocks with
// one of those take the encoder in software, whose bytes are the ones promised.
__device__ __forceinline__ uint2 mxfp8_encode8(const u32x4 v, uint32_t& sbyte) {
  uint32_t m = 0;                       // largest magnitude as a bf16 bit pattern (integer order = magnitude order)
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t lo = v[j] & 0x7fffu, hi = (v[j] >> 16) & 0x7fffu;
    m = lo > m ? lo : m;
    m = hi > m ? hi : m;
  }
  uint32_t o = (uint32_t)__builtin_amdgcn_mov_dpp((int)m, 0xB1, 0xf, 0xf, true);   // quad_perm 1 0 3 2
  m = o > m ? o : m;
  o = (uint32_t)__builtin_amdgcn_mov_dpp((int)m, 0x4E, 0xf, 0xf, true);            // quad_perm 2 3 0 1
  m = o > m ? o : m;
  const uint32_t field = m >> 7;
  sbyte = field > 8 ? field - 8 : 0;
  const float inv = __uint_as_float((254 - sbyte) << 23);   // 2^-(sbyte - 127), a normal fp32
  uint32_t out[2];
  if (m < 0x7f80u) {
#pragma unroll
    for (int d = 0; d < 2; ++d) {
      float f[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float x = bf16_bits_to_f32((v[2 * d + (j >> 1)] >> (16 * (j & 1))) & 0xffffu) * inv;
        f[j] = __builtin_fminf(__builtin_fmaxf(x, -448.0f), 448.0f);
      }
      const int lo = __builtin_amdgcn_cvt_pk_fp8_f32(f[0], f[1], 0, false);
      out[d] = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(f[2], f[3], lo, true);
    }
  } else {
#pragma unroll
    for (int d = 0; d < 2; ++d) out[d] = e4m3_pair(v[2 * d], inv) | (e4m3_pair(v[2 * d + 1], inv) << 16);
  }
  return uint2{out[0], out[1]};
}

}  // namespace qerl
