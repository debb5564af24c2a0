// A wave's output tiles (rows of W by tokens, as the matrix instruction leaves them with the weights as first operand)
// to row-major bf16, in whole rows of RT * 64 bytes.
#pragma once
#include "common.hpp"

namespace qerl {

constexpr int tile_out_stride(int RT) { return RT * 64 + 16; }   // bytes per token in LDS
constexpr int tile_out_bytes(int RT) { return 64 * tile_out_stride(RT); }   // per wave

// acc[t][tt]: lane l holds of token 32 tt + l % 32 the outputs 32 t + 8 q + 4 (l / 32) + 0..3 as elements 4 q .. 4 q + 3.
// out: tile_out_bytes(RT) of LDS that belong to the wave alone; 64 tokens at a time pass through it.
template <int TT, int RT>
__device__ __forceinline__ void store_tiles(const f32x16 (&acc)[RT][TT], float scale, const uint16_t* bias, uint16_t* y, int64_t ldy, int64_t M,
                                            int64_t N, int64_t m0, int64_t n0, uint8_t* out, int lane) {
  static_assert(TT % 2 == 0, "pairs of token tiles");
  constexpr int kStride = tile_out_stride(RT);
  const int n32 = lane & 31, kg = lane >> 5;
  const bool vec = aligned_dev(y, 16) && ldy % 8 == 0;
#pragma unroll
  for (int half = 0; half < TT / 2; ++half) {
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x16& v = acc[t][half * 2 + tt];
          float o[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            o[e] = v[4 * q + e] * scale;
            if (bias) {
              const int64_t n = n0 + t * 32 + 8 * q + 4 * kg + e;
              o[e] += bf16_bits_to_f32(bias[n < N ? n : N - 1]);
            }
          }
          *reinterpret_cast<u32x2*>(out + (tt * 32 + n32) * kStride + t * 64 + q * 16 + kg * 8) = u32x2{pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3])};
        }
    __builtin_amdgcn_wave_barrier();
    constexpr int CH = RT * 4, RPI = 64 / CH;      // 16-byte chunks of a row, rows per instruction
#pragma unroll 4
    for (int i = 0; i < 64 / RPI; ++i) {
      const int row = i * RPI + lane / CH, ch = lane % CH;
      const u32x4 v = *reinterpret_cast<const u32x4*>(out + row * kStride + ch * 16);
      const int64_t m = m0 + half * 64 + row, n = n0 + ch * 8;
      if (m < M) {
        uint16_t* dst = y + m * ldy + n;
        if (vec && n + 8 <= N) {
          *reinterpret_cast<u32x4*>(dst) = v;
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (n + e < N) dst[e] = (uint16_t)(v[e >> 1] >> (16 * (e & 1)));
        }
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
}

}  // namespace qerl
