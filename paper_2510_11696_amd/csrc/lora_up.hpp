// LoRA up-projection of a 128-token workgroup tile: 3 r more input columns [hi | mid | lo] . [B ; B ; B]^T on the bf16 matrix
// instruction.  The columns of ts go to LDS in slabs of 64 (rows of 128 bytes, the layout of the x slabs), up to XB at a time;
// the rows of B come straight from memory, a slab's fragments requested before the slab is waited for.
#pragma once
#include "common.hpp"
#include "lds_dma.hpp"

namespace qerl {

static __device__ const u32x4 g_lora_up_zeros = {0u, 0u, 0u, 0u};

// acc[t][tt] += B rows 32 (rt0 + t) .. x tokens m0 + 32 tt ..; every wave of the W takes part.  On entry nothing is on its way to
// LDS and nobody reads it; so it is on return.
template <int TT, int RT, int W, int XB>
__device__ __forceinline__ void lora_up(f32x16 (&acc)[RT][TT], const uint16_t* ts, int64_t ts_ld, const uint16_t* B, int r, int64_t M, int64_t N, int64_t m0,
                                        int rt0, u32x4* xs, int wave, int lane) {
  constexpr int kSlab = TT * 256, XI = TT * 4 / W;
  const int n32 = lane & 31, kg = lane >> 5;
  const uint32_t lds0 = lds_address(xs);
  const int row0 = wave * 8 + (lane >> 3), col = ((lane & 7) ^ ((row0 >> 1) & 7)) * 8;
  const int n_slabs = (3 * r + 63) / 64;
  const uint16_t* brow[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    int64_t row = (int64_t)(rt0 + t) * 32 + n32;
    row = row < N ? row : N - 1;
    brow[t] = B + row * r;
  }
  auto load_b = [&](u32x4 (&b)[4][RT], int e) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int c = e * 64 + 16 * j + 8 * kg;
      const bool in = c < 3 * r;
      const int cb = !in ? 0 : c >= 2 * r ? c - 2 * r : c >= r ? c - r : c;
      const uint32_t mask = in ? ~0u : 0u;
#pragma unroll
      for (int t = 0; t < RT; ++t) b[j][t] = *reinterpret_cast<const u32x4*>(brow[t] + cb) & u32x4{mask, mask, mask, mask};
    }
  };
  for (int e0 = 0; e0 < n_slabs; e0 += XB) {
    const int n_e = n_slabs - e0 < XB ? n_slabs - e0 : XB;
    for (int e = 0; e < n_e; ++e) {
      const int c = (e0 + e) * 64 + col;
#pragma unroll
      for (int i = 0; i < XI; ++i) {
        int64_t m = m0 + row0 + 8 * W * i;
        m = m < M ? m : M - 1;
        lds_request64(lds0 + (uint32_t)((e * kSlab + (i * W + wave) * 64) * 16), c < ts_ld ? (const void*)(ts + m * ts_ld + c) : (const void*)&g_lora_up_zeros);
      }
    }
    u32x4 b[4][RT];
    load_b(b, e0);
    lds_wait_barrier<0>();
    for (int e = 0; e < n_e; ++e) {
      u32x4 bn[4][RT];
      load_b(bn, e0 + e + 1);                      // (beyond the last: masked)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
          const bf16x8 xf = __builtin_bit_cast(bf16x8, xs[e * kSlab + tt * 256 + n32 * 8 + ((2 * j + kg) ^ ((n32 >> 1) & 7))]);
#pragma unroll
          for (int t = 0; t < RT; ++t) acc[t][tt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, b[j][t]), xf, acc[t][tt], 0, 0, 0);
        }
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int t = 0; t < RT; ++t) b[j][t] = bn[j][t];
    }
    lds_wait_barrier<0>();
  }
}

}  // namespace qerl
