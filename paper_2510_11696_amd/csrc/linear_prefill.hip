// Prefill-sized NVFP4 + LoRA linears: the bf16 MFMA GEMM for launches that fill the chip with 128 x 256 tiles.
//
//   y[m,n] = S32 * sum_k x[m,k] * (s[n,k/16] * e[n,k]) + lora_scale * sum_j t[m,j] * B[n,j]
//                                                                    (Eq. 6, Eq. 2)
// A workgroup of four waves owns 128 tokens x 256 output rows, a wave 64 of the rows for all 128 tokens: each x fragment
// read from LDS feeds two matrix instructions, each weight is dequantised once per 128 tokens.  Stages of 64 inputs:
// x slabs go from memory to LDS directly, three stages ahead, weights into a register ring four stages ahead.  The
// workgroup meets once a stage, three quarters into it, when the next slab is needed: the first fragments of the next
// stage are read, and its first weights converted, between the last quarter's matrix instructions, so that nothing
// waits at a stage's start.  Two workgroups share a CU (64 KB of LDS and 256 registers per lane each) and run against each
// other's waits; one of eight waves and 512 rows, which fetches a third less, is 5 % slower (27648 + 27648 rows, K = 5120,
// 4096 tokens: 1780 us against 1700), one of four waves with 256 x 256, which converts half as often, 9 % (1855).
// The output leaves through LDS in whole 128-byte rows.
//
// What bounds it, at that shape: the chip's power.  The matrix pipe is busy 61 % of the cycles at a clock of 1.9 GHz; leaving
// out the conversions, the x requests, the weight requests or the fragment reads gains 9..12, 10, 7 and 6 % each, the matrix
// instructions alone take 1380 us (1.68 PFLOP/s).  Against gemm32_kernel (registers between memory and LDS, a barrier that
// drains them): 1903 -> 1700 us; 13824 rows, 2048 tokens 281 -> 246; 18944 + 18944 rows, K = 3584, 777 tokens 322 -> 214.
//
// LoRA and the operand layouts as in linear_gemm.hip.
#include "linear.hpp"
#include "lds_dma.hpp"
#include "lora_up.hpp"
#include "tile_out.hpp"

namespace qerl {

template <int RT> struct PrefillWeights { u32x4 c[RT]; uint32_t sc[RT]; };   // one stage of a wave: 64 inputs of its row tiles

// TT token tiles and RT row tiles of 32 per wave, W waves
template <int TT, int RT, int W>
struct PrefillCfg {
  static constexpr int kTokens = TT * 32, kRows = W * RT * 32;
  static constexpr int kSlab = TT * 256;          // 16-byte chunks of a slab: TT * 32 rows x 8; chunk c of row r sits at r * 8 + (c ^ ((r >> 1) & 7))
  static constexpr int XB = 4;                    // slabs in LDS
  static constexpr int kLdsSlabs = XB * kSlab * 16;
  static constexpr int kLdsOut = W * tile_out_bytes(RT);
  static constexpr int kLds = kLdsSlabs > kLdsOut ? kLdsSlabs : kLdsOut;
};

template <int TT, int RT, int W>
__global__ __launch_bounds__(W * 64, 2) void prefill_kernel(const GemmArgs a) {
  using C = PrefillCfg<TT, RT, W>;
  constexpr int XB = C::XB, kSlab = C::kSlab;
  constexpr int XI = TT * 4 / W;                   // slab requests per wave and stage (8 rows each)
  constexpr int R = 4;                             // weight stages in registers
  extern __shared__ __attribute__((aligned(256))) u32x4 xs[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n32 = lane & 31, kg = lane >> 5;
  const uint32_t lds0 = lds_address(xs);
  const int bid = (int)blockIdx.x;
  const int xcd = bid & 7, local = bid >> 3;
  // XCD-aware map: workgroup ids go round-robin to the 8 XCDs, each of which takes a contiguous eighth of the column blocks
  const int nb_local = local % a.nblk_per_xcd, mb = local / a.nblk_per_xcd;
  const int nb = xcd * a.nblk_per_xcd + nb_local;
  if (nb >= a.n_blocks) return;
  const int64_t m0 = (int64_t)mb * C::kTokens;
  int mi = 0;
#pragma unroll
  for (int i = 1; i < kMaxGroup; ++i) mi = (i < a.m_n && nb >= a.m[i].block_begin) ? i : mi;
  const GemmMember& mem = a.m[__builtin_amdgcn_readfirstlane(mi)];
  const int rt0 = ((nb - mem.block_begin) * W + wave) * RT;

  // ---- x
  const int row0 = wave * 8 + (lane >> 3);
  const uint32_t col_bytes = (uint32_t)(((lane & 7) ^ ((row0 >> 1) & 7)) * 16), k_cap = (uint32_t)(a.K * 2 - 16);
  const uint8_t* xbase = uniform_pointer(a.x + m0 * a.ldx);
  uint32_t row_off[XI];
#pragma unroll
  for (int i = 0; i < XI; ++i) {
    int64_t m = row0 + 8 * W * i;
    m = m0 + m < a.M ? m : a.M - 1 - m0;
    row_off[i] = (uint32_t)(m * a.ldx * 2) + col_bytes;
  }
  auto request_x = [&](int stage, int buf) {
    const uint32_t dst = lds0 + (uint32_t)((buf * kSlab + wave * 64) * 16), k = (uint32_t)stage * 128u;
    if (k + 112u <= k_cap) {
#pragma unroll
      for (int i = 0; i < XI; ++i) lds_request(dst + (uint32_t)(i * W * 1024), xbase + k, row_off[i]);
    } else {                                       // the last stage of a K that is no multiple of 64
      const uint32_t at = k + col_bytes, back = at > k_cap ? at - k_cap : 0u;   // past the end the other operand is zero; any finite value will do
#pragma unroll
      for (int i = 0; i < XI; ++i) lds_request(dst + (uint32_t)(i * W * 1024), xbase + k - 128, row_off[i] + 128u - back);
    }
  };
  const int frag = n32 * 8, sw = (n32 >> 1) & 7;
  auto x_frag = [&](int buf, int j, int tt) {
    return __builtin_bit_cast(bf16x8, xs[buf * kSlab + (frag + ((2 * j + kg) ^ sw)) + tt * 256]);
  };
  // ---- weights
  const uint8_t* wbase[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    int tile = rt0 + t;
    tile = tile < mem.n_tiles ? tile : mem.n_tiles - 1;
    wbase[t] = mem.packed + (int64_t)tile * a.k_tiles * kPackTileBytes;
  }
  auto load_w = [&](PrefillWeights<RT>& w, int stage) {
    const uint32_t c_off = (uint32_t)((stage & 1) * 1024 + lane * 16), s_off = (uint32_t)(2048 + (stage & 1) * 4 + n32 * 8);
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const uint8_t* p = wbase[t] + (int64_t)(stage >> 1) * kPackTileBytes;
      w.c[t] = *reinterpret_cast<const u32x4*>(p + c_off);
      w.sc[t] = *reinterpret_cast<const uint32_t*>(p + s_off);
    }
  };
  f32x16 acc[RT][TT];
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int tt = 0; tt < TT; ++tt)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[t][tt][i] = 0.f;

  const int n_st = (int)((a.K + 63) >> 6), last = n_st - 1;
  auto clamp = [&](int s) { return s < last ? s : last; };
  PrefillWeights<RT> w[R];
#pragma unroll
  for (int p = 0; p < XB - 1; ++p) request_x(clamp(p), p);
  asm volatile("" ::: "memory");
#pragma unroll
  for (int p = 0; p < R; ++p) load_w(w[p], clamp(p));
  lds_wait_barrier<(XB - 2) * XI>();
  bf16x8 xf[TT], wf[RT];
#pragma unroll
  for (int tt = 0; tt < TT; ++tt) xf[tt] = x_frag(0, 0, tt);
#pragma unroll
  for (int t = 0; t < RT; ++t) wf[t] = dequant8_bf16(w[0].c[t][0], e4m3_byte_f32(w[0].sc[t], 0));
  // Stage s, its slab in buffer `buf`: on entry the fragments of its first step are in registers.  Between its third and
  // fourth step the workgroup meets with slab s + 1 in LDS, whose first fragments are read during the fourth; slab s + XB - 1
  // then goes into the buffer of s - 1.
  int buf = 0;
  auto stage = [&](int s, auto ring_c, auto tail) {
    constexpr int ring = decltype(ring_c)::value;
    const int next = buf + 1 == XB ? 0 : buf + 1, before = buf == 0 ? XB - 1 : buf - 1;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (j == 3) {
        __builtin_amdgcn_sched_barrier(0);
        lds_wait_barrier<(XB - 3) * XI + (decltype(tail)::value ? 0 : (XB - 2) * 2 * RT)>();
        request_x(clamp(s + XB - 1), before);
        load_w(w[ring], clamp(s + R));             // behind the slab's requests: the compiler, which does not count those, then waits for less
        __builtin_amdgcn_sched_barrier(0);
      }
      const PrefillWeights<RT>& wr = w[j < 3 ? ring : (ring + 1) % R];
      bf16x8 wn[RT];
#pragma unroll
      for (int t = 0; t < RT; ++t) wn[t] = dequant8_bf16(wr.c[t][(j + 1) & 3], e4m3_byte_f32(wr.sc[t], (j + 1) & 3));
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) {
#pragma unroll
        for (int t = 0; t < RT; ++t) acc[t][tt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[t], xf[tt], acc[t][tt], 0, 0, 0);
        xf[tt] = j < 3 ? x_frag(buf, j + 1, tt) : x_frag(next, 0, tt);
      }
#pragma unroll
      for (int t = 0; t < RT; ++t) wf[t] = wn[t];
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) {
#pragma unroll
        for (int t = 0; t < RT; ++t) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, (19 + TT - 1) / TT, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    buf = next;
  };
  int s = 0;
  for (; s + R <= n_st; s += R) {
    stage(s, std::integral_constant<int, 0>{}, std::false_type{});
    stage(s + 1, std::integral_constant<int, 1>{}, std::false_type{});
    stage(s + 2, std::integral_constant<int, 2>{}, std::false_type{});
    stage(s + 3, std::integral_constant<int, 3>{}, std::false_type{});
  }
  if (s < n_st) {
    stage(s, std::integral_constant<int, 0>{}, std::true_type{});
    if (s + 1 < n_st) {
      stage(s + 1, std::integral_constant<int, 1>{}, std::true_type{});
      if (s + 2 < n_st) stage(s + 2, std::integral_constant<int, 2>{}, std::true_type{});
    }
  }
  lds_wait_barrier<0>();                           // nothing on its way to LDS, nobody reading

  if (mem.r > 0) lora_up<TT, RT, W, XB>(acc, mem.ts, mem.ts_ld, mem.B, mem.r, a.M, mem.N, m0, rt0, xs, wave, lane);
  const int64_t n0 = (int64_t)rt0 * 32;
  if (n0 >= mem.N) return;                         // a wave beyond the member's rows
  store_tiles<TT, RT>(acc, *mem.tensor_scale, mem.bias, mem.y, mem.ldy, a.M, mem.N, m0, n0, reinterpret_cast<uint8_t*>(xs) + wave * tile_out_bytes(RT), lane);
}

// 32-bit offsets inside a token block
bool prefill_takes(const GemmArgs& a) {
  return !a.transposed && a.ldx < (int64_t)1 << 23 && a.K >= 16 && a.K < (int64_t)1 << 30;
}

template <int TT, int RT, int W>
static int launch_prefill_t(const GemmArgs& a0, hipStream_t st) {
  using C = PrefillCfg<TT, RT, W>;
  GemmArgs a = a0;
  a.n_blocks = 0;
  for (int i = 0; i < a.m_n; ++i) {
    a.m[i].block_begin = a.n_blocks;
    a.n_blocks += (int)ceil_div(a.m[i].n_tiles, W * RT);
  }
  a.nblk_per_xcd = (int)ceil_div(a.n_blocks, 8);
  prefill_kernel<TT, RT, W><<<dim3((unsigned)(8 * a.nblk_per_xcd * ceil_div(a.M, C::kTokens))), dim3(W * 64), C::kLds, st>>>(a);
  return launch_status();
}

int launch_prefill(const GemmArgs& a, hipStream_t st) {
  if (!prefill_takes(a)) return QERL_ERR_SHAPE;
  return launch_prefill_t<4, 2, 4>(a, st);
}

}  // namespace qerl
