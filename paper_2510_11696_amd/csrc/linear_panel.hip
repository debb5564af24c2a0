// NVFP4 + LoRA linear (or a group of linears that read the same x) for 9..128 tokens, and up to 1024 on launches of few rows.
//
//   y[m,n] = S32 * sum_k x[m,k] * (s[n,k/16] * e[n,k]) + lora_scale * sum_j t[m,j] * B[n,j],   t = x A^T
//                                                                    (Eq. 6, Eq. 2)
// Two launches, or without adapters and with whole units one, and no wait between workgroups:
//
//   panel_kernel   sums of x against the rows of W and of A.  The weights are cut into units of 64, 128 or 256 output rows and
//                  stages of 128 or 256 inputs; each unit goes to the consumer workgroups (one or two per CU, all resident) in a whole
//                  number of pieces where that leaves less than a fifth of them idle, else the line "unit 0's stages, unit 1's stages, ..." is
//                  divided evenly over them, so that a launch fills most of the chip whatever N and K are.
//                  Each piece of a unit leaves its fp32 sums in a slot of the workspace.  A's rows are units of
//                  their own: dense bf16 rows in the same loop, a few K-parts each, by workgroups of the same launch.
//   panel_finish   adds a unit's slots and t's parts in K order, applies S32, B, lora_scale and bias with one rounding
//                  (gate / up pairs: SiLU(gate) * up on the rounded values) and stores bf16.
//
// A workgroup of eight waves holds a unit's rows x all tokens (of a block of at most 128): wave (rgrp, kgrp) owns one or two row tiles and
// the 64-input slice kgrp of every stage, of which there are two or four.  Each x fragment read from LDS feeds two matrix instructions (one row tile per
// wave would need the whole LDS bandwidth at 128 tokens), every weight is dequantised once a token block, and the slices are
// added through LDS at the end of a piece.  x slabs go from memory to LDS directly (16 bytes per lane, the XOR swizzle
// applied to the source address), XB - 1 stages ahead; weights into a register ring three stages ahead.  One
// barrier per stage, which waits for the slab of that stage only: all counts of outstanding loads are exact
// because requests past the end of a piece are redirected to its last stage rather than left out.
//
// What bounds it: up to 64 tokens the conversions (19 vector instructions per 512 weights and wave, of which at most three
// run beside a matrix instruction), at 128 tokens these and the matrix pipe together (a 128-input stage of 256 rows takes 1.55 us,
// 0.9 of it matrix instructions); for narrow linears the fixed chain, about 5 us of the first launch and 6 of the second.
// Measured, whole layers in graph replay, before (one workgroup per CU owning whole rows, down-projections waited for inside the
// launch, or the prefill GEMM) / now, us, the range over several cards: 7B shapes, r = 32, 32 tokens 154 / 97, 64 tokens 184 / 110..115; 14B,
// r = 64, 77 tokens 249 / 143..146; 32B, r = 64, 64 tokens 239 / 151..156, 128 tokens 272 / 204..212.
//
// Operand layouts and the packed tile format are described in linear_decode.hip.
#include "linear.hpp"
#include "lds_dma.hpp"

namespace qerl {

constexpr int kPanelRing = 4;                    // weight stages in registers per wave: one in use, three requested

// x slabs in LDS, and the LDS of a workgroup (A's rows: three stages of 16 KB + 8 KB per token tile)
template <int NT, int KW> constexpr int kPanelSlabs = KW == 2 ? 4 : (NT <= 2 ? 4 : (NT == 3 ? 3 : 2));
template <int NT, int KW> constexpr int kPanelLds = kPanelSlabs<NT, KW> * NT * KW * 4096 > 3 * (16384 + NT * 8192) ? kPanelSlabs<NT, KW> * NT * KW * 4096
                                                                                                                      : 3 * (16384 + NT * 8192);

__device__ const u32x4 g_panel_zeros = {0u, 0u, 0u, 0u};   // what is beyond the end of a row of x or A

constexpr int kPanelTParts = 8, kPanelTPartsPair = 4;     // most K-parts of t: the second launch requests them together (32B down at 128 tokens, 8 / 4 / 2: 53 / 63 / 101 us)

template <int RT> struct PanelWeights { u32x4 c[RT]; uint32_t sc[RT]; };   // one stage of a wave: 64 inputs of its row tiles

// DIRECT: no adapters, whole units; the outputs are stored here and there is no second launch, nor the sums' way through memory
// (64 tokens, two launches / one: 512 x 512 10.0 / 6.1 us, 8192 x 1024 12.0 / 7.6, 55296 x 5120 53 / 45).
template <int NT, int KW, int RT, bool DIRECT>
__global__ __launch_bounds__(512, NT == 1 ? 4 : 2) void panel_kernel(const PanelArgs a) {
  static_assert(KW == 2 || KW == 4, "a K-slice is one plane of a packed tile");
  constexpr int XB = kPanelSlabs<NT, KW>;
  constexpr int XI = NT * KW / 2;                // slab requests per wave and stage
  constexpr int RC = KW * 8;                     // 16-byte chunks of a slab row
  constexpr int kSlab = NT * 32 * RC;            // chunk c of row r sits at r * RC + (c ^ (r & 15))
  constexpr int RPI = 64 / RC;                   // rows of one request: 2 or 4
  constexpr int kUnitTiles = RT * 8 / KW;        // row tiles of a unit
  extern __shared__ __attribute__((aligned(256))) u32x4 xs[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n32 = lane & 31, kg = lane >> 5;
  const int kgrp = wave & (KW - 1), rgrp = wave / KW;
  const uint32_t lds0 = lds_address(xs);

  // ---- x: request i of a wave covers RPI whole slab rows
  const int row0 = wave * RPI + lane / RC;
  const uint32_t col_bytes = (uint32_t)(((lane % RC) ^ (row0 & 15)) * 16), k_cap = (uint32_t)(a.K * 2 - 16);
  uint32_t row_off[XI];
  auto set_tokens = [&](int tb) {
#pragma unroll
    for (int i = 0; i < XI; ++i) {
      const int m = tb * (NT * 32) + row0 + 8 * RPI * i;
      row_off[i] = (uint32_t)(m < a.M ? m : a.M - 1) * (uint32_t)(a.ldx * 2);
    }
  };
  auto request_x = [&](int stage, int buf) {
    uint32_t k = (uint32_t)stage * (uint32_t)(RC * 16) + col_bytes;
    k = k < k_cap ? k : k_cap;                   // past the end: read again, never multiplied
#pragma unroll
    for (int i = 0; i < XI; ++i)
      lds_request(lds0 + (uint32_t)((buf * kSlab + (i * 8 + wave) * 64) * 16), a.x, row_off[i] + k);
  };
  // x fragment of step j, token tile nt: row nt * 32 + n32, chunk 8 kgrp + 2 j + kg
  auto x_frag = [&](int buf, int j, int nt) {
    return __builtin_bit_cast(bf16x8, xs[buf * kSlab + (nt * 32 + n32) * RC + ((kgrp * 8 + 2 * j + kg) ^ (n32 & 15))]);
  };

  f32x16 acc[RT][NT];
  auto clear = [&]() {
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[t][nt][i] = 0.f;
  };
  // The K-slices of a row tile are added through LDS: slices 2, 3 into 0, 1, then 1 into 0 (fixed order).  On return the
  // slabs may be overwritten once every wave has passed another barrier.
  float* red = reinterpret_cast<float*>(xs);
  auto add_slices = [&]() {
    lds_wait_barrier<0>();                     // nothing is on its way to LDS any more
    float* mine = red + (rgrp * (KW / 2) + (kgrp & (KW / 2 - 1))) * (RT * NT * 1024) + lane * 4;
    auto put = [&]() {
#pragma unroll
      for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            *reinterpret_cast<f32x4*>(mine + ((t * NT + nt) * 4 + q) * 256) =
                f32x4{acc[t][nt][4 * q], acc[t][nt][4 * q + 1], acc[t][nt][4 * q + 2], acc[t][nt][4 * q + 3]};
    };
    auto get = [&](const float* p) {
#pragma unroll
      for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f32x4 v = *reinterpret_cast<const f32x4*>(p + ((t * NT + nt) * 4 + q) * 256);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[t][nt][4 * q + e] += v[e];
          }
    };
    if (kgrp >= KW / 2) put();
    lds_barrier();
    if (kgrp < KW / 2) get(mine);
    if constexpr (KW == 4) {
      if (kgrp == 1) put();                      // the place it has just read, nobody else's
      lds_barrier();
      if (kgrp == 0) get(mine + RT * NT * 1024);
    }
  };
  auto store = [&](float* p, int t) {            // one row tile: [NT][4][64 lanes][4]
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<f32x4*>(p + (nt * 4 + q) * 256 + lane * 4) =
            f32x4{acc[t][nt][4 * q], acc[t][nt][4 * q + 1], acc[t][nt][4 * q + 2], acc[t][nt][4 * q + 3]};
  };

  if (!DIRECT && (int)blockIdx.x < a.n_lora) {
    // ---- rows of the adapters' A: two rank tiles against every token tile, one K-part in stages of 128 inputs.  Both
    // operands go to LDS row by row (256 bytes of a row per 16 lanes; fetched in operand layout, 32 bytes of 32 rows
    // per request, the same bytes took 3 us a stage); a wave owns one output tile, or with few tokens a share
    // of its steps.
    constexpr int LB = 3;                        // stages in LDS
    constexpr int kXChunks = NT * 512, kStage = kXChunks + 1024;   // 16-byte chunks: x, then 64 rows of A; chunk c of row r sits at r * 16 + (c ^ (r & 15))
    constexpr int KS = NT == 1 ? 4 : NT == 2 ? 2 : 1;               // waves that share an output tile
    const int id = (int)blockIdx.x / a.tbs, tb = (int)blockIdx.x % a.tbs;
    const int blk = id / a.t_parts, part = id % a.t_parts;
    const int n_st = (int)((a.K + 127) >> 7);
    const int s0 = (int)((int64_t)part * n_st / a.t_parts), s1 = (int)((int64_t)(part + 1) * n_st / a.t_parts);
    const int lrow = wave * 4 + (lane >> 4), lcol = ((lane & 15) ^ (lrow & 15)) * 8;
    const uint16_t* xr[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const int m = tb * (NT * 32) + lrow + 32 * i;
      xr[i] = a.x + (int64_t)(m < a.M ? m : a.M - 1) * a.ldx;
    }
    const uint16_t* ar[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      int q = blk * 2 + t;
      q = q < a.rank_tiles ? q : a.rank_tiles - 1;
      const uint16_t* A = nullptr;
      int row = 0, r = 1;
#pragma unroll
      for (int i = 0; i < kMaxGroup; ++i)
        if (a.mem[i].r > 0 && q >= a.mem[i].rt_begin) { A = a.mem[i].A; row = (q - a.mem[i].rt_begin) * 32 + lrow; r = a.mem[i].r; }
      row = row < r ? row : r - 1;
      ar[t] = A + (int64_t)row * a.K;
    }
    auto request = [&](int stage, int buf) {
      const int64_t k = (int64_t)stage * 128 + lcol;
      const bool in = k < a.K;                   // past the end: zeros
      const uint32_t dst = lds0 + (uint32_t)((buf * kStage + wave * 64) * 16);
#pragma unroll
      for (int i = 0; i < NT; ++i) lds_request64(dst + (uint32_t)(i * 512 * 16), in ? (const void*)(xr[i] + k) : (const void*)&g_panel_zeros);
#pragma unroll
      for (int t = 0; t < 2; ++t) lds_request64(dst + (uint32_t)((kXChunks + t * 512) * 16), in ? (const void*)(ar[t] + k) : (const void*)&g_panel_zeros);
    };
    // wave -> rank tile t, token tile nt, steps sub, sub + KS, ... of the stage's eight (three token tiles: two waves idle)
    const int t = wave & 1, nt_raw = KS == 4 ? 0 : KS == 2 ? (wave >> 1) & 1 : wave >> 1, sub = KS == 4 ? wave >> 1 : KS == 2 ? wave >> 2 : 0;
    const bool idle = nt_raw >= NT;
    const int nt = idle ? 0 : nt_raw;
    // fp32 chains of at most 16 instructions (32 roundings; a part of a long K has 400), then added up: relative to
    // float64 the error of x A^T is that of many short parts (5120 x 27648, r = 64, 777 tokens: outputs not the nearest bf16 to the exact value 1096
    // of 4 million, 3144 with one chain; no time lost: 32B layer at 128 tokens 206.5 us both ways)
    constexpr int kChain = 2 * KS;               // stages
    f32x16 sum, chain;
#pragma unroll
    for (int i = 0; i < 16; ++i) sum[i] = chain[i] = 0.f;
    const int last = s1 - 1;
    auto clamp = [&](int s) { return s < last ? s : last; };
#pragma unroll
    for (int p = 0; p < LB - 1; ++p) request(clamp(s0 + p), p);
    int buf = 0;
    for (int s = s0; s < s1; ++s) {
      lds_wait_barrier<(LB - 2) * (NT + 2)>();
      int nbuf = buf + LB - 1;
      nbuf = nbuf >= LB ? nbuf - LB : nbuf;
      request(clamp(s + LB - 1), nbuf);
#pragma unroll
      for (int jj = 0; jj < 8 / KS; ++jj) {
        const int c = (2 * (jj * KS + sub) + kg) ^ (n32 & 15);
        const bf16x8 xf = __builtin_bit_cast(bf16x8, xs[buf * kStage + nt * 512 + n32 * 16 + c]);
        const bf16x8 af = __builtin_bit_cast(bf16x8, xs[buf * kStage + kXChunks + t * 512 + n32 * 16 + c]);
        chain = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af, xf, chain, 0, 0, 0);
      }
      buf = buf + 1 == LB ? 0 : buf + 1;
      if (((s - s0) & (kChain - 1)) == kChain - 1) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          sum[i] += chain[i];
          chain[i] = 0.f;
        }
      }
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) sum[i] += chain[i];
    if constexpr (KS > 1) {                      // the shares of a tile, in order
      lds_wait_barrier<0>();
      float* mine = red + wave * 1024 + lane;
      if (sub > 0) {
#pragma unroll
        for (int i = 0; i < 16; ++i) mine[i * 64] = sum[i];
      }
      lds_barrier();
      if (sub == 0) {
#pragma unroll
        for (int o = 1; o < KS; ++o)
#pragma unroll
          for (int i = 0; i < 16; ++i) sum[i] += mine[o * (8 / KS) * 1024 + i * 64];
      }
    } else {
      lds_wait_barrier<0>();                   // nothing may be on its way to LDS when the workgroup ends
    }
    const int rt = blk * 2 + t;
    if (sub == 0 && !idle && rt < a.rank_tiles) {
      float* p = a.t_sums + (((int64_t)part * a.rank_tiles + rt) * (a.tbs * NT) + tb * NT + nt) * 1024 + lane * 4;
#pragma unroll
      for (int q = 0; q < 4; ++q) *reinterpret_cast<f32x4*>(p + q * 256) = f32x4{sum[4 * q], sum[4 * q + 1], sum[4 * q + 2], sum[4 * q + 3]};
    }
    return;
  }

  // ---- rows of W
  const int b = (int)blockIdx.x - a.n_lora;
  int lo, hi;                                    // this workgroup's piece of the line of units x stages
  if (a.split > 0) {                             // every unit in `split` pieces, one per workgroup
    const int u = b / a.split, i = b - u * a.split;
    lo = u * a.stages + i * a.stages / a.split;
    hi = u * a.stages + (i + 1) * a.stages / a.split;
  } else {                                       // equal pieces of the line, wherever units end
    lo = b * a.per + (b < a.rem ? b : a.rem);
    hi = lo + a.per + (b < a.rem ? 1 : 0);
  }
  const int plane = kgrp & 1;
  bool first = true;
  while (lo < hi) {
    const int u = lo / a.stages;
    const int s0 = lo - u * a.stages;
    const int s1 = s0 + (hi - lo) < a.stages ? s0 + (hi - lo) : a.stages;
    lo += s1 - s0;
    const int ru = a.tbs == 1 ? u : u / a.tbs;   // unit of rows; token block
    set_tokens(u - ru * a.tbs);
    int mi = 0;
#pragma unroll
    for (int i = 1; i < kMaxGroup; ++i) mi = ru >= a.mem[i].unit_begin ? i : mi;
    const PanelMember& mem = a.mem[__builtin_amdgcn_readfirstlane(mi)];
    const uint8_t* wbase[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      int tile = (ru - mem.unit_begin) * kUnitTiles + rgrp * RT + t;
      tile = tile < mem.n_tiles ? tile : mem.n_tiles - 1;     // repeated; its slot is not read
      wbase[t] = mem.packed + (int64_t)tile * a.k_tiles * kPackTileBytes;
    }
    const uint32_t c_off = (uint32_t)(plane * 1024 + lane * 16), sc_off = (uint32_t)(2048 + n32 * 8 + plane * 4);
    const int last = s1 - 1;
    auto clamp = [&](int s) { return s < last ? s : last; };
    auto load_w = [&](PanelWeights<RT>& w, int stage) {
      int kt = stage * (KW / 2) + (kgrp >> 1);
      kt = kt < a.k_tiles ? kt : a.k_tiles - 1;
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        const uint8_t* p = wbase[t] + (int64_t)kt * kPackTileBytes;
        w.c[t] = *reinterpret_cast<const u32x4*>(p + c_off);
        w.sc[t] = *reinterpret_cast<const uint32_t*>(p + sc_off);
      }
    };
    clear();
    PanelWeights<RT> w[kPanelRing];
    if (!first) lds_barrier();             // the sums of the previous piece have been read
    first = false;
#pragma unroll
    for (int p = 0; p < XB - 1; ++p) request_x(clamp(s0 + p), p);
    asm volatile("" ::: "memory");
#pragma unroll
    for (int p = 0; p < kPanelRing - 1; ++p) load_w(w[p], clamp(s0 + p));
    bf16x8 wf[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) wf[t] = dequant8_bf16(w[0].c[t][0], e4m3_byte_f32(w[0].sc[t], 0));
    int buf = 0;
    auto stage = [&](int s, int ring, auto tail) {
      // behind slab s: the slabs of XB - 2 stages and, inside the loop, the weights of XB - 1 (two requests a row tile; in
      // the stages behind it the compiler drops requests whose data nothing uses)
      lds_wait_barrier<(XB - 2) * XI + (decltype(tail)::value ? 0 : (XB - 1) * 2 * RT)>();
      int nbuf = buf + XB - 1;
      nbuf = nbuf >= XB ? nbuf - XB : nbuf;
      request_x(clamp(s + XB - 1), nbuf);
      asm volatile("" ::: "memory");
      load_w(w[(ring + kPanelRing - 1) % kPanelRing], clamp(s + kPanelRing - 1));
      // Each stage is scheduled by itself (four at a time take the compiler minutes).  Boundary here / at the stage's end, us of o and down of the
      // 7B, 14B and 32B layers together: 128 tokens 185 / 192, 16 tokens 105 / 99; ten linears at 64 tokens, end / both 232.6 / 230.3.
      if constexpr (NT == 2 || NT == 4) __builtin_amdgcn_sched_barrier(0);
      // The conversions of step j + 1 (at the end: of the next stage's first step) and the x fragments of step j + 1
      // stand between the matrix instructions of step j.
      bf16x8 xf[NT];
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) xf[nt] = x_frag(buf, 0, nt);
      __builtin_amdgcn_sched_group_barrier(0x100, NT, 0);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        bf16x8 wn[RT];
        const PanelWeights<RT>& wr = w[j < 3 ? ring : (ring + 1) % kPanelRing];
#pragma unroll
        for (int t = 0; t < RT; ++t) wn[t] = dequant8_bf16(wr.c[t][(j + 1) & 3], e4m3_byte_f32(wr.sc[t], (j + 1) & 3));
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
          for (int t = 0; t < RT; ++t) acc[t][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[t], xf[nt], acc[t][nt], 0, 0, 0);
          if (j < 3) xf[nt] = x_frag(buf, j + 1, nt);
        }
#pragma unroll
        for (int t = 0; t < RT; ++t) wf[t] = wn[t];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
          for (int t = 0; t < RT; ++t) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                     // a matrix instruction
            __builtin_amdgcn_sched_group_barrier(0x002, (19 + NT - 1) / NT, 0);   // its share of the step's conversions
          }
          if (j < 3) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);            // an x fragment
        }
      }
      if constexpr (NT < 4) __builtin_amdgcn_sched_barrier(0);
      buf = buf + 1 == XB ? 0 : buf + 1;
    };
    int s = s0;
    const int full = (int)(a.K / (KW * 64)), s_full = s1 < full ? s1 : full;   // whole stages of 64 KW inputs
    for (; s + kPanelRing <= s_full; s += kPanelRing) {
#pragma unroll
      for (int ring = 0; ring < kPanelRing; ++ring) stage(s + ring, ring, std::false_type{});
    }
    PanelWeights<RT> wlast;
#pragma unroll
    for (int ring = 0; ring < kPanelRing; ++ring) {
      wlast = w[ring];
      if (ring == kPanelRing - 1 || s + ring >= s_full) break;
      stage(s + ring, ring, std::true_type{});
    }
    if (s_full < s1) {
      // The stage that passes the end of K stops at its last step (16 inputs) inside: what lies in the slab beyond K may be an
      // infinity, and zero weights times that are NaN.
      lds_wait_barrier<(XB - 2) * XI>();
      const int steps = (int)((a.K - (int64_t)full * (KW * 64) - kgrp * 64) >> 4);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (j >= steps) break;
        bf16x8 wl[RT];
#pragma unroll
        for (int t = 0; t < RT; ++t) wl[t] = dequant8_bf16(wlast.c[t][j], e4m3_byte_f32(wlast.sc[t], j));
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const bf16x8 xf = x_frag(buf, j, nt);
#pragma unroll
          for (int t = 0; t < RT; ++t) acc[t][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wl[t], xf, acc[t][nt], 0, 0, 0);
        }
      }
    }
    add_slices();
    if constexpr (DIRECT) {                      // the outputs, as the second launch would round them
      if (kgrp != 0) return;
      int col4 = 4 * kg, token = n32;
      asm volatile("" : "+v"(col4), "+v"(token));   // indexes that depend on the lane alone would be computed before the main loop, and spilled
      const float S32 = *mem.tensor_scale;
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        const int64_t n0 = ((int64_t)(ru - mem.unit_begin) * kUnitTiles + rgrp * RT + t) * 32;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
          for (int i = 0; i < 16; ++i) acc[t][nt][i] *= S32;
        if (mem.bias) {
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int64_t n = n0 + 8 * (i >> 2) + col4 + (i & 3);
            const float b = bf16_bits_to_f32(mem.bias[n < mem.N ? n : mem.N - 1]);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) acc[t][nt][i] += b;
          }
        }
        const bool whole = mem.y_vec && n0 + 32 <= mem.N;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          __builtin_amdgcn_sched_barrier(0);     // tile by tile: all addresses at once would be spilled
          const int tok = (u - ru * a.tbs) * (NT * 32) + nt * 32 + token;
          if (tok >= a.M) continue;
          uint16_t* dst = mem.y + (int64_t)tok * mem.ldy + n0 + col4;
          const int left = (int)(mem.N - n0 - col4 < 32 ? mem.N - n0 - col4 : 32);
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const u32x2 w = {pack_bf16x2(acc[t][nt][4 * q], acc[t][nt][4 * q + 1]), pack_bf16x2(acc[t][nt][4 * q + 2], acc[t][nt][4 * q + 3])};
            if (whole) {
              *reinterpret_cast<u32x2*>(dst + 8 * q) = w;
            } else {
#pragma unroll
              for (int e = 0; e < 4; ++e)
                if (8 * q + e < left) dst[8 * q + e] = (uint16_t)(w[e >> 1] >> (16 * (e & 1)));
            }
          }
        }
      }
    } else if (kgrp == 0) {
      float* slot = a.sums + (int64_t)(a.split > 0 ? b : b + u) * (kUnitTiles * NT * 1024);
#pragma unroll
      for (int t = 0; t < RT; ++t) store(slot + (rgrp * RT + t) * (NT * 1024), t);
    }
  }
}

// ---- second launch --------------------------------------------------------------------------------
// A workgroup of eight waves takes eight row tiles and one token tile (blockIdx.y).  It is a chain of memory round trips --
// arguments, sums, store -- so everything else is requested beside the sums: t's parts (each thread one 16-byte
// piece of up to 64 ranks), the rows of B.  t goes through LDS and the matrix instruction as three bf16 terms,
// exact to 2^-24.  WIDE: adapters of more than 64 ranks, in chunks of 64.
// PAIR: members 0 and 1 are gate_proj and up_proj, act[M, N] = bf16(bf16(SiLU(gate)) * up) is stored.
// Tiles of sums: lane l holds of token l % 32 the outputs (t: ranks) 8 q + 4 (l / 32) + 0..3 as its q-th four floats.
constexpr int kFinishStride = 72;   // bf16 per token and term in LDS: 64 ranks, rows 16-byte aligned and four banks apart

template <bool PAIR, bool WIDE>
__global__ __launch_bounds__(512, PAIR || WIDE ? 2 : 4) void panel_finish_kernel(const PanelArgs a) {
  constexpr int NM = PAIR ? 2 : 1;
  constexpr int ZB = PAIR ? 2 : 4;               // slots requested at once
  constexpr int TB = PAIR ? kPanelTPartsPair : kPanelTParts;
  __shared__ __attribute__((aligned(16))) uint16_t tl[NM][3][32 * kFinishStride];
  const int tid = threadIdx.x, lane = tid & 63, n32 = lane & 31, kg = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int NT = a.NT, nt_all = blockIdx.y;
  const int tb = a.tbs == 1 ? 0 : nt_all / NT, nt = nt_all - tb * NT;   // token block, tile in it
  const PanelMember& m0 = a.mem[PAIR ? 0 : (int)blockIdx.z];
  const int n_tiles = m0.n_tiles;
  if ((int)blockIdx.x * 8 >= n_tiles) return;    // (members of one launch differ in width)
  const int rt = (int)blockIdx.x * 8 + wave;
  const int rt_ld = rt < n_tiles ? rt : n_tiles - 1;
  // No request below stands behind a branch (each would wait for the ones before it): what does not exist is read from
  // a place that does and masked to zero.
  auto masked = [](f32x4 v, uint32_t m) { return __builtin_bit_cast(f32x4, __builtin_bit_cast(u32x4, v) & u32x4{m, m, m, m}); };

  // t: wave (h, q4) owns ranks 8 q4 + 4 (lane / 32) + 0..3 of rank tile 2 chunk + h, token lane % 32
  const int h = wave >> 2, q4 = wave & 3;
  const int64_t t_stride = (int64_t)a.rank_tiles * (a.tbs * NT) * 1024;
  f32x4 tp[NM][TB];
  auto load_t = [&](int i, const PanelMember& m, int c0) {
    int q = m.rt_begin + (c0 >> 5) + h;
    q = q < a.rank_tiles ? q : 0;
    const float* p = a.t_sums + ((int64_t)q * (a.tbs * NT) + nt_all) * 1024 + q4 * 256 + lane * 4;
#pragma unroll
    for (int z = 0; z < TB; ++z) tp[i][z] = *reinterpret_cast<const f32x4*>(p + (z < a.t_parts ? z : 0) * t_stride);
  };
  auto put_t = [&](int i, const PanelMember& m, int c0) {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int z = 0; z < TB; ++z) v += masked(tp[i][z], z < a.t_parts ? ~0u : 0u);
    const int c = h * 32 + 8 * q4 + 4 * kg;      // (r is a multiple of 8)
    v = masked(v, c0 + c < m.r ? ~0u : 0u);
#pragma unroll
    for (int k = 0; k < 3; ++k) {                // three bf16 terms, what is left each time exact in fp32
      const u32x2 w = {pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
      *reinterpret_cast<u32x2*>(&tl[i][k][n32 * kFinishStride + c]) = w;
      v -= f32x4{bf16_bits_to_f32(w[0] & 0xffffu), __uint_as_float(w[0] & 0xffff0000u), bf16_bits_to_f32(w[1] & 0xffffu), __uint_as_float(w[1] & 0xffff0000u)};
    }
  };
  u32x4 bw[NM][4];
  auto load_b = [&](int i, const PanelMember& m, int c0) {
    int64_t row = (int64_t)rt_ld * 32 + n32;
    row = row < m.N ? row : m.N - 1;
    const uint16_t* p = m.B + row * m.r;         // (r == 0: the packed weights' first bytes)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int c = c0 + 16 * j + 8 * kg;
      bw[i][j] = *reinterpret_cast<const u32x4*>(p + (c < m.r ? c : 0));
    }
  };
  f32x4 zs[NM][ZB][4];
  const float* zp[NM];
  int n_z[NM];
  const int unit_shift = a.unit_shift;
  const int64_t slot_floats = (int64_t)NT * 1024 << unit_shift;
  auto load_z = [&](int i, int z0) {
#pragma unroll
    for (int z = 0; z < ZB; ++z) {
      const float* p = zp[i] + (int64_t)(z0 + z < n_z[i] ? z0 + z : 0) * slot_floats;
#pragma unroll
      for (int q = 0; q < 4; ++q) zs[i][z][q] = *reinterpret_cast<const f32x4*>(p + q * 256);
    }
  };
#pragma unroll
  for (int i = 0; i < NM; ++i) {
    const PanelMember& m = PAIR ? a.mem[i] : m0;
    // the pieces of this row tile's unit, in K order
    const int ul = rt_ld >> unit_shift, u = (m.unit_begin + ul) * a.tbs + tb;
    // split == 0: the workgroups that own the unit's first and last stage.  A stage x belongs to x / (per + 1) below
    // `big`, counted in pieces of `per` from there on
    const int big = a.rem * (a.per + 1);
    auto owner = [&](int x) {
      return x < big ? (int)__umulhi((uint32_t)x, a.per1_inv) : a.rem + (int)__umulhi((uint32_t)(x - big), a.per_inv);
    };
    const int o0 = owner(u * a.stages), o1 = owner((u + 1) * a.stages - 1);
    const int b0 = a.split == 0 ? o0 + u : u * a.split;
    n_z[i] = a.split == 0 ? o1 - o0 + 1 : a.split;
    zp[i] = a.sums + (int64_t)b0 * slot_floats + (int64_t)((rt_ld - (ul << unit_shift)) * NT + nt) * 1024 + lane * 4;
    load_t(i, m, 0);
    load_b(i, m, 0);
    load_z(i, 0);
  }
  float S32[NM], ls[NM];
#pragma unroll
  for (int i = 0; i < NM; ++i) {
    const PanelMember& m = PAIR ? a.mem[i] : m0;
    S32[i] = *m.tensor_scale;
    ls[i] = m.lora_scale;
  }
#pragma unroll
  for (int i = 0; i < NM; ++i) put_t(i, PAIR ? a.mem[i] : m0, 0);
  __syncthreads();
  f32x4 out[NM][4];
#pragma unroll
  for (int i = 0; i < NM; ++i) {
    const PanelMember& m = PAIR ? a.mem[i] : m0;
    f32x16 up;
#pragma unroll
    for (int e = 0; e < 16; ++e) up[e] = 0.f;
    auto chunk = [&](int c0) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (WIDE || c0 + 16 * j < m.r) {         // (beyond r: t is zero)
          const bf16x8 bf = __builtin_bit_cast(bf16x8, bw[i][j]);
          const uint16_t* tq = &tl[i][0][n32 * kFinishStride + 16 * j + 8 * kg];
#pragma unroll
          for (int k = 2; k >= 0; --k)
            up = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf, *reinterpret_cast<const bf16x8*>(tq + k * 32 * kFinishStride), up, 0, 0, 0);
        }
      }
    };
    if constexpr (WIDE) {
      for (int c0 = 0; c0 < m.r; c0 += 64) {
        if (c0 > 0) {
          load_t(i, m, c0);
          load_b(i, m, c0);
          __syncthreads();
          put_t(i, m, c0);
          __syncthreads();
        }
        chunk(c0);
      }
    } else {
      chunk(0);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) out[i][q] = zs[i][0][q];
#pragma unroll
    for (int z = 1; z < ZB; ++z) {
      const uint32_t mk = z < n_z[i] ? ~0u : 0u;
#pragma unroll
      for (int q = 0; q < 4; ++q) out[i][q] += masked(zs[i][z][q], mk);
    }
    for (int z0 = ZB; z0 < n_z[i]; z0 += ZB) {   // (few rows and a long K)
      load_z(i, z0);
#pragma unroll
      for (int z = 0; z < ZB; ++z) {
        const uint32_t mk = z0 + z < n_z[i] ? ~0u : 0u;
#pragma unroll
        for (int q = 0; q < 4; ++q) out[i][q] += masked(zs[i][z][q], mk);
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float o = out[i][q][e] * S32[i];
        out[i][q][e] = m.r > 0 ? o + ls[i] * up[4 * q + e] : o;
      }
    if (m.bias) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int64_t n = (int64_t)rt_ld * 32 + 8 * q + 4 * kg + e;
          out[i][q][e] += bf16_bits_to_f32(m.bias[n < m.N ? n : m.N - 1]);
        }
    }
  }
  const int tok = nt_all * 32 + n32;
  if (rt >= n_tiles || tok >= a.M) return;
  uint16_t* dst = PAIR ? a.act + (int64_t)tok * a.ld_act : m0.y + (int64_t)tok * m0.ldy;
  const int64_t n0 = (int64_t)rt * 32 + 4 * kg;
  u32x2 w[4];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      w[q][e] = pack_bf16x2(out[0][q][2 * e], out[0][q][2 * e + 1]);
      if constexpr (PAIR) w[q][e] = silu_mul2(w[q][e], pack_bf16x2(out[NM - 1][q][2 * e], out[NM - 1][q][2 * e + 1]));
    }
  if (m0.y_vec && (int64_t)(rt + 1) * 32 <= m0.N) {
#pragma unroll
    for (int q = 0; q < 4; ++q) *reinterpret_cast<u32x2*>(dst + n0 + 8 * q) = w[q];
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (n0 + 8 * q + e < m0.N) dst[n0 + 8 * q + e] = (uint16_t)(w[q][e >> 1] >> (16 * (e & 1)));
  }
}

// ---- host -----------------------------------------------------------------------------------------
// Fills in the plan: token tiles, units, workgroups and the places of the sums in `area` bytes of workspace.
// QERL_ERR_SHAPE: not a shape for these kernels (no rows, the sums do not fit the area, or x's rows are too far apart).
int plan_panel(PanelArgs& a, float* area, size_t area_bytes) {
  if (a.M < 1 || a.M > kPanelMaxTokens || a.K < 16 || a.K % 16 != 0 || a.n_members < 1 || a.n_members > kMaxGroup) return QERL_ERR_SHAPE;
  if ((int64_t)a.M * a.ldx * 2 + a.K * 2 >= (int64_t)1 << 31) return QERL_ERR_SHAPE;   // 32-bit offsets into x
  a.tbs = (int)ceil_div(a.M, 128);               // token blocks of NT tiles each
  a.NT = (int)ceil_div(ceil_div(a.M, a.tbs), 32);
  a.k_tiles = (int)ceil_div(a.K, kPackTileK);
  a.rank_tiles = 0;
  int64_t tiles = 0;
  for (int i = 0; i < kMaxGroup; ++i) {
    if (i < a.n_members) {
      PanelMember& m = a.mem[i];
      m.n_tiles = (int)ceil_div(m.N, kPackTileRows);
      m.rt_begin = a.rank_tiles;
      if (m.r == 0) m.B = (const uint16_t*)m.packed;   // read and masked, never used
      m.y_vec = a.pairs ? aligned(a.act, 8) && a.ld_act % 4 == 0 : aligned(m.y, 8) && m.ldy % 4 == 0;
      a.rank_tiles += (int)ceil_div(m.r, 32);
      tiles += m.n_tiles;
    } else {
      a.mem[i] = a.mem[0];
      a.mem[i].r = 0;
    }
  }
  const int slots = a.NT == 1 ? 512 : 256;       // resident workgroups
  a.t_parts = 0; a.n_lora = 0;
  const int k128 = (int)ceil_div(a.K, 128);
  if (a.rank_tiles > 0) {
    const int64_t blocks = ceil_div(a.rank_tiles, 2);
    int64_t parts = slots / 4 / blocks;          // at most a quarter of the chip
    const int64_t t_most = a.pairs ? kPanelTPartsPair : kPanelTParts;
    parts = parts > t_most ? t_most : parts;
    parts = parts > k128 ? k128 : parts;
    if (a.tbs > 1) {
      // a stage of A's rows takes 0.75 us, one of a unit 1.8: as many parts as let both end together
      const int64_t main_us10 = ceil_div(ceil_div(tiles, 4) * a.tbs * ceil_div(a.k_tiles, 2), 256) * 18;
      const int64_t want = ceil_div((int64_t)k128 * 15, 2 * (main_us10 > 100 ? main_us10 : 100));
      parts = parts > want ? want : parts;
    }
    a.t_parts = (int)(parts < 1 ? 1 : parts);
    a.n_lora = (int)(blocks * a.t_parts * a.tbs);
  }
  const int64_t t_bytes = (int64_t)a.t_parts * a.rank_tiles * a.tbs * a.NT * 4096;
  if (tiles < 1 || t_bytes >= (int64_t)area_bytes) return QERL_ERR_SHAPE;   // no rows, or ranks whose sums alone exceed the area
  const int64_t room = slots - a.n_lora > 1 ? slots - a.n_lora : 1;
  // Units of 256 rows (two K-slices per workgroup, half the sums through LDS) when whole units of that size fill the
  // chip (32B gate + up at 128 tokens 98 us against 111), else of 128 (down 53 against 59); of 64 where few tokens meet few rows,
  // so that half as many pieces of K fill the chip (7B o at 32 tokens 13.1 against 14.8, 14B 15.8 against 18.1; not for a long K
  // with more than 32 tokens, where twice the slab traffic per weight shows: 32B down at 64 tokens 45 against 40).  Of 256 rows too where
  // that is one round of the chip and units of 128 would be two (40000 x 5120, r = 16, 128 tokens 79 -> 71 us; 50000 x 3584 72 -> 62).
  const int64_t big_units = ceil_div(tiles, 8) * a.tbs;
  const bool one_round = a.tbs == 1 && big_units <= slots && ceil_div(tiles, 4) > slots;   // of the large units; of the small ones it would be two
  a.KW = (a.NT >= 2 && (big_units * 5 >= slots * 4 || one_round)) ? 2 : 4;
  const int64_t one_each = 256 - a.n_lora > 1 ? 256 - a.n_lora : 1;   // consumers at one workgroup per CU
  a.RT = (a.NT <= 2 && a.tbs == 1 && ceil_div(tiles, 4) * 2 <= one_each && (a.NT == 1 || a.k_tiles <= 64)) ? 1 : 2;
  a.unit_shift = a.RT == 1 ? 1 : a.KW == 2 ? 3 : 2;
  a.unit_tiles = 1 << a.unit_shift;
  a.units = 0;
  for (int i = 0; i < a.n_members; ++i) {
    a.mem[i].unit_begin = a.units;
    a.units += (int)ceil_div(a.mem[i].n_tiles, a.unit_tiles);
  }
  for (int i = a.n_members; i < kMaxGroup; ++i) a.mem[i].unit_begin = 0x7fffffff;
  a.units *= a.tbs;
  a.stages = (int)ceil_div(a.k_tiles, a.KW / 2);
  const int64_t total = (int64_t)a.units * a.stages;
  if (total >= (int64_t)1 << 30 || a.units > 1 << 20) return QERL_ERR_SHAPE;
  const int64_t slot_bytes = (int64_t)a.unit_tiles * a.NT * 4096, avail = (int64_t)area_bytes - t_bytes;
  // Whole numbers of pieces per unit where that leaves less than a fifth of the chip idle: every workgroup then has one
  // piece, one fill and one exchange.  One workgroup per CU: 7B down at 32 tokens 22.4 us with 4 pieces (224 workgroups), 27.2 with
  // 5 (280); no more than six pieces (7B down in units of 128 rows: 26 us with 5 or 6, 30 with 10, 33 with 17).
  int64_t split = one_each / a.units;
  int64_t most = a.stages >= 7 ? a.stages * 2 / 7 : 1;   // pieces of 3.5 stages at least, and few enough for the second launch
  most = most > 6 ? 6 : most;
  split = split > most ? most : split;
  const bool even = split >= 1 && (a.units * split * 5 >= one_each * 4 || split == most);
  a.split = (int)(even ? split : 0);
  a.n_main = (int)(a.units * split);
  if (!even) {
    // as many equal pieces of the line as are resident and have a slot, or whole units, whichever is done sooner (in stages
    // per workgroup; a second piece costs about two).  The second launch divides stage indexes by multiplication, exact below 2^16.
    int64_t pieces = avail / slot_bytes - a.units + 1;
    pieces = pieces > room ? room : pieces;
    const bool fits = pieces >= 1 && total >= 2 * pieces && total < 65536;
    const int64_t second = 2 + (a.rank_tiles == 0 && !a.pairs ? 6 : 0);   // without adapters whole units need no second launch
    if (fits && total / pieces + second < ceil_div(a.units, slots) * a.stages) a.n_main = (int)pieces;
    else { a.split = 1; a.n_main = a.units; }
  }
  while (a.split > 1 && a.n_main * slot_bytes > avail) { --a.split; a.n_main = a.units * a.split; }
  a.direct = a.split == 1 && a.rank_tiles == 0 && !a.pairs ? 1 : 0;
  if (a.split == 1 && (!a.direct || a.tbs > 1) && a.n_main * slot_bytes > avail) return QERL_ERR_SHAPE;   // (beyond 128 tokens: wide enough for the GEMM)
  a.per = (int)(total / a.n_main); a.rem = (int)(total - (int64_t)a.per * a.n_main);
  auto inverse = [](int d) { return d > 1 ? (uint32_t)((((uint64_t)1 << 32) + d - 1) / d) : 0xffffffffu; };
  a.per_inv = inverse(a.per); a.per1_inv = inverse(a.per + 1);
  a.used_bytes = (size_t)(t_bytes + (a.direct ? 0 : (a.split > 0 ? a.n_main : a.n_main + a.units - 1) * slot_bytes));
  a.t_sums = area;
  a.sums = area + t_bytes / 4;
  return QERL_OK;
}

// Time of both launches beyond 128 tokens (blocks of 65 tokens and more): a stage of 256 inputs 1.7 us (three token tiles: 1.4),
// every slot written and read once at about 4 TB/s, 12 us of fixed chain, 6 us for each further round of workgroups (A's rows
// take places of the first: one unit more than the rest holds costs a round).  Measured / estimated, us, r = 64: 5120 x 5120, 256 tokens
// 30 / 32; 5120 x 13824, 256 tokens 50 / 50; 3584 x 18944, 777 tokens (r = 32) 131 / 144; 18944 x 256, 160 tokens 30 / 28; 4096 x 4096, 1000
// tokens 73 / 81 (GEMM 67).
double panel_estimate_us(const PanelArgs& a) {
  const int64_t rounds = a.split > 0 ? ceil_div(a.n_main + a.n_lora, 256) : 1;   // (A's rows take their places first)
  const double per = a.split > 0 ? (double)(ceil_div(a.stages, a.split) * rounds) : (double)(a.per + 2);
  const double stage = (a.NT == 4 ? 1.7 : 1.4) * (a.KW == 2 ? 0.5 : 1.0);
  const double slots = (double)(a.split > 0 ? a.n_main : a.n_main + a.units) * a.unit_tiles * a.NT * 4096.0;
  return per * stage + 2.0 * slots / 4.0e6 + 12.0 + 6.0 * (double)(rounds - 1);
}

template <int NT, int KW, int RT>
static int launch_panel_t(const PanelArgs& a, hipStream_t st) {
  const dim3 grid((unsigned)(a.n_lora + a.n_main));
  if (a.direct) panel_kernel<NT, KW, RT, true><<<grid, dim3(512), (kPanelLds<NT, KW>), st>>>(a);
  else panel_kernel<NT, KW, RT, false><<<grid, dim3(512), (kPanelLds<NT, KW>), st>>>(a);
  return launch_status();
}

int launch_panel(const PanelArgs& a, hipStream_t st) {
  // every pointer and size the kernels' indexing assumes
  if (!a.x || !a.sums || (a.rank_tiles > 0 && !a.t_sums) || (a.pairs && !a.act)) return QERL_ERR_NULL;
  if (a.M < 1 || a.NT < 1 || a.NT > 4 || a.tbs < 1 || a.M > a.tbs * a.NT * 32 || (a.KW != 2 && a.KW != 4) || a.unit_tiles * a.KW != 8 * a.RT ||
      a.unit_tiles != 1 << a.unit_shift || a.K < 16 ||
      (int64_t)a.k_tiles * kPackTileK < a.K || a.stages * (a.KW / 2) < a.k_tiles || a.units < 1 || a.per < 1 ||
      a.n_main < 1 || (a.split > 0 && (a.n_main != a.units * a.split || a.split > a.stages)) ||
      (int64_t)a.per * a.n_main + a.rem != (int64_t)a.units * a.stages || a.n_lora != ceil_div(a.rank_tiles, 2) * a.t_parts * a.tbs ||
      (a.direct && (a.split != 1 || a.rank_tiles > 0 || a.pairs)) || a.t_parts > (a.pairs ? kPanelTPartsPair : kPanelTParts) || (a.pairs && (a.n_members != 2 || a.mem[0].N != a.mem[1].N)))
    return QERL_ERR_SHAPE;
  int tiles_max = 0, r_max = 0;
  for (int i = 0; i < a.n_members; ++i) {
    const PanelMember& m = a.mem[i];
    if (!m.packed || !m.tensor_scale || (!a.pairs && !m.y) || (m.r > 0 && (!m.A || !m.B))) return QERL_ERR_NULL;
    tiles_max = tiles_max > m.n_tiles ? tiles_max : m.n_tiles;
    r_max = r_max > m.r ? r_max : m.r;
  }
  int rc = QERL_ERR_SHAPE;
  if (a.RT == 1 && a.KW == 4) rc = a.NT == 1 ? launch_panel_t<1, 4, 1>(a, st) : a.NT == 2 ? launch_panel_t<2, 4, 1>(a, st) : rc;
  else if (a.KW == 4) rc = a.NT == 1 ? launch_panel_t<1, 4, 2>(a, st) : a.NT == 2 ? launch_panel_t<2, 4, 2>(a, st) : a.NT == 3 ? launch_panel_t<3, 4, 2>(a, st) : launch_panel_t<4, 4, 2>(a, st);
  else if (a.RT == 2) rc = a.NT == 2 ? launch_panel_t<2, 2, 2>(a, st) : a.NT == 3 ? launch_panel_t<3, 2, 2>(a, st) : a.NT == 4 ? launch_panel_t<4, 2, 2>(a, st) : rc;
  if (rc != QERL_OK || a.direct) return rc;
  const dim3 grid((unsigned)ceil_div(tiles_max, 8), (unsigned)(a.tbs * a.NT), (unsigned)(a.pairs ? 1 : a.n_members));
  const bool wide = r_max > 64;
  if (a.pairs && wide) panel_finish_kernel<true, true><<<grid, dim3(512), 0, st>>>(a);
  else if (a.pairs) panel_finish_kernel<true, false><<<grid, dim3(512), 0, st>>>(a);
  else if (wide) panel_finish_kernel<false, true><<<grid, dim3(512), 0, st>>>(a);
  else panel_finish_kernel<false, false><<<grid, dim3(512), 0, st>>>(a);
  return launch_status();
}

}  // namespace qerl
