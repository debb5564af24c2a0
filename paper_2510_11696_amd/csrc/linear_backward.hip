// Backward pass of the NVFP4 + LoRA linear: only the adapters are trained, the gradient flows through the
// frozen quantised weights (Preliminary, "Low-rank Adaptation"; Eq. 2, Eq. 6).  For an upstream dY [M, N]:
//
//   dX = dY W_hat + s (dY B) A          [M, K]  bf16
//   dA = s (dY B)^T x                   [r, K]  fp32
//   dB = s dY^T (x A^T)                 [N, r]  fp32          (s = lora_scale)
//
// dX contracts over N, i.e. over the ROWS of the packed weight tiles, so the same bytes are needed in a second,
// transposed tile order (nvfp4_prepack_t; the weights are frozen, the order is made once):
//   tile (kt, nt) = 32 inputs k = 32 kt .. + 31  x  128 rows n = 128 nt .. + 127, 2304 bytes like the forward tile:
//   two 1 KiB planes of codes (plane p = rows 64 p .. 64 p + 63; lane l = (c = l % 32, g = l / 32) owns 16 bytes:
//   dword j holds the codes of rows 64 p + 16 j + 8 g .. + 7 at input 32 kt + c, nibble i = row + i), then 256 scale
//   bytes [plane][input block 0..1][64 rows].  Tiles of one kt are consecutive along nt.
// gemm32_kernel<.., TR = true> multiplies dY with it (the eight weights of a lane and step carry eight different
// E4M3 scales; products stay exact in bf16), the LoRA term enters as 3r more contraction columns exactly as in
// the forward pass with the roles of A and B exchanged (both transposed once per call: they change with every
// optimiser step).  dA and dB are skinny products over the token dimension (MFMA, operands transposed through LDS),
// tokens split over a few workgroups whose partial sums are added in order.
// Several linears that read the same x (q / k / v, gate / up: Section 3.3) go through one call: dX is the sum of the
// members' terms, formed by ONE launch of the transposed GEMM whose contraction runs over the members' rows one
// after the other (fp32 throughout, one rounding), and the down-projections of x for all adapters share a launch.
#include "linear.hpp"

namespace qerl {

// ---- transposed tile order -----------------------------------------------------------------------------
__global__ __launch_bounds__(256) void prepack_t_kernel(const uint8_t* __restrict__ codes, const uint8_t* __restrict__ scales,
                                                        int64_t N, int64_t K, int64_t k_tiles32, int64_t n_tiles128,
                                                        uint8_t* __restrict__ out) {
  // one thread per (tile, plane, lane) for the codes; the first 256 threads-worth of each tile also place a scale byte
  const int64_t total = k_tiles32 * n_tiles128 * 128;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
    const int lane = (int)(i & 63), plane = (int)((i >> 6) & 1);
    const int64_t tile = i >> 7, nt = tile % n_tiles128, kt = tile / n_tiles128;
    const int c = lane & 31, g = lane >> 5;
    const int64_t k = kt * 32 + c;
    uint8_t* t = out + tile * kPackTileBytes;
    u32x4 v = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      uint32_t w = 0;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int64_t n = nt * 128 + plane * 64 + 16 * j + 8 * g + e;
        uint32_t nib = 0;
        if (n < N && k < K) nib = (codes[n * (K / 2) + k / 2] >> (4 * (int)(k & 1))) & 0xFu;
        w |= nib << (4 * e);
      }
      v[j] = w;
    }
    *reinterpret_cast<u32x4*>(t + plane * 1024 + lane * 16) = v;
    // scale bytes: [plane][input block kb][64 rows]; this thread places two of the tile's 256
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int idx = plane * 128 + h * 64 + lane;          // = plane * 128 + kb * 64 + row, kb = h, row = lane
      const int64_t n = nt * 128 + plane * 64 + lane, kb = kt * 2 + h;
      uint8_t sc = 0;
      if (n < N && kb * 16 < K) sc = scales[n * (K / 16) + kb];
      t[2048 + idx] = sc;
    }
  }
}

// One launch before the products of a call: AT[c, j] = A[j, c] and BT[j, n] = B[n, j] of every member (the adapters
// change with every optimiser step, so they are transposed per call), and the arrival counters of the K-split
// down-projections set to zero by the last block.  64 x 64 tiles through LDS, whole rows of a tile on both sides.
struct TransposeJob { const uint16_t* in; uint16_t* out; int64_t R, C; int block0; };   // in [R, C], out [C, R]
struct PrepareArgs { TransposeJob job[2 * kMaxGroup]; int n; int n_blocks; uint32_t* counters; int n_counters; };
__global__ __launch_bounds__(256) void backward_prepare_kernel(const PrepareArgs a) {
  __shared__ uint16_t lds[64 * 66];    // 64 x 64 elements; the odd number of dwords per row spreads the banks
  const int b = blockIdx.x;
  if (b >= a.n_blocks) {
    for (int i = threadIdx.x; i < a.n_counters; i += 256) a.counters[i] = 0u;
    return;
  }
  int ji = 0;
#pragma unroll
  for (int i = 1; i < 2 * kMaxGroup; ++i) ji = i < a.n && b >= a.job[i].block0 ? i : ji;
  const TransposeJob t = a.job[ji];
  const int c_tiles = (int)ceil_div_dev(t.C, 64), tile = b - t.block0, rt = tile / c_tiles;
  const int64_t r0 = (int64_t)rt * 64, c0 = (int64_t)(tile - rt * c_tiles) * 64;
  const int i = threadIdx.x & 63, j0 = threadIdx.x >> 6;
  uint16_t v[16];                      // all requested before the first is stored; rows and columns outside are redirected
  const int64_t ci = c0 + i < t.C ? c0 + i : t.C - 1;
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int64_t rj = r0 + j0 + 4 * k;
    v[k] = t.in[(rj < t.R ? rj : t.R - 1) * t.C + ci];
  }
#pragma unroll
  for (int k = 0; k < 16; ++k) lds[(j0 + 4 * k) * 66 + i] = v[k];
  __syncthreads();
#pragma unroll
  for (int j = j0; j < 64; j += 4)
    if (c0 + j < t.C && r0 + i < t.R) t.out[(c0 + j) * t.R + r0 + i] = lds[i * 66 + j];
}

// ---- dA, dB: sum over the tokens of P[m, j] * Q[m, c], all of a call's products in one launch --------------------
// P [M, r] arrives as the three bf16 terms the LoRA down-projection kernel writes ([M, ts_ld]: hi | mid | lo,
// their sum exact to 2^-24); Q is x (dA) or dY (dB), bf16, row-major.  Both operands are contracted over their ROWS, so a
// lane's eight consecutive contraction values lie in eight different rows.  A thread therefore fetches two columns of
// eight tokens (256 contiguous bytes per wave and row), turns them in registers and leaves two 16-byte MFMA operands in
// LDS ([8-token group][column][8 tokens]), which the products read back with one ds_read_b128 each: seven reads for
// six MFMAs, the two pipes about level.  With row-major tiles and sixteen-bit reads, 56 of them for the same six, the LDS
// pipe was the bound, and each product was a launch of its own: the fourteen products of a 14B layer (2048 tokens, r = 64)
// took 364 us and their sums 78 us in 28 launches, against 178 us and 29 us in ten.  Guarded 64-bit loads instead of buffer
// loads (a branch and an argument fetch each) cost 404 us.
// A workgroup owns 128 columns of one product (32 per wave), all ranks and one chunk of the tokens; three MFMAs per rank tile and
// 16 tokens (one per term).  Chunks: as many as give a product 128 workgroups -- their partial sums, 4 r bytes per
// column and chunk, are written and read once each, so no more than that.  The count depends on the product alone, not on
// the group it comes in, so a member's dA is the same bits in a group and by itself (dB need not be: the K-parts of
// t = x A^T, which it is made from, depend on the number of adapters that share its launch).  The partial sums are added in
// order by a second launch.
constexpr int kGradRanks = 64;       // most ranks
constexpr int kGradChunksMax = 8;    // token chunks (workgroups along M)
constexpr int kGradTokens = 64;      // tokens per LDS tile
constexpr int kGradGroups = kGradTokens / 8, kGradCols = 128, kGradPCols = 3 * kGradRanks;
constexpr int64_t kGradWorkgroups = 128;
constexpr int64_t kGradOneChunkTiles = 8;   // a product of more tiles takes at least two chunks: its error then stays below that of eight chunks in plain chains
struct GradSplit { int n_chunks; int64_t tokens_per_chunk; };
static GradSplit grad_split(int64_t M, int64_t C) {
  const int64_t tiles = ceil_div(M, kGradTokens);
  int64_t chunks = ceil_div(kGradWorkgroups, ceil_div(C, kGradCols));
  const int64_t by_tiles = tiles > kGradOneChunkTiles ? 2 : 1;
  chunks = chunks < by_tiles ? by_tiles : chunks;
  chunks = chunks > kGradChunksMax ? kGradChunksMax : chunks;
  chunks = chunks > tiles ? tiles : chunks;
  const int64_t tokens = ceil_div(tiles, chunks) * kGradTokens;
  return GradSplit{(int)ceil_div(M, tokens), tokens};
}
struct GradJob {
  const uint16_t* P; int64_t p_ld; const uint16_t* Q; int64_t q_ld; int64_t C; int r;
  int rank_major;                    // result wanted as [r, C] (dA), else [C, r] (dB)
  const float* mult; float* out;
  int n_chunks; int64_t tokens_per_chunk;
  int col_blocks, block0;            // the product's workgroups: [chunk][column block] from block0 on
  float* partial;                    // [chunk][C r] in the order of the result
  int64_t elem0;                     // first of the product's elements among those the second launch sums
};
struct GradArgs { GradJob job[2 * kMaxGroup]; int n; int n_blocks; int64_t M, elems; };

// RANK_MAJOR: the MFMA operands change places, so that a lane owns a column and the results leave as rows of C.
template <bool RANK_MAJOR>
__device__ __forceinline__ void lora_grad_block(const GradJob& jb, int64_t c0, int64_t m_lo, int64_t m_hi, float mult, float* dst,
                                                u32x4* sQ, u32x4* sP) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n32 = lane & 31, kg = lane >> 5;
  const int r = jb.r;
  const int64_t C = jb.C;
  // The leading term is summed tile by tile (four MFMAs) and the tiles' sums are added up; the small terms, at most a 256th
  // of its size, run through.  That keeps the fp32 chains short where a chunk is long.  Relative error of a product against
  // float64, eight chunks of one chain each / one chain for the leading term in the chunks of grad_split / these two
  // levels: 640 tokens, C = 18944: 7.4e-8 / 1.41e-7 / 6.8e-8; 2048 tokens, C = 13824: 1.02e-7 / 1.31e-7 / 9.2e-8.
  f32x16 sum[2], small[2];
#pragma unroll
  for (int jt = 0; jt < 2; ++jt)
#pragma unroll
    for (int i = 0; i < 16; ++i) sum[jt][i] = small[jt][i] = 0.f;
  // The tile after the current one is requested before the current one is multiplied.  Buffer loads relative to the
  // tile: tokens past the chunk's end lie behind the descriptor's range and read as zero, without a branch per load.
  // Columns of Q past C read whatever follows inside the range (their sums are dropped), columns of P past 3 r are not fetched.
  // Rows so far apart that 32 bits do not span a tile take guarded loads.
  constexpr int kQTasks = kGradGroups * (kGradCols / 2) / 256, kPTasks = kGradGroups * (kGradPCols / 2) / 256;
  uint32_t qreg[kQTasks][8], preg[kPTasks][8];
  const uint16_t* const Q = jb.Q;
  const uint16_t* const P = jb.P;
  const int64_t q_ld = jb.q_ld, p_ld = jb.p_ld;
  const bool far = q_ld >= (int64_t)1 << 24;
  const uint32_t q_row = (uint32_t)q_ld * 2, p_row = (uint32_t)p_ld * 2;
  const int p_pairs = 3 * r / 2;
  uint32_t q_off[kQTasks], p_off[kPTasks];
  int p_slot[kPTasks];
#pragma unroll
  for (int i = 0; i < kQTasks; ++i) {
    const int idx = tid + 256 * i;
    q_off[i] = (uint32_t)(idx >> 6) * 8 * q_row + (uint32_t)(idx & 63) * 4;
  }
#pragma unroll
  for (int i = 0; i < kPTasks; ++i) {
    const int idx = tid + 256 * i, g = idx / p_pairs, pair = idx - g * p_pairs;
    p_off[i] = g < kGradGroups ? (uint32_t)g * 8 * p_row + (uint32_t)pair * 4 : 0x80000000u;   // past any range
    p_slot[i] = g < kGradGroups ? g * kGradPCols + 2 * pair : -1;
  }
  auto request = [&](int64_t m0) {
    const int64_t left = m_hi - m0;
    const uint32_t rows = left <= 0 ? 0u : (uint32_t)(left < kGradTokens ? left : kGradTokens);
    const int64_t mb = rows ? m0 : m_lo;
    if (far) {
#pragma unroll
      for (int i = 0; i < kQTasks; ++i) {
        const int idx = tid + 256 * i, g = 8 * (idx >> 6);
        const int64_t c = c0 + 2 * (idx & 63);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          qreg[i][e] = 0u;
          if ((uint32_t)(g + e) < rows && c < C) qreg[i][e] = *reinterpret_cast<const uint32_t*>(Q + (mb + g + e) * q_ld + c);
        }
      }
    } else {
      const uint32_t bytes = rows ? (rows - 1) * q_row + (uint32_t)(C - c0 < kGradCols ? C - c0 : kGradCols) * 2 : 0u;
      const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(Q + mb * q_ld + c0), 0, (int)bytes, 0x00027000);
#pragma unroll
      for (int i = 0; i < kQTasks; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) qreg[i][e] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)(q_off[i] + e * q_row), 0, 0);
    }
    const uint32_t bytes = rows ? (rows - 1) * p_row + (uint32_t)r * 6 : 0u;
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(P + mb * p_ld), 0, (int)bytes, 0x00027000);
#pragma unroll
    for (int i = 0; i < kPTasks; ++i)
#pragma unroll
      for (int e = 0; e < 8; ++e) preg[i][e] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)(p_off[i] + e * p_row), 0, 0);
  };
  auto turn = [](const uint32_t (&v)[8], u32x4* to) {   // eight tokens of two columns -> two operands
    u32x4 a, b;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      a[e] = __builtin_amdgcn_perm(v[2 * e + 1], v[2 * e], 0x05040100u);
      b[e] = __builtin_amdgcn_perm(v[2 * e + 1], v[2 * e], 0x07060302u);
    }
    to[0] = a;
    to[1] = b;
  };
  request(m_lo);
  for (int64_t m0 = m_lo; m0 < m_hi; m0 += kGradTokens) {
    __syncthreads();                   // the previous tile has been read
#pragma unroll
    for (int i = 0; i < kQTasks; ++i) turn(qreg[i], sQ + 2 * (tid + 256 * i));
#pragma unroll
    for (int i = 0; i < kPTasks; ++i)
      if (p_slot[i] >= 0) turn(preg[i], sP + p_slot[i]);
    __syncthreads();
    request(m0 + kGradTokens);         // past the chunk's end every guard fails: zeros, no access
    f32x16 tile[2];
#pragma unroll
    for (int jt = 0; jt < 2; ++jt)
#pragma unroll
      for (int i = 0; i < 16; ++i) tile[jt][i] = 0.f;
#pragma unroll
    for (int ks = 0; ks < kGradTokens / 16; ++ks) {
      const int g = 2 * ks + kg;       // this lane's eight tokens of the step
      const bf16x8 af = __builtin_bit_cast(bf16x8, sQ[g * kGradCols + wave * 32 + n32]);
#pragma unroll
      for (int jt = 0; jt < 2; ++jt) {
        const int j = jt * 32 + n32;
        if (jt * 32 < r) {             // uniform
#pragma unroll
          for (int t = 0; t < 3; ++t) {
            u32x4 b = sP[g * kGradPCols + t * r + (j < r ? j : 0)];
            if (j >= r) b = u32x4{0u, 0u, 0u, 0u};
            const bf16x8 bf = __builtin_bit_cast(bf16x8, b);
            f32x16& acc = t == 0 ? tile[jt] : small[jt];
            if constexpr (RANK_MAJOR) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf, af, acc, 0, 0, 0);
            else acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af, bf, acc, 0, 0, 0);
          }
        }
      }
    }
#pragma unroll
    for (int jt = 0; jt < 2; ++jt)
#pragma unroll
      for (int i = 0; i < 16; ++i) sum[jt][i] += tile[jt][i];
  }
#pragma unroll
  for (int jt = 0; jt < 2; ++jt)
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const float v = (sum[jt][q] + small[jt][q]) * mult;
      const int inner = 8 * (q >> 2) + 4 * kg + (q & 3);     // MFMA result: row inner, column n32
      const int j = jt * 32 + (RANK_MAJOR ? inner : n32);
      const int64_t c = c0 + wave * 32 + (RANK_MAJOR ? n32 : inner);
      if (c < C && j < r) dst[RANK_MAJOR ? j * C + c : c * r + j] = v;
    }
}

// two workgroups per CU: without the bound the registers of lora_grad_block's sums leave one
__global__ __launch_bounds__(256, 2) void lora_grad_kernel(const GradArgs a) {
  __shared__ u32x4 sQ[kGradGroups * kGradCols];
  __shared__ u32x4 sP[kGradGroups * kGradPCols];
  int ji = 0;
#pragma unroll
  for (int i = 1; i < 2 * kMaxGroup; ++i) ji = i < a.n && (int)blockIdx.x >= a.job[i].block0 ? i : ji;
  const GradJob jb = a.job[ji];
  const int b = (int)blockIdx.x - jb.block0, chunk = b / jb.col_blocks;
  const int64_t c0 = (int64_t)(b - chunk * jb.col_blocks) * kGradCols;
  const int64_t m_lo = chunk * jb.tokens_per_chunk;
  const int64_t m_hi = m_lo + jb.tokens_per_chunk < a.M ? m_lo + jb.tokens_per_chunk : a.M;
  // the three-term values carry lora_scale / S32, the gradients want lora_scale: one multiplication by S32, here if there is
  // one chunk, behind the sum of the chunks otherwise
  const bool last = jb.n_chunks == 1;
  float* dst = last ? jb.out : jb.partial + chunk * (jb.C * jb.r);
  const float mult = last ? *jb.mult : 1.f;
  if (jb.rank_major) lora_grad_block<true>(jb, c0, m_lo, m_hi, mult, dst, sQ, sP);
  else lora_grad_block<false>(jb, c0, m_lo, m_hi, mult, dst, sQ, sP);
}

typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));   // the results are only known to lie on four bytes
// out = S32 * sum over chunks (in chunk order) of every product with more than one
__global__ __launch_bounds__(256) void lora_grad_reduce_kernel(const GradArgs a) {
  // four consecutive elements per thread: C r is a multiple of eight
  for (int64_t i = 4 * ((int64_t)blockIdx.x * 256 + threadIdx.x); i < a.elems; i += 4 * (int64_t)gridDim.x * 256) {
    int ji = 0;
#pragma unroll
    for (int k = 1; k < 2 * kMaxGroup; ++k) ji = k < a.n && i >= a.job[k].elem0 ? k : ji;
    const GradJob& jb = a.job[ji];
    const int64_t e = i - jb.elem0, stride = jb.C * jb.r;
    const float* src = jb.partial + e;
    f32x4 v[kGradChunksMax];
#pragma unroll
    for (int z = 0; z < kGradChunksMax; ++z) {
      v[z] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (z < jb.n_chunks) v[z] = *reinterpret_cast<const f32x4*>(src + z * stride);
    }
    const float mult = *jb.mult;
    f32x4_any out;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      float sum = v[0][k];
#pragma unroll
      for (int z = 1; z < kGradChunksMax; ++z) sum += v[z][k];
      out[k] = sum * mult;
    }
    *reinterpret_cast<f32x4_any*>(jb.out + e) = out;
  }
}

static size_t al256(size_t v) { return (v + 255) & ~(size_t)255; }
// Workspace of a backward call over n members that read the same x: the arrival counters of the K-split
// down-projections, then per member A^T, B^T and the two three-term products, then one area that first holds the
// down-projections' K-part sums and later the partial sums of the gradient products.  The area holds the widest product in
// the most chunks there can be (grad_split never takes more than kGradChunksMax, nor more than one per 64 tokens), so that
// every product fits and the size never falls when M, a width or a rank grows, which the chunk counts themselves do (8 at
// 512 tokens, 5 at 513): a buffer sized for the largest call serves the smaller ones.  Products that do not fit
// together take more than one launch.
struct BackwardMemberLayout { size_t at_off, bt_off, tsu_off, tst_off; int64_t ts_ld; int ext_stages; };
struct BackwardLayout { size_t ctr_off, part_off, part_bytes, total; BackwardMemberLayout mem[kMaxGroup]; };
static BackwardLayout backward_layout(int64_t M, int64_t K, const int64_t* Ns, const int64_t* rs, int n) {
  BackwardLayout L{};
  const size_t m = (size_t)(M > 0 ? M : 1), k = (size_t)(K > 0 ? K : 1);
  L.ctr_off = 0;                                   // zeroed by every call
  size_t off = al256(kDownMaxSlots * sizeof(uint32_t));
  size_t widest = 0;
  bool any = false;
  for (int i = 0; i < n; ++i) {
    const size_t nn = (size_t)(Ns[i] > 0 ? Ns[i] : 1), rr = (size_t)(rs[i] > 0 ? rs[i] : 0);
    BackwardMemberLayout& b = L.mem[i];
    b.ext_stages = (int)ceil_div(3 * (int64_t)rr, 64);
    b.ts_ld = (int64_t)b.ext_stages * 64;
    b.at_off = off;  off += al256(k * rr * 2);
    b.bt_off = off;  off += al256(nn * rr * 2);
    b.tsu_off = off; off += al256(m * (size_t)b.ts_ld * 2);
    b.tst_off = off; off += al256(m * (size_t)b.ts_ld * 2);
    if (rr) { any = true; widest = widest > nn ? widest : nn; }
  }
  L.part_off = off;
  if (any) {
    widest = widest > k ? widest : k;
    size_t chunks = (m + kGradTokens - 1) / kGradTokens;
    chunks = chunks < (size_t)kGradChunksMax ? chunks : (size_t)kGradChunksMax;
    L.part_bytes = al256(chunks * widest * kGradRanks * sizeof(float));
    if (L.part_bytes < kDownExchangeBytes) L.part_bytes = kDownExchangeBytes;
  }
  L.total = L.part_off + L.part_bytes;
  return L;
}
static int grid_for(int64_t items) {
  int64_t b = ceil_div(items, 256);
  return (int)(b < 1 ? 1 : (b > 8192 ? 8192 : b));
}

struct BackwardMember {
  const uint16_t* dy; int64_t lddy; int64_t N; const uint8_t* packed_t; const float* tensor_scale;
  const uint16_t* A; const uint16_t* B; int64_t r; float lora_scale; float* dA; float* dB;
};

static int backward_validate(const void* x, int64_t M, int64_t K, int64_t ldx, const BackwardMember* mem, int n, const void* dx, int64_t lddx) {
  if (n < 1 || n > kMaxGroup) return QERL_ERR_SHAPE;
  if (M < 0 || K < 0 || K % kBlock != 0 || ldx < K || lddx < K) return QERL_ERR_SHAPE;
  bool any = false;
  for (int i = 0; i < n; ++i) {
    const BackwardMember& b = mem[i];
    if (b.N < 0 || b.r < 0 || b.N % 8 != 0 || b.lddy < b.N || b.r > kGradRanks || b.r % 8 != 0) return QERL_ERR_SHAPE;
    any = any || b.r > 0;
  }
  if (M == 0) return 1;   // nothing to do
  if (K == 0) return QERL_ERR_SHAPE;
  for (int i = 0; i < n; ++i) if (mem[i].N == 0) return QERL_ERR_SHAPE;
  if (!dx) return QERL_ERR_NULL;
  if (any && !x) return QERL_ERR_NULL;
  for (int i = 0; i < n; ++i) {
    const BackwardMember& b = mem[i];
    if (!b.dy || !b.packed_t || !b.tensor_scale) return QERL_ERR_NULL;
    if (b.r > 0 && (!b.A || !b.B || !b.dA || !b.dB)) return QERL_ERR_NULL;
  }
  if (!aligned(dx, 2)) return QERL_ERR_ALIGN;
  if (any && (!aligned(x, 16) || ldx % 8 != 0)) return QERL_ERR_ALIGN;
  for (int i = 0; i < n; ++i) {
    const BackwardMember& b = mem[i];
    if (!aligned(b.dy, 16) || b.lddy % 8 != 0 || !aligned(b.packed_t, 16)) return QERL_ERR_ALIGN;
    if (b.r > 0 && (!aligned(b.A, 16) || !aligned(b.B, 16) || !aligned(b.dA, 4) || !aligned(b.dB, 4))) return QERL_ERR_ALIGN;
  }
  return QERL_OK;
}

// A call's launches: one that transposes all adapters, per member a down-projection of its own dY, the
// down-projections of x (one launch over all adapters), dX -- ONE GEMM whose contraction runs over the members' rows one
// after the other, so that dX is summed in fp32 and rounded once -- and one or two for the gradient products of all
// members, or as often as their partial sums fill the area.
static int backward_run(const uint16_t* x, int64_t M, int64_t K, int64_t ldx, const BackwardMember* mem, int n, uint16_t* dx, int64_t lddx,
                        void* workspace, size_t workspace_bytes, hipStream_t st) {
  int64_t Ns[kMaxGroup], rs[kMaxGroup];
  for (int i = 0; i < n; ++i) { Ns[i] = mem[i].N; rs[i] = mem[i].r; }
  const BackwardLayout L = backward_layout(M, K, Ns, rs, n);
  if (!workspace || !aligned(workspace, 256) || workspace_bytes < L.total) return QERL_ERR_WORKSPACE;
  uint8_t* ws = (uint8_t*)workspace;
  uint32_t* counters = (uint32_t*)(ws + L.ctr_off);
  float* part = (float*)(ws + L.part_off);
  int rc = QERL_OK;
  GemmArgs down{};   // t_i = x A_i^T of all adapters, one launch
  down.x = x; down.ldx = ldx; down.M = M; down.K = K; down.k_tiles = ceil_div(K, kPackTileK);
  down.tpart = (uint32_t*)part; down.counters = counters;
  PrepareArgs prep{};
  for (int i = 0; i < n; ++i) {
    const BackwardMember& b = mem[i];
    if (b.r == 0) continue;
    const BackwardMemberLayout& l = L.mem[i];
    prep.job[prep.n++] = TransposeJob{b.A, (uint16_t*)(ws + l.at_off), b.r, K, prep.n_blocks};
    prep.n_blocks += (int)(ceil_div(b.r, 64) * ceil_div(K, 64));
    prep.job[prep.n++] = TransposeJob{b.B, (uint16_t*)(ws + l.bt_off), b.N, b.r, prep.n_blocks};
    prep.n_blocks += (int)(ceil_div(b.N, 64) * ceil_div(b.r, 64));
  }
  if (prep.n > 0) {
    prep.counters = counters;
    prep.n_counters = kDownMaxSlots;
    backward_prepare_kernel<<<dim3((unsigned)(prep.n_blocks + 1)), dim3(256), 0, st>>>(prep);
    if ((rc = launch_status()) != QERL_OK) return rc;
  }
  int tiles = 0;
  for (int i = 0; i < n; ++i) {
    const BackwardMember& b = mem[i];
    if (b.r == 0) continue;
    const BackwardMemberLayout& l = L.mem[i];
    uint16_t* BT = (uint16_t*)(ws + l.bt_off);
    // U_i = dY_i B_i as three bf16 terms of (lora_scale / S32) times the product
    GemmArgs d{};
    d.x = b.dy; d.ldx = b.lddy; d.M = M; d.K = b.N; d.k_tiles = ceil_div(b.N, kPackTileK);
    d.N = b.r; d.wbf16 = BT; d.n_tiles = (int)ceil_div(b.r, 32); d.ts = (const uint16_t*)(ws + l.tsu_off); d.ts_ld = l.ts_ld; d.ext_stages = l.ext_stages;
    d.r = (int)b.r; d.lora_scale = b.lora_scale; d.tensor_scale = b.tensor_scale;
    d.tpart = (uint32_t*)part; d.counters = counters;   // K split over workgroups while token blocks alone do not fill the chip
    if ((rc = launch_lora_down_gemm(d, st)) != QERL_OK) return rc;
    const int gi = down.g_n++;
    down.g_tile0[gi] = tiles; down.g_A[gi] = b.A; down.g_ts[gi] = (const uint16_t*)(ws + l.tst_off); down.g_ts_ld[gi] = l.ts_ld;
    down.g_r[gi] = (int)b.r; down.g_lora_scale[gi] = b.lora_scale; down.g_tensor_scale[gi] = b.tensor_scale;
    tiles += (int)ceil_div(b.r, 32);
  }
  if (down.g_n > 0) {
    down.g_tile0[down.g_n] = tiles;
    if ((rc = launch_lora_down_gemm(down, st)) != QERL_OK) return rc;
  }
  {
    GemmArgs g{};
    g.M = M; g.N = K; g.n_tiles = (int)ceil_div(K, 32); g.y = dx; g.ldy = lddx; g.transposed = 1;
    g.seg_n = n;
    int64_t rows = 0;
    for (int i = 0; i < n; ++i) {
      const BackwardMember& b = mem[i];
      const BackwardMemberLayout& l = L.mem[i];
      GemmSeg& sgm = g.seg[i];
      sgm.x = b.dy; sgm.ldx = b.lddy; sgm.K = b.N; sgm.packed = b.packed_t; sgm.k_tiles = ceil_div(b.N, kPackTileK);
      sgm.tensor_scale = b.tensor_scale;
      if (b.r > 0) {
        sgm.ts = (const uint16_t*)(ws + l.tsu_off); sgm.ts_ld = l.ts_ld; sgm.ext_stages = l.ext_stages;
        sgm.B = (const uint16_t*)(ws + l.at_off); sgm.r = (int)b.r;
      }
      rows += b.N;
    }
    // the launcher's own fields describe the first segment (it validates them; the kernel reads the segments)
    g.x = g.seg[0].x; g.ldx = g.seg[0].ldx; g.K = rows; g.k_tiles = g.seg[0].k_tiles; g.packed = g.seg[0].packed; g.tensor_scale = g.seg[0].tensor_scale;
    if ((rc = launch_gemm(g, st)) != QERL_OK) return rc;
  }
  // The gradient products; the down-projections are done with the area, and a launch's sums with it before the next one writes.
  GradArgs grad{};
  grad.M = M;
  size_t used = 0;
  auto launch_grads = [&]() -> int {
    lora_grad_kernel<<<dim3((unsigned)grad.n_blocks), dim3(256), 0, st>>>(grad);
    int status = launch_status();
    if (status == QERL_OK && grad.elems > 0) {
      lora_grad_reduce_kernel<<<dim3((unsigned)grid_for(ceil_div(grad.elems, 4))), dim3(256), 0, st>>>(grad);
      status = launch_status();
    }
    grad.n = grad.n_blocks = 0;
    grad.elems = 0;
    used = 0;
    return status;
  };
  for (int i = 0; i < 2 * n; ++i) {
    const BackwardMember& b = mem[i / 2];
    if (b.r == 0) continue;
    const BackwardMemberLayout& l = L.mem[i / 2];
    const bool da = i % 2 == 0;        // dA = U^T x as [r, K], then dB = dY^T t as [N, r]
    const int64_t C = da ? K : b.N;
    const GradSplit sp = grad_split(M, C);
    const size_t bytes = sp.n_chunks > 1 ? (size_t)sp.n_chunks * (size_t)(C * b.r) * sizeof(float) : 0;   // a multiple of 256
    if (used + bytes > L.part_bytes && (rc = launch_grads()) != QERL_OK) return rc;
    const int cols = (int)ceil_div(C, kGradCols);
    grad.job[grad.n++] = GradJob{(const uint16_t*)(ws + (da ? l.tsu_off : l.tst_off)), l.ts_ld, da ? x : b.dy, da ? ldx : b.lddy, C, (int)b.r, da,
                                 b.tensor_scale, da ? b.dA : b.dB, sp.n_chunks, sp.tokens_per_chunk, cols, grad.n_blocks, part + used / sizeof(float), grad.elems};
    grad.n_blocks += cols * sp.n_chunks;
    if (bytes > 0) grad.elems += C * b.r;
    used += bytes;
  }
  if (grad.n > 0) rc = launch_grads();
  return rc;
}

}  // namespace qerl

using namespace qerl;

extern "C" size_t nvfp4_prepack_t_bytes(int64_t N, int64_t K) {
  if (N <= 0 || K <= 0) return 0;
  return (size_t)ceil_div(K, 32) * (size_t)ceil_div(N, 128) * kPackTileBytes;
}

extern "C" int nvfp4_prepack_t(const uint8_t* codes, const uint8_t* scales, int64_t N, int64_t K, void* packed_t, void* stream) {
  if (N < 0 || K < 0 || K % kBlock != 0) return QERL_ERR_SHAPE;
  if (N == 0 || K == 0) return QERL_OK;
  if (!codes || !scales || !packed_t) return QERL_ERR_NULL;
  if (!aligned(packed_t, 16)) return QERL_ERR_ALIGN;
  const int64_t kt = ceil_div(K, 32), nt = ceil_div(N, 128);
  prepack_t_kernel<<<dim3((unsigned)grid_for(kt * nt * 128)), dim3(256), 0, (hipStream_t)stream>>>(codes, scales, N, K, kt, nt, (uint8_t*)packed_t);
  return launch_status();
}

extern "C" size_t nvfp4_lora_linear_backward_workspace_bytes(int64_t M, int64_t N, int64_t K, int64_t r) {
  const size_t t = backward_layout(M, K, &N, &r, 1).total;
  return t ? t : 256;
}

extern "C" int nvfp4_lora_linear_backward(const void* x, const void* dy, int64_t M, int64_t K, int64_t N, int64_t ldx, int64_t lddy,
                                          const void* packed_t, const float* tensor_scale, const void* A, const void* B,
                                          int64_t r, float lora_scale, void* dx, int64_t lddx, float* dA, float* dB,
                                          void* workspace, size_t workspace_bytes, void* stream) {
  const BackwardMember b{(const uint16_t*)dy, lddy, N, (const uint8_t*)packed_t, tensor_scale, (const uint16_t*)A, (const uint16_t*)B, r, lora_scale, dA, dB};
  const int vr = backward_validate(x, M, K, ldx, &b, 1, dx, lddx);
  if (vr != QERL_OK) return vr > 0 ? QERL_OK : vr;
  return backward_run((const uint16_t*)x, M, K, ldx, &b, 1, (uint16_t*)dx, lddx, workspace, workspace_bytes, (hipStream_t)stream);
}

extern "C" size_t nvfp4_lora_linear_backward_group_workspace_bytes(int64_t M, int64_t K, const qerl_backward_desc* members, int n_members) {
  if (!members || n_members < 1 || n_members > kMaxGroup) return 0;
  int64_t Ns[kMaxGroup], rs[kMaxGroup];
  for (int i = 0; i < n_members; ++i) { Ns[i] = members[i].N; rs[i] = members[i].r; }
  const size_t t = backward_layout(M, K, Ns, rs, n_members).total;
  return t ? t : 256;
}

extern "C" int nvfp4_lora_linear_backward_group(const void* x, int64_t M, int64_t K, int64_t ldx, const qerl_backward_desc* members,
                                                int n_members, void* dx, int64_t lddx, void* workspace, size_t workspace_bytes, void* stream) {
  if (!members) return QERL_ERR_NULL;
  if (n_members < 1 || n_members > kMaxGroup) return QERL_ERR_SHAPE;
  BackwardMember b[kMaxGroup];
  for (int i = 0; i < n_members; ++i) {
    const qerl_backward_desc& d = members[i];
    b[i] = BackwardMember{(const uint16_t*)d.dy_bf16, d.lddy, d.N, (const uint8_t*)d.packed_t, d.tensor_scale, (const uint16_t*)d.A_bf16,
                          (const uint16_t*)d.B_bf16, d.r, d.lora_scale, d.dA_f32, d.dB_f32};
  }
  const int vr = backward_validate(x, M, K, ldx, b, n_members, dx, lddx);
  if (vr != QERL_OK) return vr > 0 ? QERL_OK : vr;
  return backward_run((const uint16_t*)x, M, K, ldx, b, n_members, (uint16_t*)dx, lddx, workspace, workspace_bytes, (hipStream_t)stream);
}
