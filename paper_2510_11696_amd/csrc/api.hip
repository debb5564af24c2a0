// C-ABI entry points that are not kernels themselves: status strings, the
// sigma schedule, workspace layout and the dispatch of nvfp4_lora_linear.
#include <math.h>
#include "linear.hpp"

namespace qerl {

static thread_local int g_last_hip_error = 0;
void set_last_hip_error(int e) { g_last_hip_error = e; }

// Workspace layout of one linear call (offsets in bytes, all 256-aligned):
//   [0, ctrl_bytes)     arrival counters (uint32): main tiles, then LoRA-down tiles
//   [t_off, ...)        t = x A^T, fp32 [M, r]
//   [partial_off, ...)  split-K partial tiles, fp32
struct WorkspaceLayout { size_t ctrl_bytes, n_main_ctr, n_down_ctr, t_off, partial_off, total; };

constexpr size_t kDecodeTpartWords = 16 * 16 * 256;   // producer partial sums of the fused LoRA down-projection: <= 16 producers x 16 tokens x stacked rank <= 256
constexpr size_t kMaxCounterTiles = 16384;   // rows / 16 the control region can serve

static size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

// The control region has a FIXED size and position (linear.hpp) so that calls of different shapes can share one
// workspace: no call's data region may overlap another call's control words (they must stay zero).
constexpr size_t kCtrlBytes = kCtrlRegionBytes;

// 17..128 tokens: room for the sums of linear_panel.hip (eight times the outputs in fp32, capped, and a little for t); calls of 9..16 tokens and
// of more than 128 place them where the other kernels of these counts have their scratch, or do not take those kernels
static size_t panel_area_bytes(int64_t M, int64_t N) {
  const size_t b = (size_t)8 * (size_t)(M > 0 ? M : 1) * (size_t)(N > 0 ? N : 1) * sizeof(float);
  return align256(b < kPanelSumsCap ? b : kPanelSumsCap) + kPanelTBytes;
}

static WorkspaceLayout workspace_layout(int64_t M, int64_t N, int64_t K, int64_t r) {
  WorkspaceLayout L;
  L.n_main_ctr = kCtrlMainWords;
  const size_t n_down_ctr = (size_t)ceil_div(r > 0 ? r : 1, 16);
  L.n_down_ctr = kCtrlDownWords;
  L.ctrl_bytes = kCtrlBytes;
  L.t_off = L.ctrl_bytes;
  // t = x A^T: fp32 [M, r] for the decode kernels, or three bf16 terms [M, ceil64(3r)] for the GEMM
  const size_t rows = (size_t)(M > 0 ? M : 1), rr = (size_t)(r > 0 ? r : 1);
  const size_t t_f32 = rows * rr * sizeof(float), t_split = rows * (size_t)(ceil_div(3 * rr, 128) + kMaxGroup - 1) * 128 * 2;   // each member of a group pads its 3r columns to 128
  const size_t t_bytes = align256(t_f32 > t_split ? t_f32 : t_split);
  L.partial_off = L.t_off + t_bytes;
  // worst case over the plans the dispatchers can choose (one K-tile per wave)
  const size_t S_max = (size_t)ceil_div(ceil_div(K > 0 ? K : 1, 256), 8);
  const size_t S_down = (size_t)ceil_div(ceil_div(K > 0 ? K : 1, 256), 2) + 1;
  const size_t n_rows16 = (size_t)ceil_div(N > 0 ? N : 1, 16);
  const size_t skinny_bytes = (S_max * n_rows16 + S_down * n_down_ctr) * 64 * sizeof(f32x4);
  const size_t S_dec = (size_t)ceil_div(ceil_div(K > 0 ? K : 1, kPackTileK), 7);
  const size_t decode_bytes = S_dec * (size_t)ceil_div(N > 0 ? N : 1, kPackTileRows) * 8 * 64 * sizeof(float) +
                              S_down * n_down_ctr * 64 * sizeof(f32x4) + kDecodeTpartWords * sizeof(uint32_t);
  size_t need = skinny_bytes > decode_bytes ? skinny_bytes : decode_bytes;
  if (M > 16 && M <= 128) {
    const size_t panel = panel_area_bytes(M, N);
    need = need > panel ? need : panel;
  }
  if (M > 128 && need < kDownExchangeBytes) need = kDownExchangeBytes;   // K-parts of the prefill path's LoRA down-projection
  if (M > 16) {
    // the GEMM path: a down-projection launched by itself has the whole area for its K-part
    // sums and is through with it when the GEMM starts; one that rides inside the GEMM launch needs the first
    // kFusedDownBytes at most, and the GEMM's own K-parts start behind them
    size_t g = kFusedDownBytes + gemm_split_bytes(M, N);
    g = g > kDownExchangeBytes ? g : kDownExchangeBytes;
    need = need > g ? need : g;
  }
  L.total = L.partial_off + align256(need);
  return L;
}
size_t linear_need_bytes(int64_t M, int64_t N, int64_t K, int64_t r) { return workspace_layout(M, N, K, r).total; }

// What the size function answers: the call's own need (all that a call is checked against), and from 17 tokens on the areas that
// fewer tokens or rows take and this call does not, so that a buffer for the largest call holds every smaller one.
static size_t linear_bytes_of_largest(int64_t M, int64_t N, int64_t K, int64_t r) {
  const WorkspaceLayout L = workspace_layout(M, N, K, r);
  if (M <= 16) return L.total;
  const size_t panel = panel_area_bytes(M < 128 ? M : 128, N);
  size_t g = gemm_split_bytes(M, N);
  if (g == 0 && N > 0) g = kGemmSplitCap;        // tiles enough to fill the chip; a smaller call may split K up to the cap
  g += kFusedDownBytes;
  const size_t most = L.partial_off + align256(panel > g ? panel : g);
  return most > L.total ? most : L.total;
}

// act[m, k] = bf16(bf16(SiLU(gate[m, k])) * up[m, k]), eight values per thread
__global__ __launch_bounds__(256) void silu_mul_kernel(const uint16_t* __restrict__ gate, int64_t ldg, const uint16_t* __restrict__ up,
                                                       int64_t ldu, int64_t M, int64_t K, uint16_t* __restrict__ act) {
  const int64_t chunks = K / 8, total = M * chunks;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
    const int64_t m = i / chunks, c = i - m * chunks;
    const u32x4 g = *reinterpret_cast<const u32x4*>(gate + m * ldg + c * 8);
    const u32x4 u = *reinterpret_cast<const u32x4*>(up + m * ldu + c * 8);
    *reinterpret_cast<u32x4*>(act + m * K + c * 8) = silu_mul8(g, u);
  }
}

__global__ void zero_words_kernel(uint32_t* p, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    p[i] = 0u;
}

}  // namespace qerl

using namespace qerl;

extern "C" const char* qerl_status_string(int status) {
  switch (status) {
    case QERL_OK: return "ok";
    case QERL_ERR_NULL: return "a required pointer is NULL";
    case QERL_ERR_SHAPE: return "invalid shape or leading dimension";
    case QERL_ERR_ALIGN: return "pointer or leading dimension not aligned as required";
    case QERL_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case QERL_ERR_LAUNCH: return "HIP runtime error at launch (see qerl_last_hip_error)";
    case QERL_ERR_TIMEOUT: return "a kernel's bounded wait on another workgroup gave up: results unreliable, re-initialise the workspace";
    default: return "unknown status";
  }
}

extern "C" int qerl_last_hip_error(void) { return g_last_hip_error; }

extern "C" double aqn_sigma(int k, int num_stages, double s0, double s1) {
  if (num_stages < 1 || k < 0 || k > num_stages) return NAN;
  if (k == 0) return 0.0;
  if (num_stages == 1) return s0;
  return s0 * pow(s1 / s0, (double)(k - 1) / (double)(num_stages - 1));
}

extern "C" size_t nvfp4_lora_linear_workspace_bytes(int64_t M, int64_t N, int64_t K, int64_t r) {
  return linear_bytes_of_largest(M, N, K, r);
}

extern "C" int qerl_workspace_init(void* workspace, size_t bytes, void* stream) {
  if (!workspace) return QERL_ERR_NULL;
  if (!aligned(workspace, 256)) return QERL_ERR_ALIGN;
  // the control region is a prefix; clearing the whole buffer keeps this independent of shapes
  const size_t words = bytes / 4;
  if (words == 0) return QERL_OK;
  size_t nb = (words + 255) / 256;
  if (nb > 4096) nb = 4096;
  zero_words_kernel<<<(int)nb, 256, 0, (hipStream_t)stream>>>((uint32_t*)workspace, words);
  return launch_status();
}

namespace qerl {

struct LinearCall {
  const uint16_t* x; int64_t M, K, ldx; const float* tensor_scale; int64_t N;
  const uint16_t* A; const uint16_t* B; int64_t r; float lora_scale; uint16_t* y; int64_t ldy;
  void* workspace; size_t workspace_bytes; hipStream_t st;
};

// Checks shared by the canonical and the packed entry point.
static int validate(const LinearCall& c, const void* w0, const void* w1) {
  if (c.M < 0 || c.N < 0 || c.K < 0 || c.r < 0 || c.K % kBlock != 0 || c.ldx < c.K || c.ldy < c.N)
    return QERL_ERR_SHAPE;
  if (c.N / 16 >= (int64_t)kMaxCounterTiles || c.r > 4096) return QERL_ERR_SHAPE;
  if (c.M == 0 || c.N == 0) return 1;   // nothing to do
  if (!c.x || !c.y || !c.tensor_scale) return QERL_ERR_NULL;
  if (c.K > 0 && (!w0 || !w1)) return QERL_ERR_NULL;
  if (c.r > 0 && (!c.A || !c.B)) return QERL_ERR_NULL;
  if (!aligned(c.x, 2) || !aligned(c.y, 2) || (c.r > 0 && (!aligned(c.A, 2) || !aligned(c.B, 2))))
    return QERL_ERR_ALIGN;
  const WorkspaceLayout L = workspace_layout(c.M, c.N, c.K, c.r);
  if (!c.workspace || !aligned(c.workspace, 256) || c.workspace_bytes < L.total) return QERL_ERR_WORKSPACE;
  return QERL_OK;
}

// t[m0 .. m0+mc) = x A^T for one pass of at most 16 tokens.
static int lora_down_pass(const LinearCall& c, const WorkspaceLayout& L, int64_t m0, int mc, f32x4* partial) {
  uint8_t* ws = (uint8_t*)c.workspace;
  float* t = (float*)(ws + L.t_off) + m0 * c.r;
  const bool tiled = (c.K % 64 == 0) && aligned(c.x, 16) && c.ldx % 8 == 0 && aligned(c.A, 16);
  if (!tiled) return launch_generic_lora_down(c.x + m0 * c.ldx, c.ldx, mc, c.K, c.A, c.r, t, c.st);
  const SkinnyPlan pd = plan_skinny(c.r, c.K, kFmtBf16);
  SkinnyArgs d{};
  d.x = c.x + m0 * c.ldx; d.ldx = c.ldx; d.M = mc; d.K = c.K;
  d.N = c.r; d.wbf16 = c.A; d.t_out = t;
  d.partial = partial; d.counters = (uint32_t*)ws + L.n_main_ctr; d.n_tiles = pd.n_tiles;
  return launch_skinny(pd, d, kFmtBf16, c.st);
}

}  // namespace qerl

extern "C" int nvfp4_lora_linear(const void* x, int64_t M, int64_t K, int64_t ldx, const uint8_t* codes,
                                 const uint8_t* scales, const float* tensor_scale, int64_t N,
                                 const void* A, const void* B, int64_t r, float lora_scale, void* y,
                                 int64_t ldy, void* workspace, size_t workspace_bytes, void* stream) {
  LinearCall c{(const uint16_t*)x, M, K, ldx, tensor_scale, N, (const uint16_t*)A, (const uint16_t*)B, r,
               lora_scale, (uint16_t*)y, ldy, workspace, workspace_bytes, (hipStream_t)stream};
  const int vr = validate(c, codes, scales);
  if (vr != QERL_OK) return vr > 0 ? QERL_OK : vr;
  if (K == 0) c.r = r = 0;   // empty sums: y = 0 through the general kernel
  const WorkspaceLayout L = workspace_layout(M, N, K, r);
  uint8_t* ws = (uint8_t*)workspace;
  float* t = (float*)(ws + L.t_off);
  f32x4* partial = (f32x4*)(ws + L.partial_off);

  // The tiled kernels use 16-byte loads; anything else goes to the general kernels.
  const bool tiled = (K % 64 == 0) && K > 0 && aligned(x, 16) && ldx % 8 == 0 && aligned(codes, 16) &&
                     aligned(scales, 4) && (r == 0 || aligned(A, 16));
  if (!tiled) {
    int rc = QERL_OK;
    if (r > 0) rc = launch_generic_lora_down(c.x, ldx, M, K, c.A, r, t, c.st);
    if (rc != QERL_OK) return rc;
    return launch_generic_linear(c.x, ldx, M, K, codes, scales, tensor_scale, N, r > 0 ? t : nullptr, c.B, r,
                                 lora_scale, c.y, ldy, c.st);
  }

  // Tiled path on the canonical layout: passes of up to 16 tokens.
  const SkinnyPlan pm = plan_skinny(N, K, kFmtNvfp4);
  for (int64_t m0 = 0; m0 < M; m0 += 16) {
    const int mc = (int)((M - m0 < 16) ? M - m0 : 16);
    if (r > 0) {
      const int rc = lora_down_pass(c, L, m0, mc, partial + (size_t)pm.S * pm.n_tiles * 64);
      if (rc != QERL_OK) return rc;
    }
    SkinnyArgs a{};
    a.x = c.x + m0 * ldx; a.ldx = ldx; a.M = mc; a.K = K;
    a.N = N; a.codes = codes; a.scales = scales; a.tensor_scale = tensor_scale;
    a.t_in = t + m0 * r; a.B = c.B; a.r = (int)r; a.lora_scale = lora_scale;
    a.y = c.y + m0 * ldy; a.ldy = ldy;
    a.y_vec = aligned(y, 8) && ldy % 4 == 0;
    a.b_vec = r % 8 == 0 && aligned(B, 16);
    a.partial = partial; a.counters = (uint32_t*)ws; a.n_tiles = pm.n_tiles;
    const int rc = launch_skinny(pm, a, kFmtNvfp4, c.st);
    if (rc != QERL_OK) return rc;
  }
  return QERL_OK;
}

namespace qerl {
static bool g_use_stream = true;
// From here to 128 tokens linear_panel.hip takes the packed linears (to kPanelMaxTokens where it is estimated faster than the GEMM).  Whole layers, us per layer, the 1..16-token kernels / the
// panel kernels: 9 tokens 106 / 93 (7B shapes), 125 / 101 (14B), 140 / 131 (32B); 8 tokens 91 / 93, 108 / 101, 122 / 130 (the
// decode kernels' cost follows the tokens in steps of eight, the panel kernels' in steps of 32).
constexpr int64_t kPanelMinTokens = 9;

// One streaming launch for a group of packed linears sharing x (M <= 16; every r in {0} or 8..64 step 8): its plan.
static int stream_plan(StreamArgs& a, size_t* lds, int* MR, const uint16_t* x, int64_t M, int64_t K, int64_t ldx, const qerl_linear_desc* d, int n,
                       const uint16_t* x2 = nullptr, int64_t ldx2 = 0) {
  a = StreamArgs{};
  a.x = x; a.ldx = ldx; a.M = (int)M; a.K = K; a.k_tiles = (int)ceil_div(K, kPackTileK);
  a.x2 = x2; a.ldx2 = ldx2;
  a.n_members = n;
  int tiles = 0, rt = 0, any = 0;
  for (int i = 0; i < n; ++i) {
    StreamMember& m = a.mem[i];
    m.packed = (const uint8_t*)d[i].packed; m.tensor_scale = d[i].tensor_scale;
    m.A = (const uint16_t*)d[i].A_bf16; m.B = (const uint16_t*)d[i].B_bf16; m.y = (uint16_t*)d[i].y_bf16;
    m.ldy = d[i].ldy; m.N = d[i].N; m.n_tiles = (int)ceil_div(d[i].N, kPackTileRows); m.tile_begin = tiles;
    m.r = (int)d[i].r; m.lora_scale = d[i].lora_scale;
    m.y_vec = aligned(d[i].y_bf16, 16) && d[i].ldy % 8 == 0;
    m.t_ext = m.r > 0 ? d[i].t_f32 : nullptr;
    m.bias = (const uint16_t*)d[i].bias_bf16;
    m.t_off = 0x7fffffff;                 // not part of the producers' stack ...
    if (m.r > 0 && !m.t_ext) { m.t_off = rt; rt += m.r; }   // ... unless the launch has to compute its t
    any |= m.r > 0;
    a.any_bias |= m.bias != nullptr;
    tiles += m.n_tiles;
  }
  for (int i = n; i < kMaxGroup; ++i) {   // unused entries: never selected, but valid to read
    a.mem[i] = a.mem[0];
    a.mem[i].tile_begin = 0x7fffffff; a.mem[i].n_tiles = 0; a.mem[i].r = 0; a.mem[i].t_off = 0x7fffffff; a.mem[i].t_ext = nullptr;
  }
  a.tb1 = a.mem[1].tile_begin; a.tb2 = a.mem[2].tile_begin; a.tb3 = a.mem[3].tile_begin;
  a.mp0 = a.mem[0].packed; a.mp1 = a.mem[1].packed; a.mp2 = a.mem[2].packed; a.mp3 = a.mem[3].packed;
  a.total_tiles = tiles; a.r_total = rt; a.any_lora = any;
  if (rt > 0) {
    int64_t np = ceil_div(2 * (int64_t)a.k_tiles, 8);   // one half K-tile per producer wave and tile pair
    a.n_producers = (int)(np < 1 ? 1 : (np > 16 ? 16 : np));
  }
  return plan_stream(a, lds, MR);
}
// need != null: nothing is launched, *need = the bytes of the workspace that the launch would touch.
static int stream_group(const uint16_t* x, int64_t M, int64_t K, int64_t ldx, const qerl_linear_desc* d, int n,
                        uint8_t* ws, const WorkspaceLayout& L, hipStream_t st, const uint16_t* x2 = nullptr, int64_t ldx2 = 0, size_t* need = nullptr) {
  StreamArgs a;
  size_t lds = 0;
  int MR = 4;
  const int prc = stream_plan(a, &lds, &MR, x, M, K, ldx, d, n, x2, ldx2);
  if (prc != QERL_OK) return prc;
  uint32_t* partial = (uint32_t*)(ws + L.partial_off);
  const size_t part_words = a.Sk > 1 ? ((size_t)a.Sk * a.total_tiles * MR * 64 + 3) & ~(size_t)3 : 0;
  if (need) {
    *need = align256(L.partial_off + (part_words + (a.r_total > 0 ? kDecodeTpartWords : 0)) * sizeof(uint32_t));
    return QERL_OK;
  }
  a.partial = partial; a.counters = (uint32_t*)ws;
  a.t = (float*)(ws + L.t_off);
  a.lora_ctl = (uint32_t*)ws + L.n_main_ctr + L.n_down_ctr;
  a.tpart = partial + part_words;
  return launch_stream(a, lds, MR, st);
}

// The GEMM launch and the LoRA down-projections it depends on (dn: the group form, tiles rank tiles; g_n == 0: none).
// launch_gemm either takes the down-projections into its own launch (few tokens) or runs them first; the scratch
// serves the down-projection's K-parts from its front and the GEMM's own K-parts from kFusedDownBytes on (inside
// one launch both are alive at once, and the down-projection stays below that mark).
static int gemm_with_down(GemmArgs& g, GemmArgs& dn, int tiles, int64_t n_sum, uint8_t* ws, const WorkspaceLayout& L, hipStream_t st, double* estimate_us) {
  if (dn.g_n > 0) {
    dn.g_tile0[dn.g_n] = tiles;
    g.g_n = dn.g_n;
    for (int i = 0; i <= dn.g_n; ++i) g.g_tile0[i] = dn.g_tile0[i];
    for (int i = 0; i < dn.g_n; ++i) {
      g.g_A[i] = dn.g_A[i]; g.g_ts[i] = dn.g_ts[i]; g.g_ts_ld[i] = dn.g_ts_ld[i]; g.g_r[i] = dn.g_r[i];
      g.g_lora_scale[i] = dn.g_lora_scale[i]; g.g_tensor_scale[i] = dn.g_tensor_scale[i];
    }
    g.tpart = (uint32_t*)(ws + L.partial_off); g.counters = (uint32_t*)ws + L.n_main_ctr;   // K-parts while token blocks alone do not fill the chip
    g.ready = (uint32_t*)ws + L.n_main_ctr + L.n_down_ctr;                                   // the hand-over words (zero between calls)
    g.done = g.ready + 2;
    g.n_prod = -1;                                                                           // not run yet: the launcher's to place
  }
  g.kpartial = (float*)(ws + L.partial_off + kFusedDownBytes); g.kpartial_bytes = gemm_split_bytes(g.M, n_sum);
  g.estimate_us = estimate_us;
  return launch_gemm(g, st);
}

// More than 128 tokens: one launch of the LoRA down-projection for all adapters of the group, then
// one GEMM launch whose column blocks run over all members (k and v alone would fill half the chip).
static int gemm_group(const uint16_t* x, int64_t M, int64_t K, int64_t ldx, const qerl_linear_desc* d, int n,
                      uint8_t* ws, const WorkspaceLayout& L, hipStream_t st, double* estimate_us = nullptr) {
  GemmArgs g{};
  g.x = x; g.ldx = ldx; g.M = M; g.K = K; g.k_tiles = ceil_div(K, kPackTileK); g.m_n = n;
  GemmArgs dn{};
  dn.x = x; dn.ldx = ldx; dn.M = M; dn.K = K; dn.k_tiles = g.k_tiles;
  uint16_t* ts = (uint16_t*)(ws + L.t_off);
  int tiles = 0;
  for (int i = 0; i < n; ++i) {
    GemmMember& m = g.m[i];
    m.packed = (const uint8_t*)d[i].packed; m.tensor_scale = d[i].tensor_scale; m.N = d[i].N;
    m.n_tiles = (int)ceil_div(d[i].N, kPackTileRows);
    m.r = (int)d[i].r; m.B = (const uint16_t*)d[i].B_bf16; m.y = (uint16_t*)d[i].y_bf16; m.ldy = d[i].ldy;
    m.bias = (const uint16_t*)d[i].bias_bf16;
    m.ext_stages = (int)ceil_div(3 * d[i].r, 64); m.ts_ld = (int64_t)m.ext_stages * 64; m.ts = ts;
    ts += M * m.ts_ld;
    if (d[i].r > 0) {
      const int gi = dn.g_n++;
      dn.g_tile0[gi] = tiles; dn.g_A[gi] = (const uint16_t*)d[i].A_bf16; dn.g_ts[gi] = m.ts; dn.g_ts_ld[gi] = m.ts_ld;
      dn.g_r[gi] = (int)d[i].r; dn.g_lora_scale[gi] = d[i].lora_scale; dn.g_tensor_scale[gi] = d[i].tensor_scale;
      tiles += (int)ceil_div(d[i].r, 32);
    }
  }
  int64_t n_sum = 0;
  for (int i = 0; i < n; ++i) n_sum += d[i].N;
  return gemm_with_down(g, dn, tiles, n_sum, ws, L, st, estimate_us);
}
// 9..128 tokens, one linear or a group reading the same x, in one or two launches (linear_panel.hip); up to 64 tokens, where the sums
// of all rows do not fit the workspace's area, the rows in several parts of two launches each.  act != null: members 0 and 1 are
// gate_proj and up_proj and act = SiLU(gate) (.) up is stored instead of their outputs.
// Beyond 128 tokens the same kernels take several token blocks, where they are estimated faster than the GEMM: launches of few
// rows, whose tiles do not fill the chip (5120 x 5120, r = 64, 256 tokens 49 -> 30 us, 3584 x 18944, r = 32, 777 tokens 216 -> 135).
// QERL_ERR_SHAPE: not a shape for it (nothing has been launched).
// need (M <= 128): as in stream_group.
static int panel_group(const uint16_t* x, int64_t M, int64_t K, int64_t ldx, const qerl_linear_desc* d, int n, uint8_t* ws,
                       const WorkspaceLayout& L, uint16_t* act, hipStream_t st, size_t* need = nullptr) {
  const int64_t k_tiles = ceil_div(K, kPackTileK);
  auto part = [&](int c, int parts, PanelArgs& a) {
    a = PanelArgs{};
    a.x = x; a.ldx = ldx; a.M = (int)M; a.K = K; a.n_members = n;
    for (int i = 0; i < n; ++i) {
      PanelMember& m = a.mem[i];
      const int64_t tiles = ceil_div(d[i].N, kPackTileRows), t0 = tiles * c / parts, t1 = tiles * (c + 1) / parts, row0 = t0 * kPackTileRows;
      m.packed = (const uint8_t*)d[i].packed + t0 * k_tiles * kPackTileBytes; m.tensor_scale = d[i].tensor_scale;
      m.N = (t1 * kPackTileRows < d[i].N ? t1 * kPackTileRows : d[i].N) - row0;
      m.A = (const uint16_t*)d[i].A_bf16; m.r = (int)d[i].r; m.lora_scale = d[i].lora_scale;
      m.B = d[i].r > 0 ? (const uint16_t*)d[i].B_bf16 + row0 * d[i].r : nullptr;
      m.bias = d[i].bias_bf16 ? (const uint16_t*)d[i].bias_bf16 + row0 : nullptr;
      m.y = d[i].y_bf16 ? (uint16_t*)d[i].y_bf16 + row0 : nullptr; m.ldy = d[i].ldy;
      if (act && i == 0) { a.pairs = 1; a.act = act + row0; a.ld_act = d[0].N; }
    }
    return plan_panel(a, (float*)(ws + L.partial_off), L.total - L.partial_off);
  };
  PanelArgs a;
  if (M > 128) {
    double gemm_us = 0;
    if (part(0, 1, a) != QERL_OK || gemm_group(x, M, K, ldx, d, n, ws, L, st, &gemm_us) != QERL_OK) return QERL_ERR_SHAPE;
    if (act) gemm_us += 5.0 + 6.0 * (double)M * (double)d[0].N / 5.0e6;   // and the elementwise pass
    return panel_estimate_us(a) < gemm_us ? launch_panel(a, st) : QERL_ERR_SHAPE;
  }
  int64_t tiles = 0, r_max = 0;
  bool bias = false;
  for (int i = 0; i < n; ++i) {
    tiles += ceil_div(d[i].N, kPackTileRows);
    r_max = d[i].r > r_max ? d[i].r : r_max;
    bias = bias || (d[i].bias_bf16 && d[i].r > 64);
  }
  // Where the sums do not fit at once, the other kernels of the token count are faster than several pairs of launches: the decode
  // kernels (r = 32, 9 tokens: 8192 x 512 13.1 us against 17.0), beyond 64 tokens the GEMM (151936 x 3584, r = 16, 100 tokens 165 / 227;
  // at 64 tokens 155 / 122).  Beyond 64 tokens and K = 512 many rows are the GEMM's as well: writing and reading the sums
  // takes longer than the product (50000 x 512, r = 16, 100 tokens 22 / 30; 40000 x 1024 30 / 32).
  const bool one_part = part(0, 1, a) == QERL_OK;
  if (M > 64 && (!one_part || (K <= 512 && tiles > 1024))) return QERL_ERR_SHAPE;
  if (M <= 16 && !bias) {   // (the decode kernels take no bias with more than 64 ranks)
    if (!one_part) return QERL_ERR_SHAPE;
    if (!act && r_max <= 64) {
      // The streaming kernel is faster where every CU would have more than one unit of some length and it need not split K (two of 18944 x
      // 3584, r = 32, 9..16 tokens 25 us against 30; 40000 x 5120, r = 16, 9 tokens 31 / 33, but 40000 x 1024, four stages, 20 / 18, and
      // at 12 tokens 40000 x 5120, K in two ranges, 39 / 34), and
      // without adapters wherever the panel kernels need their second launch (4096 x 4096, 16 tokens 9.9 / 11.4, 13824 x 5120 in one 17 / 13).
      StreamArgs sa;
      size_t lds = 0;
      int MR = 4;
      if (a.rank_tiles == 0 && !a.direct) return QERL_ERR_SHAPE;
      if (a.units > 256 && (a.rank_tiles == 0 || a.stages >= 8) && stream_plan(sa, &lds, &MR, x, M, K, ldx, d, n) == QERL_OK && sa.Sk == 1) return QERL_ERR_SHAPE;
    }
  }
  for (int parts = 1; parts <= 64 && parts <= tiles; parts *= 2) {   // (ranks whose sums alone exceed the area fit in no number of parts)
    bool fits = true;
    size_t used = 0;
    for (int c = 0; c < parts && fits; ++c) {
      fits = part(c, parts, a) == QERL_OK;
      used = a.used_bytes > used ? a.used_bytes : used;
    }
    if (!fits) continue;
    if (need) {
      *need = align256(L.partial_off + used);
      return QERL_OK;
    }
    for (int c = 0; c < parts; ++c) {
      int rc = part(c, parts, a);
      if (rc == QERL_OK) rc = launch_panel(a, st);
      if (rc != QERL_OK) return rc;
    }
    return QERL_OK;
  }
  return QERL_ERR_SHAPE;
}
}  // namespace qerl

#ifdef QERL_TUNING_HOOKS   // built only for tuning sessions: they change process-wide state
extern "C" QERL_API void qerl_debug_use_stream(int on) { qerl::g_use_stream = on != 0; }
#endif  // QERL_TUNING_HOOKS

static int packed_single(const void* x, int64_t M, int64_t K, int64_t ldx, const void* packed,
                         const float* tensor_scale, int64_t N, const void* A, const void* B,
                         int64_t r, float lora_scale, const void* bias, void* y, int64_t ldy, void* workspace,
                         size_t workspace_bytes, void* stream);

// act != null: members 0 and 1 are gate_proj and up_proj; act[M, N] = SiLU(gate) (.) up is stored instead of their
// outputs where the shape has a kernel for it (QERL_OK), else nothing is launched (kNoFusedAct).
// need != null: nothing is launched, *need = the bytes of the workspace that the call would touch.  exact: up to 16 tokens the workspace may
// be as small as that (a composed call has sized it), instead of what the public entry point asks for.
static int packed_group_impl(const void* x, int64_t M, int64_t K, int64_t ldx, const qerl_linear_desc* members, int n_members,
                             void* workspace, size_t workspace_bytes, uint16_t* act, void* stream, bool exact = false, size_t* need = nullptr) {
  if (!members) return QERL_ERR_NULL;
  if (n_members < 1 || n_members > kMaxGroup) return QERL_ERR_SHAPE;
  int64_t n_sum = 0, r_sum = 0;
  bool stream_ok = M <= 16, lora_ok = true, t_given = false;   // (t handed in: only the decode kernels read it)
  for (int i = 0; i < n_members; ++i) {
    const qerl_linear_desc& d = members[i];
    LinearCall c{(const uint16_t*)x, M, K, ldx, d.tensor_scale, d.N, (const uint16_t*)d.A_bf16, (const uint16_t*)d.B_bf16,
                 d.r, d.lora_scale, (uint16_t*)d.y_bf16, d.ldy, workspace, ~(size_t)0, (hipStream_t)stream};
    const int vr = validate(c, d.packed, d.packed);
    if (vr < 0) return vr;
    if (d.N < 1) return QERL_ERR_SHAPE;
    n_sum += d.N; r_sum += d.r;
    stream_ok = stream_ok && (d.r == 0 || (d.r <= 64 && d.r % 8 == 0 && aligned(d.A_bf16, 16) && aligned(d.B_bf16, 16)));
    lora_ok = lora_ok && (d.r == 0 || (d.r % 8 == 0 && aligned(d.A_bf16, 16) && aligned(d.B_bf16, 16)));
    t_given = t_given || (d.r > 0 && d.t_f32);
    if (M > 0 && !aligned(d.packed, 16)) return QERL_ERR_ALIGN;
    if (d.r > 0 && d.t_f32 && !aligned(d.t_f32, 32)) return QERL_ERR_ALIGN;
  }
  if (M == 0) return QERL_OK;
  if (K == 0) return QERL_ERR_SHAPE;
  if (!aligned(x, 16) || ldx % 8 != 0) return QERL_ERR_ALIGN;
  const WorkspaceLayout L = workspace_layout(M, n_sum, K, r_sum);
  if (need) *need = L.total;
  else if (!workspace || !aligned(workspace, 256) || (!(exact && M <= 16) && workspace_bytes < L.total)) return QERL_ERR_WORKSPACE;
  if (M > 16 && need) return QERL_OK;
  if (lora_ok && M >= kPanelMinTokens && M <= kPanelMaxTokens && (M > 16 || !t_given)) {
    const int rc = panel_group((const uint16_t*)x, M, K, ldx, members, n_members, (uint8_t*)workspace, L, act, (hipStream_t)stream, need);
    if (rc != QERL_ERR_SHAPE) return rc;
  }
  if (act) return kNoFusedAct;
  if (stream_ok && g_use_stream)
    return stream_group((const uint16_t*)x, M, K, ldx, members, n_members, (uint8_t*)workspace, L, (hipStream_t)stream, nullptr, 0, need);
  if (need) return QERL_OK;
  if (M > 16 && lora_ok && n_members > 1)
    return gemm_group((const uint16_t*)x, M, K, ldx, members, n_members, (uint8_t*)workspace, L, (hipStream_t)stream);
  for (int i = 0; i < n_members; ++i) {   // general case: member by member
    const qerl_linear_desc& d = members[i];
    const int rc = packed_single(x, M, K, ldx, d.packed, d.tensor_scale, d.N, d.A_bf16, d.B_bf16, d.r,
                                 d.lora_scale, d.bias_bf16, d.y_bf16, d.ldy, workspace, workspace_bytes, stream);
    if (rc != QERL_OK) return rc;
  }
  return QERL_OK;
}

extern "C" int nvfp4_lora_linear_packed_group(const void* x, int64_t M, int64_t K, int64_t ldx,
                                              const qerl_linear_desc* members, int n_members, void* workspace,
                                              size_t workspace_bytes, void* stream) {
  return packed_group_impl(x, M, K, ldx, members, n_members, workspace, workspace_bytes, nullptr, stream);
}

int qerl::packed_gate_up_act(const void* x, int64_t M, int64_t K, int64_t ldx, const qerl_linear_desc* gate_up, void* workspace,
                             size_t workspace_bytes, uint16_t* act, void* stream, size_t* need) {
  return packed_group_impl(x, M, K, ldx, gate_up, 2, workspace, workspace_bytes, act, stream, true, need);
}

int qerl::packed_group_exact(const void* x, int64_t M, int64_t K, int64_t ldx, const qerl_linear_desc* members, int n_members, void* workspace,
                             size_t workspace_bytes, void* stream, size_t* need) {
  return packed_group_impl(x, M, K, ldx, members, n_members, workspace, workspace_bytes, nullptr, stream, true, need);
}

// SiLU(gate) (.) up formed while the streaming kernel stages its input: M <= 16, the adapter as the decode kernels take it
int qerl::packed_swiglu_exact(const void* gate, const void* up, int64_t M, int64_t K, const qerl_linear_desc* down, void* workspace,
                              size_t workspace_bytes, void* stream, size_t* need) {
  LinearCall c{(const uint16_t*)gate, M, K, K, down->tensor_scale, down->N, (const uint16_t*)down->A_bf16, (const uint16_t*)down->B_bf16, down->r,
               down->lora_scale, (uint16_t*)down->y_bf16, down->ldy, workspace, ~(size_t)0, (hipStream_t)stream};
  if (!need) {
    const int vr = validate(c, down->packed, down->packed);
    if (vr != QERL_OK) return vr > 0 ? QERL_OK : vr;
  }
  const WorkspaceLayout L = workspace_layout(M, down->N, K, down->r);
  return stream_group(c.x, M, K, K, down, 1, (uint8_t*)workspace, L, c.st, (const uint16_t*)up, K, need);
}

extern "C" size_t nvfp4_prepack_bytes(int64_t N, int64_t K) {
  if (N <= 0 || K <= 0) return 0;
  return (size_t)ceil_div(N, kPackTileRows) * (size_t)ceil_div(K, kPackTileK) * kPackTileBytes;
}

extern "C" int nvfp4_prepack(const uint8_t* codes, const uint8_t* scales, int64_t N, int64_t K, void* packed,
                             void* stream) {
  if (N < 0 || K < 0 || K % kBlock != 0) return QERL_ERR_SHAPE;
  if (N == 0 || K == 0) return QERL_OK;
  if (!codes || !scales || !packed) return QERL_ERR_NULL;
  if (!aligned(packed, 16)) return QERL_ERR_ALIGN;
  return launch_prepack(codes, scales, N, K, (uint8_t*)packed, (hipStream_t)stream);
}

extern "C" int nvfp4_lora_linear_packed(const void* x, int64_t M, int64_t K, int64_t ldx, const void* packed,
                                        const float* tensor_scale, int64_t N, const void* A, const void* B,
                                        int64_t r, float lora_scale, void* y, int64_t ldy, void* workspace,
                                        size_t workspace_bytes, void* stream) {
  return packed_single(x, M, K, ldx, packed, tensor_scale, N, A, B, r, lora_scale, nullptr, y, ldy, workspace,
                       workspace_bytes, stream);
}

extern "C" size_t nvfp4_lora_linear_swiglu_workspace_bytes(int64_t M, int64_t N, int64_t K, int64_t r) {
  return linear_bytes_of_largest(M, N, K, r) + align256((size_t)(M > 0 ? M : 0) * (size_t)(K > 0 ? K : 0) * sizeof(uint16_t));
}

extern "C" int nvfp4_lora_linear_packed_swiglu(const void* gate, const void* up, int64_t M, int64_t K, int64_t ldg, int64_t ldu,
                                               const void* packed, const float* tensor_scale, int64_t N, const void* A,
                                               const void* B, int64_t r, float lora_scale, void* y, int64_t ldy,
                                               void* workspace, size_t workspace_bytes, void* stream) {
  LinearCall c{(const uint16_t*)gate, M, K, ldg, tensor_scale, N, (const uint16_t*)A, (const uint16_t*)B, r,
               lora_scale, (uint16_t*)y, ldy, workspace, ~(size_t)0, (hipStream_t)stream};
  const int vr = validate(c, packed, packed);
  if (vr != QERL_OK) return vr > 0 ? QERL_OK : vr;
  if (K == 0 || ldu < K) return QERL_ERR_SHAPE;
  if (!up) return QERL_ERR_NULL;
  if (!aligned(packed, 16) || !aligned(gate, 16) || ldg % 8 != 0 || !aligned(up, 16) || ldu % 8 != 0) return QERL_ERR_ALIGN;
  const WorkspaceLayout L = workspace_layout(M, N, K, r);
  const size_t act_bytes = align256((size_t)M * (size_t)K * sizeof(uint16_t));
  if (!workspace || !aligned(workspace, 256) || workspace_bytes < L.total + act_bytes) return QERL_ERR_WORKSPACE;
  uint8_t* ws = (uint8_t*)workspace;
  if (g_use_stream && M <= 16 && (r == 0 || (r <= 64 && r % 8 == 0 && aligned(A, 16) && aligned(B, 16)))) {
    // decode: the product is formed while the kernel stages its input; no intermediate tensor
    qerl_linear_desc d{packed, tensor_scale, N, A, B, r, lora_scale, y, ldy, nullptr, nullptr};
    return stream_group(c.x, M, K, ldg, &d, 1, ws, L, c.st, (const uint16_t*)up, ldu);
  }
  // more tokens: one elementwise pass into the workspace, then the linear on it
  uint16_t* act = (uint16_t*)(ws + L.total);
  const int64_t total = M * (K / 8);
  int64_t blocks = ceil_div(total, 256);
  blocks = blocks > 4096 ? 4096 : blocks;
  silu_mul_kernel<<<dim3((unsigned)blocks), dim3(256), 0, c.st>>>(c.x, ldg, (const uint16_t*)up, ldu, M, K, act);
  const int rc = launch_status();
  if (rc != QERL_OK) return rc;
  return packed_single(act, M, K, K, packed, tensor_scale, N, A, B, r, lora_scale, nullptr, y, ldy, workspace, L.total, stream);
}

static int packed_single(const void* x, int64_t M, int64_t K, int64_t ldx, const void* packed,
                         const float* tensor_scale, int64_t N, const void* A, const void* B,
                         int64_t r, float lora_scale, const void* bias, void* y, int64_t ldy, void* workspace,
                         size_t workspace_bytes, void* stream) {
  LinearCall c{(const uint16_t*)x, M, K, ldx, tensor_scale, N, (const uint16_t*)A, (const uint16_t*)B, r,
               lora_scale, (uint16_t*)y, ldy, workspace, workspace_bytes, (hipStream_t)stream};
  const int vr = validate(c, packed, packed);
  if (vr != QERL_OK) return vr > 0 ? QERL_OK : vr;
  if (K == 0) return QERL_ERR_SHAPE;
  if (!aligned(packed, 16) || !aligned(x, 16) || ldx % 8 != 0) return QERL_ERR_ALIGN;
  const WorkspaceLayout L = workspace_layout(M, N, K, r);
  uint8_t* ws = (uint8_t*)workspace;
  float* t = (float*)(ws + L.t_off);
  uint32_t* partial = (uint32_t*)(ws + L.partial_off);

  const bool lora_gemm_ok = r == 0 || (r % 8 == 0 && aligned(A, 16) && aligned(B, 16));
  if (M >= kPanelMinTokens && M <= kPanelMaxTokens && lora_gemm_ok) {
    qerl_linear_desc d{packed, tensor_scale, N, A, B, r, lora_scale, y, ldy, nullptr, bias};
    const int rc = panel_group(c.x, M, K, ldx, &d, 1, ws, L, nullptr, c.st);
    if (rc != QERL_ERR_SHAPE) return rc;
  }
  if (M > 16 && lora_gemm_ok) {
    // Prefill: one split-K GEMM writes lora_scale * x A^T as three bf16 terms into the workspace,
    // then one GEMM computes the layer with those 3r columns appended to K.
    GemmArgs g{};
    g.x = c.x; g.ldx = ldx; g.M = M; g.K = K; g.k_tiles = ceil_div(K, kPackTileK);
    g.ts = (const uint16_t*)(ws + L.t_off); g.ext_stages = (int)ceil_div(3 * r, 64); g.ts_ld = (int64_t)g.ext_stages * 64;
    g.r = (int)r; g.lora_scale = lora_scale; g.tensor_scale = tensor_scale;
    GemmArgs dn{};
    int tiles = 0;
    if (r > 0) {
      dn.g_n = 1;
      dn.g_tile0[0] = 0; dn.g_A[0] = c.A; dn.g_ts[0] = g.ts; dn.g_ts_ld[0] = g.ts_ld; dn.g_r[0] = (int)r;
      dn.g_lora_scale[0] = lora_scale; dn.g_tensor_scale[0] = tensor_scale;
      tiles = (int)ceil_div(r, 32);
    }
    g.N = N; g.packed = (const uint8_t*)packed; g.n_tiles = (int)ceil_div(N, 32);
    g.B = c.B; g.y = c.y; g.ldy = ldy; g.bias = (const uint16_t*)bias;
    return gemm_with_down(g, dn, tiles, N, ws, L, c.st, nullptr);
  }

  if (g_use_stream && M <= 16 && (r == 0 || (r <= 64 && r % 8 == 0 && aligned(A, 16) && aligned(B, 16)))) {
    qerl_linear_desc d{packed, tensor_scale, N, A, B, r, lora_scale, y, ldy, nullptr, bias};
    return stream_group(c.x, M, K, ldx, &d, 1, ws, L, c.st);
  }
  if (bias) return QERL_ERR_SHAPE;   // the remaining kernels (adapters of unusual rank or alignment) add no bias

  // Decode: passes of up to 16 tokens.  For the usual adapters (r <= 64, 16-byte aligned) the LoRA
  // down-projection runs on the first workgroups of the same launch; otherwise it gets a launch of its own.
  const bool fused_lora = r > 0 && r <= 64 && r % 8 == 0 && aligned(A, 16) && aligned(B, 16);
  for (int64_t m0 = 0; m0 < M; m0 += 16) {
    const int mc = (int)((M - m0 < 16) ? M - m0 : 16);
    const DecodePlan p = plan_decode(mc, N, K, r);
    const size_t dec_words = ((size_t)p.S * p.n_tiles * p.MR * 64 + 3) & ~(size_t)3;
    if (r > 0 && !fused_lora) {
      const int rc = lora_down_pass(c, L, m0, mc, (f32x4*)(partial + dec_words + kDecodeTpartWords));
      if (rc != QERL_OK) return rc;
    }
    DecodeArgs a{};
    a.x = c.x + m0 * ldx; a.ldx = ldx; a.M = mc; a.K = K; a.N = N;
    a.packed = (const uint8_t*)packed; a.k_tiles = p.k_tiles; a.tensor_scale = tensor_scale;
    a.A = c.A; a.B = c.B; a.r = (int)r; a.lora_scale = lora_scale;
    a.b_vec = r % 8 == 0 && aligned(B, 16);
    a.t = t + m0 * r;
    if (fused_lora) {
      int64_t np = ceil_div(2 * p.k_tiles, p.waves);   // one half K-tile per producer wave
      a.n_producers = (int)(np < 1 ? 1 : (np > 16 ? 16 : np));
      a.lora_ctl = (uint32_t*)ws + L.n_main_ctr + L.n_down_ctr;
      a.tpart = partial + dec_words;
    }
    a.y = c.y + m0 * ldy; a.ldy = ldy;
    a.partial = partial; a.counters = (uint32_t*)ws; a.n_tiles = p.n_tiles; a.S = p.S; a.n_groups = p.groups;
    const int rc = launch_decode(p, a, c.st);
    if (rc != QERL_OK) return rc;
  }
  return QERL_OK;
}

// ---- nvfp4_lora_linear_packed_noalloc: the packed linear for callers that cannot allocate ----------------------
// The scratch that nvfp4_lora_linear_packed takes as its workspace argument lives here in a file-scope device
// array instead.  Each GPU holds its own copy of the array at its own address: the address is looked up once per
// device (with that device current) and only that pointer is ever handed to kernels.
namespace qerl {
constexpr size_t kNoallocScratchBytes = (size_t)36 << 20;   // covers every single linear of the five benchmark configurations (largest: 32.7 MiB)
static __device__ __align__(256) unsigned char scratch[kNoallocScratchBytes];
constexpr int kMaxDevices = 64;
static void* g_scratch_ptr[kMaxDevices];   // device address of `scratch` per device, nullptr until first used there

static int noalloc_scratch(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return launch_status();
  if (dev < 0 || dev >= kMaxDevices) return QERL_ERR_SHAPE;
  void* p = __atomic_load_n(&g_scratch_ptr[dev], __ATOMIC_ACQUIRE);
  if (!p) {
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) { set_last_hip_error((int)e); (void)hipGetLastError(); return QERL_ERR_LAUNCH; }
    __atomic_store_n(&g_scratch_ptr[dev], p, __ATOMIC_RELEASE);   // racing first calls look up the same address
  }
  *out = p;
  return QERL_OK;
}
}  // namespace qerl

extern "C" size_t nvfp4_lora_linear_packed_noalloc_max_bytes(void) { return kNoallocScratchBytes; }

extern "C" int nvfp4_lora_linear_packed_noalloc(const void* x, int64_t M, int64_t K, int64_t ldx, const void* packed,
                                                const float* tensor_scale, int64_t N, const void* A, const void* B,
                                                int64_t r, float lora_scale, void* y, int64_t ldy, void* stream) {
  // every host-side check of the ordinary entry point first, against the fixed scratch size: nothing is launched
  // and no device is touched for a call that would be rejected
  LinearCall c{(const uint16_t*)x, M, K, ldx, tensor_scale, N, (const uint16_t*)A, (const uint16_t*)B, r,
               lora_scale, (uint16_t*)y, ldy, (void*)(uintptr_t)256, kNoallocScratchBytes, (hipStream_t)stream};
  const int vr = validate(c, packed, packed);
  if (vr != QERL_OK) return vr > 0 ? QERL_OK : vr;
  if (K == 0) return QERL_ERR_SHAPE;
  if (!aligned(packed, 16) || !aligned(x, 16) || ldx % 8 != 0) return QERL_ERR_ALIGN;
  void* ws = nullptr;
  const int rc = noalloc_scratch(&ws);
  if (rc != QERL_OK) return rc;
  // The array keeps whatever the last call on this GPU left in it.  What must start at zero are the control
  // words at its front; they are cleared by a fill kernel (not a memset node, so the call can be captured).
  zero_words_kernel<<<dim3(16), dim3(256), 0, (hipStream_t)stream>>>((uint32_t*)ws, kCtrlBytes / sizeof(uint32_t));
  const int zr = launch_status();
  if (zr != QERL_OK) return zr;
  return packed_single(x, M, K, ldx, packed, tensor_scale, N, A, B, r, lora_scale, nullptr, y, ldy, ws,
                       kNoallocScratchBytes, stream);
}
