// C-ABI entry points of the fused decode launches (block_kernel, linear_block.hip):
//   aqn_rmsnorm_nvfp4_lora_linear_group  RMSNorm with noisy gain (Eq. 10) -> up to four NVFP4 + LoRA linears (Eq. 6, Eq. 2)
//   aqn_rmsnorm_nvfp4_lora_mlp           RMSNorm -> gate_proj, up_proj -> SiLU(gate) (.) up -> down_proj
// as separate launches of the same operators, or (up to 16 tokens) one launch each.
#include <stdlib.h>
#include "linear.hpp"

namespace qerl {

// Up to 16 tokens norm and linears can go out as ONE launch (block_kernel) or as separate ones: the norm with the adapters'
// down-projections, the grouped linear, the gated down projection (up to 8 tokens), the norm and the panel kernels (from 9 on).
// The separate launches are the faster ones; the one launch serves workspaces of the size that it needs alone where they need more (their
// areas are counted by the plans that run and shared by gate + up and down: up to 8 tokens that fits the one launch's size).
// Measured, us in graph replay, one launch / separate: feed-forward block 7B shapes 1 token 55 / 49, 8 tokens 59 / 52, 9 tokens 66 / 62;
// 14B 65 / 51, 67 / 55; 32B 75 / 73, 79 / 80, 89 / 94; 2048 x 5504 38 / 30, 39 / 34; norm + q + k + v
// 7B 18 / 14, 19 / 15, 23 / 18; 14B 21 / 17, 22 / 20; 32B 20 / 17, 22 / 20, 28 / 22; 2048 wide 18 / 13, 19 / 13.
constexpr int64_t kBlkPanelTokens = 9;

static size_t blk_align256(size_t v) { return (v + 255) & ~(size_t)255; }

// Workspace of a block launch: the control region every linear workspace starts with (arrival words of the tiles,
// hand-over words), the producers' partial t of up to three stages, the K-ranges' partial tiles, and room for
// intermediate activations.
struct BlkWorkspace { size_t tpart_off, tfinal_off, partial_off, act_off, total; };
static BlkWorkspace blk_workspace(size_t partial_floats, size_t act_bytes) {
  BlkWorkspace w;
  w.tpart_off = kCtrlRegionBytes;
  w.tfinal_off = w.tpart_off + blk_align256((size_t)kBlkMaxStages * kBlkTpartWords * sizeof(uint32_t));
  w.partial_off = w.tfinal_off + blk_align256((size_t)kBlkMaxStages * kBlkTfinalWords * sizeof(float));
  w.act_off = w.partial_off + blk_align256(partial_floats * sizeof(float));
  w.total = w.act_off + blk_align256(act_bytes);
  return w;
}

// One stage from the caller's descriptors.  Returns a status; checks what the kernel's indexing assumes.
static int blk_fill_stage(BlkStage& S, const void* x, int64_t K, int64_t ldx, const void* gain, const float* noise, float eps,
                          const qerl_linear_desc* const* d, int n, bool pairs) {
  if (n < 1 || n > kMaxGroup) return QERL_ERR_SHAPE;
  if (K < 16 || K % kBlock != 0 || ldx < K) return QERL_ERR_SHAPE;
  if (!x) return QERL_ERR_NULL;
  if (!aligned(x, 16) || ldx % 8 != 0) return QERL_ERR_ALIGN;
  if (gain && (!aligned(gain, 16) || (noise && !aligned(noise, 16)) || K % 8 != 0)) return QERL_ERR_ALIGN;
  S = BlkStage{};
  S.x = (const uint16_t*)x; S.ldx = ldx; S.K = K; S.k_tiles = (int)ceil_div(K, kPackTileK);
  S.gain = (const uint16_t*)gain; S.noise = gain ? noise : nullptr; S.eps = eps;
  S.n_members = n; S.pairs = pairs ? 1 : 0;
  int tiles = 0;
  for (int i = 0; i < n; ++i) {
    const qerl_linear_desc& m = *d[i];
    if (m.N < 1 || m.r < 0 || m.N / 16 >= 16384) return QERL_ERR_SHAPE;
    if (!m.packed || !m.tensor_scale) return QERL_ERR_NULL;
    if (!pairs && (!m.y_bf16 || m.ldy < m.N)) return m.y_bf16 ? QERL_ERR_SHAPE : QERL_ERR_NULL;
    if (m.r > 0 && (!m.A_bf16 || !m.B_bf16)) return QERL_ERR_NULL;
    if (!aligned(m.packed, 16) || (m.y_bf16 && !aligned(m.y_bf16, 2)) || (m.bias_bf16 && !aligned(m.bias_bf16, 2))) return QERL_ERR_ALIGN;
    if (m.r > 0 && (m.r > 64 || m.r % 8 != 0 || !aligned(m.A_bf16, 16) || !aligned(m.B_bf16, 16))) return QERL_ERR_SHAPE;
    BlkMember& b = S.mem[i];
    b.packed = (const uint8_t*)m.packed; b.tensor_scale = m.tensor_scale;
    b.A = (const uint16_t*)m.A_bf16; b.B = (const uint16_t*)m.B_bf16; b.bias = (const uint16_t*)m.bias_bf16;
    b.y = (uint16_t*)m.y_bf16; b.ldy = m.ldy; b.N = m.N; b.n_tiles = (int)ceil_div(m.N, kPackTileRows); b.tile_begin = tiles;
    b.r = (int)m.r; b.lora_scale = m.lora_scale;
    b.stride_k = kPackTileBytes; b.stride_n = (int64_t)S.k_tiles * kPackTileBytes;
#ifdef QERL_TUNING_HOOKS   // timing experiment only (the weights are NOT in that order: results are wrong)
    if (getenv("QERL_BLK_KMAJOR_TIMING")) { b.stride_n = kPackTileBytes; b.stride_k = (int64_t)b.n_tiles * kPackTileBytes; }
    if (getenv("QERL_BLK_SAMETILE_TIMING")) { b.stride_n = 0; b.stride_k = 0; }   // every unit reads one tile: no memory traffic to speak of
#endif
    b.y_vec = (m.y_bf16 && aligned(m.y_bf16, 16) && m.ldy % 8 == 0) ? 1 : 0;
    tiles += b.n_tiles;
  }
  for (int i = n; i < kMaxGroup; ++i) {   // unused entries: never selected, but valid to read
    S.mem[i] = S.mem[0];
    S.mem[i].tile_begin = 0x7fffffff; S.mem[i].n_tiles = 0; S.mem[i].r = 0;
  }
  S.total_tiles = tiles;
  S.total_v = pairs ? S.mem[0].n_tiles : tiles;
  if (pairs && (n != 2 || S.mem[0].N != S.mem[1].N)) return QERL_ERR_SHAPE;
  return QERL_OK;
}

static int blk_plan_and_launch(BlkArgs& a, uint8_t* ws, size_t ws_bytes, size_t act_bytes, bool launch, size_t* need, hipStream_t st) {
  size_t lds = 0, part = 0, ctrs = 0;
  int MR = 4;
  const int prc = plan_block(a, &lds, &MR, &part, &ctrs);
  if (prc != QERL_OK) return prc;
  if (ctrs > kCtrlMainWords) return QERL_ERR_SHAPE;
  const BlkWorkspace w = blk_workspace(part, act_bytes);
  if (need) *need = w.total;
  if (!launch) {
    // sizing call: the plan must also pass the launch's own checks (placeholder workspace pointers, nothing is launched),
    // so that a shape the kernel cannot take reports 0 bytes here rather than an error at the first call
    BlkArgs b = a;
    b.counters = b.ctl = b.tpart = (uint32_t*)(uintptr_t)256; b.tfinal = b.partial = (float*)(uintptr_t)256;
    return check_block(b, lds, MR);
  }
  if (!ws || !aligned(ws, 256) || ws_bytes < w.total) return QERL_ERR_WORKSPACE;
  a.counters = (uint32_t*)ws;
  a.ctl = (uint32_t*)ws + kCtrlMainWords + kCtrlDownWords;
  a.tpart = (uint32_t*)(ws + w.tpart_off);
  a.tfinal = (float*)(ws + w.tfinal_off);
  a.partial = (float*)(ws + w.partial_off);
  return launch_block(a, lds, MR, st);
}

// t of the adapters of up to 8 tokens, behind the other areas of a composed call
static size_t blk_t_bytes(int64_t M, const qerl_linear_desc* const* d, int n) {
  size_t b = 0;
  for (int i = 0; i < n; ++i) b += blk_align256((size_t)QERL_T_PARTS * (size_t)(M > 0 ? M : 1) * (size_t)(d[i]->r > 0 ? d[i]->r : 0) * sizeof(float));
  return b;
}
// The size functions: a buffer for M tokens holds every smaller count too (up to 16 tokens each has a plan of its own).  0: not a shape
// of the call.
template <class Need>
static size_t blk_bytes_of_largest(int64_t M, Need need_of) {
  size_t most = 0;
  if (need_of(M, &most) != QERL_OK) return 0;
  for (int64_t m = 1; m < M && m <= 16; ++m) {
    size_t need = 0;
    if (need_of(m, &need) == QERL_OK && need > most) most = need;
  }
  return most;
}
// Whether the norm's launch computes them (rows beyond 8192 it does not take: the linears do)
static bool blk_norm_with_t(int64_t M, int64_t K, const void* gain) { return gain && M < kBlkPanelTokens && K <= 8192; }
// The norm's launch: xn = aqn_rmsnorm(x), and with_t: t_i = xn A_i^T of the members with an adapter (m[i].t_f32) too.
static int blk_norm(const void* x, int64_t M, int64_t K, int64_t ldx, const void* gain, const float* noise, float eps, uint16_t* xn,
                    qerl_linear_desc* m, int n, bool with_t, uint8_t* t_area, void* stream) {
  const void* A[kMaxGroup];
  float* t[kMaxGroup];
  int64_t r[kMaxGroup];
  int na = 0;
  for (int i = 0; i < n; ++i) {
    m[i].t_f32 = nullptr;
    if (!with_t || m[i].r == 0) continue;
    A[na] = m[i].A_bf16; r[na] = m[i].r; t[na] = (float*)t_area; m[i].t_f32 = (float*)t_area;
    t_area += blk_align256((size_t)QERL_T_PARTS * (size_t)M * (size_t)m[i].r * sizeof(float));
    ++na;
  }
  if (na > 0) return aqn_rmsnorm_lora_down(x, M, K, ldx, gain, noise, eps, xn, K, A, r, t, na, stream);
  return aqn_rmsnorm(x, M, K, ldx, gain, noise, eps, xn, K, stream);
}

}  // namespace qerl

using namespace qerl;

static int group_impl(const void* x, int64_t M, int64_t K, int64_t ldx, const void* gain, const float* noise, float eps,
                      const qerl_linear_desc* members, int n, void* workspace, size_t bytes, void* stream, bool launch, size_t* need) {
  if (!members) return QERL_ERR_NULL;
  if (n < 1 || n > kMaxGroup || M < 0) return QERL_ERR_SHAPE;
  const qerl_linear_desc* d[kMaxGroup] = {};
  int64_t n_sum = 0, r_sum = 0;
  for (int i = 0; i < n; ++i) { d[i] = members + i; n_sum += members[i].N; r_sum += members[i].r; }
  if (M == 0 && launch) return QERL_OK;
  // up to 16 tokens what the launches touch, beyond what the linear is checked against; what the size function answers may be more
  const size_t xn_bytes = gain ? blk_align256((size_t)M * (size_t)K * sizeof(uint16_t)) : 0;
  const bool with_t = blk_norm_with_t(M, K, gain);
  qerl_linear_desc own[kMaxGroup];
  for (int i = 0; i < n; ++i) {   // this entry point computes t itself
    own[i] = members[i];
    own[i].t_f32 = with_t && own[i].r > 0 ? (const float*)(uintptr_t)256 : nullptr;
  }
  size_t lin = launch || M <= 16 ? linear_need_bytes(M, n_sum, K, r_sum) : nvfp4_lora_linear_workspace_bytes(M, n_sum, K, r_sum);
  if (M > 0 && M <= 16) (void)packed_group_exact((const void*)(uintptr_t)256, M, K, gain ? K : ldx, own, n, (void*)(uintptr_t)256, 0, nullptr, &lin);
  const size_t separate_bytes = lin + xn_bytes + (with_t ? blk_t_bytes(M, d, n) : 0);
  if (M <= 16) {
    BlkArgs a{};
    a.M = (int)(M > 0 ? M : 1); a.n_stages = 1;
    int rc = blk_fill_stage(a.st[0], launch ? x : (const void*)(uintptr_t)256, K, ldx, gain, noise, eps, d, n, false);
    if (rc != QERL_OK) return rc;
    if ((!gain && M < kBlkPanelTokens) || M == 0 || (launch && bytes < separate_bytes))
      return blk_plan_and_launch(a, (uint8_t*)workspace, bytes, 0, launch, need, (hipStream_t)stream);
    size_t one = 0;
    rc = blk_plan_and_launch(a, nullptr, 0, 0, false, &one, nullptr);   // shapes that the one launch does not take stay refused
    if (rc != QERL_OK) return rc;
    if (need) *need = one > separate_bytes ? one : separate_bytes;
    if (launch && bytes < one) return QERL_ERR_WORKSPACE;
  } else if (need) {
    *need = separate_bytes;
  }
  // the norm's launch (output in the workspace), then the grouped linear
  if (!launch) return QERL_OK;
  if (!workspace || !aligned(workspace, 256) || bytes < separate_bytes) return QERL_ERR_WORKSPACE;
  const void* xin = x;
  int64_t ldin = ldx;
  if (gain) {
    uint16_t* xn = (uint16_t*)((uint8_t*)workspace + lin);
    const int rc = blk_norm(x, M, K, ldx, gain, noise, eps, xn, own, n, with_t, (uint8_t*)workspace + lin + xn_bytes, stream);
    if (rc != QERL_OK) return rc;
    xin = xn; ldin = K;
  }
  return packed_group_exact(xin, M, K, ldin, own, n, workspace, lin, stream);
}

extern "C" size_t aqn_rmsnorm_nvfp4_lora_linear_group_workspace_bytes(int64_t M, int64_t K, const int64_t* Ns, const int64_t* rs, int n) {
  if (!Ns || !rs || n < 1 || n > kMaxGroup) return 0;
  qerl_linear_desc d[kMaxGroup] = {};
  for (int i = 0; i < n; ++i) {   // placeholders that pass the pointer checks; nothing is dereferenced or launched
    d[i].packed = (const void*)(uintptr_t)256; d[i].tensor_scale = (const float*)(uintptr_t)256; d[i].N = Ns[i];
    d[i].A_bf16 = (const void*)(uintptr_t)256; d[i].B_bf16 = (const void*)(uintptr_t)256; d[i].r = rs[i];
    d[i].y_bf16 = (void*)(uintptr_t)256; d[i].ldy = Ns[i];
  }
  return blk_bytes_of_largest(M, [&](int64_t m, size_t* need) {
    return group_impl(nullptr, m, K, K, (const void*)(uintptr_t)256, nullptr, 0.f, d, n, nullptr, 0, nullptr, false, need);
  });
}

extern "C" int aqn_rmsnorm_nvfp4_lora_linear_group(const void* x, int64_t M, int64_t K, int64_t ldx, const void* gain,
                                                   const float* noise, float eps, const qerl_linear_desc* members, int n_members,
                                                   void* workspace, size_t workspace_bytes, void* stream) {
  return group_impl(x, M, K, ldx, gain, noise, eps, members, n_members, workspace, workspace_bytes, stream, true, nullptr);
}

static int mlp_impl(const void* x, int64_t M, int64_t H, int64_t ldx, const void* gain, const float* noise, float eps,
                    const qerl_linear_desc* gate, const qerl_linear_desc* up, const qerl_linear_desc* down,
                    void* workspace, size_t bytes, void* stream, bool launch, size_t* need) {
  if (!gate || !up || !down) return QERL_ERR_NULL;
  if (M < 0 || gate->N != up->N || gate->N < 1) return QERL_ERR_SHAPE;
  const int64_t I = gate->N;
  if (I % 8 != 0) return QERL_ERR_SHAPE;             // act rows are staged with 16-byte accesses
  if (M == 0 && launch) return QERL_OK;
  if (launch && (!down->y_bf16 || down->ldy < down->N)) return down->y_bf16 ? QERL_ERR_SHAPE : QERL_ERR_NULL;
  const size_t act_bytes = blk_align256((size_t)(M > 0 ? M : 1) * (size_t)I * sizeof(uint16_t));
  const size_t xn_bytes = gain ? blk_align256((size_t)M * (size_t)H * sizeof(uint16_t)) : 0;
  const bool with_t = blk_norm_with_t(M, H, gain);
  void* const ph = (void*)(uintptr_t)256;            // for plans: checked, never read
  qerl_linear_desc gu[2] = {*gate, *up};
  for (qerl_linear_desc& m : gu) { m.y_bf16 = ph; m.ldy = I; m.t_f32 = with_t && m.r > 0 ? (const float*)ph : nullptr; }
  // gate + up, then down, in the same area: up to 16 tokens what their launches touch, beyond what the linears are checked against
  // (what the size function answers may be more)
  const bool answer = !launch && M > 16;
  size_t lin_gu = answer ? nvfp4_lora_linear_workspace_bytes(M, 2 * I, H, gate->r + up->r) : linear_need_bytes(M, 2 * I, H, gate->r + up->r);
  size_t lin_dn = (answer ? nvfp4_lora_linear_workspace_bytes(M, down->N, I, down->r) : linear_need_bytes(M, down->N, I, down->r)) + act_bytes;
  bool fused = false;                                // SiLU(gate) (.) up from one launch: neither gate nor up is stored
  if (M > 0 && M <= 16) {
    const int64_t ldin = gain ? H : ldx;
    fused = packed_gate_up_act(ph, M, H, ldin, gu, ph, 0, (uint16_t*)ph, nullptr, &lin_gu) == QERL_OK;
    if (!fused) (void)packed_group_exact(ph, M, H, ldin, gu, 2, ph, 0, nullptr, &lin_gu);
    qerl_linear_desc dn = *down;
    dn.y_bf16 = ph; dn.ldy = down->N; dn.t_f32 = nullptr;
    if (fused) (void)packed_group_exact(ph, M, I, I, &dn, 1, ph, 0, nullptr, &lin_dn);
    else (void)packed_swiglu_exact(ph, ph, M, I, &dn, ph, 0, nullptr, &lin_dn);
  }
  const size_t lin = lin_gu > lin_dn ? lin_gu : lin_dn;
  const qerl_linear_desc* gu_d[2] = {gate, up};
  const size_t separate_bytes = lin + xn_bytes + (fused ? 1 : 2) * act_bytes + (with_t ? blk_t_bytes(M, gu_d, 2) : 0);
  const bool separate = M > 0 && !down->bias_bf16 && (!launch || bytes >= separate_bytes);
  if (M <= 16) {
    BlkArgs a{};
    a.M = (int)(M > 0 ? M : 1); a.n_stages = 2;
    int rc = blk_fill_stage(a.st[0], launch ? x : (const void*)(uintptr_t)256, H, ldx, gain, noise, eps, gu_d, 2, true);
    if (rc != QERL_OK) return rc;
    // the activation's place is known once the plan (size of the partial tiles) is: plan with a placeholder first
    const qerl_linear_desc* dn[1] = {down};
    rc = blk_fill_stage(a.st[1], (const void*)(uintptr_t)256, I, I, nullptr, nullptr, 0.f, dn, 1, false);
    if (rc != QERL_OK) return rc;
    a.st[0].act = (uint16_t*)(uintptr_t)256; a.st[0].ld_act = I; a.st[0].act_vec = 1;
    size_t lds = 0, part = 0, ctrs = 0;
    int MR = 4;
    rc = plan_block(a, &lds, &MR, &part, &ctrs);
    if (rc != QERL_OK) return rc;
    if (ctrs > kCtrlMainWords) return QERL_ERR_SHAPE;
    const BlkWorkspace w = blk_workspace(part, act_bytes);
    if (need) *need = separate && separate_bytes > w.total ? separate_bytes : w.total;
    if (!launch) return QERL_OK;
    uint8_t* ws = (uint8_t*)workspace;
    if (!ws || !aligned(ws, 256) || bytes < w.total) return QERL_ERR_WORKSPACE;
    if (!separate) {
      uint16_t* act = (uint16_t*)(ws + w.act_off);
      a.st[0].act = act; a.st[1].x = act;
      a.counters = (uint32_t*)ws;
      a.ctl = (uint32_t*)ws + kCtrlMainWords + kCtrlDownWords;
      a.tpart = (uint32_t*)(ws + w.tpart_off);
      a.tfinal = (float*)(ws + w.tfinal_off);
      a.partial = (float*)(ws + w.partial_off);
      return launch_block(a, lds, MR, (hipStream_t)stream);
    }
  }
  // norm, grouped gate + up, down on the gated input, as separate launches; the intermediates live in
  // the workspace behind the linear's own area
  if (need) *need = separate_bytes;
  if (!launch) return QERL_OK;
  uint8_t* ws = (uint8_t*)workspace;
  if (!ws || !aligned(ws, 256) || bytes < separate_bytes) return QERL_ERR_WORKSPACE;
  const void* xin = x;
  int64_t ldin = ldx;
  gu[0].y_bf16 = ws + lin + xn_bytes;
  gu[1].y_bf16 = ws + lin + xn_bytes + act_bytes;   // (not written where act comes from one launch)
  if (gain) {
    uint16_t* xn = (uint16_t*)(ws + lin);
    const int rc = blk_norm(x, M, H, ldx, gain, noise, eps, xn, gu, 2, with_t, ws + lin + xn_bytes + 2 * act_bytes, stream);
    if (rc != QERL_OK) return rc;
    xin = xn; ldin = H;
  }
  uint16_t* act = (uint16_t*)(ws + lin + xn_bytes);   // gate's place: the fused form stores no gate
  qerl_linear_desc dn = *down;
  dn.t_f32 = nullptr;
  int rc = M > 16 || fused ? packed_gate_up_act(xin, M, H, ldin, gu, ws, lin, act, stream) : kNoFusedAct;
  if (rc == QERL_OK) {
    if (down->bias_bf16) return QERL_ERR_SHAPE;
    if (M <= 16) return packed_group_exact(act, M, I, I, &dn, 1, ws, lin, stream);
    return nvfp4_lora_linear_packed(act, M, I, I, down->packed, down->tensor_scale, down->N, down->A_bf16, down->B_bf16, down->r,
                                    down->lora_scale, down->y_bf16, down->ldy, ws, lin, stream);
  }
  if (rc != kNoFusedAct) return rc;
  rc = packed_group_exact(xin, M, H, ldin, gu, 2, ws, lin, stream);   // (beyond 16 tokens as nvfp4_lora_linear_packed_group)
  if (rc != QERL_OK) return rc;
  if (down->bias_bf16) return QERL_ERR_SHAPE;   // (the gated entry point takes no bias)
  if (M <= 16) return packed_swiglu_exact(gu[0].y_bf16, gu[1].y_bf16, M, I, &dn, ws, lin, stream);
  return nvfp4_lora_linear_packed_swiglu(gu[0].y_bf16, gu[1].y_bf16, M, I, I, I, down->packed, down->tensor_scale, down->N,
                                         down->A_bf16, down->B_bf16, down->r, down->lora_scale, down->y_bf16, down->ldy, ws, lin, stream);
}

extern "C" size_t aqn_rmsnorm_nvfp4_lora_mlp_workspace_bytes(int64_t M, int64_t H, int64_t I, int64_t N_down, int64_t r_gate,
                                                             int64_t r_up, int64_t r_down) {
  const void* ph = (const void*)(uintptr_t)256;
  qerl_linear_desc g{}, u{}, d{};
  g.packed = ph; g.tensor_scale = (const float*)ph; g.N = I; g.A_bf16 = ph; g.B_bf16 = ph; g.r = r_gate;
  u = g; u.r = r_up;
  d = g; d.N = N_down; d.r = r_down; d.y_bf16 = (void*)(uintptr_t)256; d.ldy = N_down;
  return blk_bytes_of_largest(M, [&](int64_t m, size_t* need) {
    return mlp_impl(nullptr, m, H, H, ph, nullptr, 0.f, &g, &u, &d, nullptr, 0, nullptr, false, need);
  });
}

extern "C" int aqn_rmsnorm_nvfp4_lora_mlp(const void* x, int64_t M, int64_t H, int64_t ldx, const void* gain, const float* noise,
                                          float eps, const qerl_linear_desc* gate, const qerl_linear_desc* up,
                                          const qerl_linear_desc* down, void* workspace, size_t workspace_bytes, void* stream) {
  return mlp_impl(x, M, H, ldx, gain, noise, eps, gate, up, down, workspace, workspace_bytes, stream, true, nullptr);
}

// Sticky error word of a linear / block workspace: non-zero after a kernel's bounded wait on another workgroup gave
// up (a result of that call is then unreliable, and the workspace must be prepared again with qerl_workspace_init).
// Synchronises with the stream.
extern "C" int qerl_workspace_status(const void* workspace, void* stream) {
  if (!workspace) return QERL_ERR_NULL;
  if (!aligned(workspace, 256)) return QERL_ERR_ALIGN;
  uint32_t word = 0;
  const uint32_t* p = (const uint32_t*)workspace + kCtrlMainWords + kCtrlDownWords + kCtlErr;
  if (hipMemcpyAsync(&word, p, sizeof(word), hipMemcpyDeviceToHost, (hipStream_t)stream) != hipSuccess) return launch_status();
  if (hipStreamSynchronize((hipStream_t)stream) != hipSuccess) return launch_status();
  return qerl_status_from_error_word(word);
}

extern "C" int qerl_status_from_error_word(uint32_t word) { return word == 0u ? QERL_OK : QERL_ERR_TIMEOUT; }

extern "C" int qerl_selftest_wait_gives_up(void* workspace, size_t workspace_bytes, uint32_t polls, void* stream) {
  if (!workspace) return QERL_ERR_NULL;
  if (!aligned(workspace, 256) || workspace_bytes < kCtrlRegionBytes) return QERL_ERR_WORKSPACE;
  if (polls < 1 || polls > 1024) return QERL_ERR_SHAPE;   // a self-test, not a way to keep a wave spinning
  return launch_block_wait_selftest((uint32_t*)workspace + kCtrlMainWords + kCtrlDownWords, polls, (hipStream_t)stream);
}
