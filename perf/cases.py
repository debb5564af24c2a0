"""The work this library is used for, as a list of cases that can be prepared, run and priced one by one.

A case is a dict of plain values; `prepare` makes what a program holds before the call (weights quantised and packed
once, adapters, activations, workspaces, for decode the recorded HIP graph that a rollout engine replays), `run` is one
pass through the public entry points and returns everything the pass computes.

Kinds
    linear    one packed NVFP4 + LoRA linear, launched eagerly
    decode    one rollout step of a few decoder layers: fresh AQN noise vectors, then per layer {norm, q, k, v}, o and
              {norm, gate, up, SiLU-mul, down}; recorded once and replayed as a HIP graph
    prefill   the same layers' linears over a prompt or a scored rollout (log-probabilities), launched eagerly
    backward  dX, dA, dB of the seven linears of a layer, q + k + v and gate + up as groups that share dX
    quantize  bf16 weights of a layer -> NVFP4 -> the tile order of the forward pass
    mx        the seven linears of a layer in the MXFP4 variant with adapters
"""
from __future__ import annotations

import torch

import paper_2510_11696_amd as qerl

EPS = 1e-6
# Decoder layers as (hidden, k/v width, intermediate): the 7B, 14B and 32B shapes of the benchmark's configurations.
LAYER_7B = dict(hidden=3584, kv=512, inter=18944)
LAYER_14B = dict(hidden=5120, kv=1024, inter=13824)
LAYER_32B = dict(hidden=5120, kv=1024, inter=27648)


def listed():
    return [
        # the smallest call: one token through one 2048 x 2048 linear; launch latency and the call path count
        dict(name="linear 2048 m1", kind="linear", M=1, N=2048, K=2048, r=16),
        # batch-8 rollout of the 7B shapes
        dict(name="decode 7b m8", kind="decode", M=8, layers=8, r=32, **LAYER_7B),
        # one sequence on the 32B shapes: nothing but weight streaming
        dict(name="decode 32b m1", kind="decode", M=1, layers=4, r=64, **LAYER_32B),
        # batch-16 rollout of the 32B shapes, the benchmark's headline
        dict(name="decode 32b m16", kind="decode", M=16, layers=4, r=64, **LAYER_32B),
        # a GRPO group of 32 completions on the 7B shapes
        dict(name="decode 7b m32", kind="decode", M=32, layers=8, r=32, **LAYER_7B),
        # a batch from which some sequences have already ended: no multiple of any tile
        dict(name="decode 14b m77", kind="decode", M=77, layers=4, r=64, **LAYER_14B),
        # the largest decode batch
        dict(name="decode 32b m128", kind="decode", M=128, layers=4, r=64, **LAYER_32B),
        # a few prompts of uneven length packed together
        dict(name="prefill 7b m777", kind="prefill", M=777, r=32, **LAYER_7B),
        # a full prefill / log-probability batch on the largest shapes
        dict(name="prefill 32b m4096", kind="prefill", M=4096, r=64, **LAYER_32B),
        # the policy update's backward through one layer
        dict(name="backward 14b m2048", kind="backward", M=2048, r=64, **LAYER_14B),
        # loading a model: quantise and pack one layer
        dict(name="quantize 7b", kind="quantize", **LAYER_7B),
        # the MXFP4 variant over a prefill batch
        dict(name="mx 14b m2048", kind="mx", M=2048, r=64, **LAYER_14B),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, round(lo * (hi / lo) ** rng.random())))


def _layer(rng, inter_max):
    """A decoder layer of generic proportions; widths are multiples of 64 as every published model's are."""
    hidden = rng.randrange(1024, 5121, 64)
    inter = min(inter_max, 64 * round(hidden * rng.uniform(2.6, 5.4) / 64))
    return dict(hidden=hidden, kv=128 * rng.randint(2, max(2, hidden // 640)), inter=inter)


def draw(rng):
    kind = rng.choice(["linear", "decode", "decode", "decode", "decode", "prefill", "prefill", "backward", "quantize", "mx"])
    r = rng.choice([8, 16, 32, 64])
    if kind == "linear":
        return dict(kind=kind, M=_log_int(rng, 1, 2048), N=16 * rng.randint(32, 512), K=64 * rng.randint(8, 128), r=r)
    if kind == "decode":
        return dict(kind=kind, M=_log_int(rng, 1, 128), layers=4, r=r, **_layer(rng, 27648))
    if kind == "prefill":
        return dict(kind=kind, M=_log_int(rng, 129, 4096), r=r, **_layer(rng, 27648))
    if kind == "backward":
        return dict(kind=kind, M=_log_int(rng, 129, 2048), r=r, **_layer(rng, 13824))
    if kind == "quantize":
        return dict(kind=kind, **_layer(rng, 18944))
    return dict(kind=kind, M=_log_int(rng, 1, 2048), r=r, **_layer(rng, 13824))


def _linears(case):
    """(name, out-features, in-features) of the case's linears."""
    if case["kind"] == "linear":
        return [("lin", case["N"], case["K"])]
    h, kv, i = case["hidden"], case["kv"], case["inter"]
    return [("q", h, h), ("k", kv, h), ("v", kv, h), ("o", h, h), ("gate", i, h), ("up", i, h), ("down", h, i)]


class _Draw:
    """Seeded device tensors with the distributions of the benchmark's synthetic layers."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed)

    def bf16(self, *shape, std=1.0, mean=0.0):
        return (torch.randn(shape, generator=self.gen, device="cuda") * std + mean).to(torch.bfloat16)

    def weight(self, N, K):
        return self.bf16(N, K, std=0.02)

    def lora(self, N, K, r):
        return self.bf16(r, K, std=1.0 / r), self.bf16(N, r, std=0.01)

    def gain(self, H):
        return self.bf16(H, std=0.05, mean=1.0)


class _State:
    pass


def prepare(case, seed):
    d = _Draw(seed)
    s = _State()
    s.kind = kind = case["kind"]
    lin = _linears(case)
    M, r = case.get("M"), case.get("r", 0)
    s.scale = 2.0      # alpha / r of every configuration
    if kind == "quantize":
        s.weights = [d.weight(N, K) for _, N, K in lin]
        return s
    if kind == "linear":
        _, N, K = lin[0]
        s.w = qerl.nvfp4_prepack(*qerl.nvfp4_quantize(d.weight(N, K)))
        s.A, s.B = d.lora(N, K, r)
        s.x = d.bf16(M, K)
        s.ws = qerl.Workspace(qerl.nvfp4_lora_linear_workspace_bytes(M, N, K, r))
        return s
    lib = qerl.load_library()
    if kind == "mx":
        s.lin = []
        for name, N, K in lin:
            s.lin.append((name, qerl.mxfp4_prepack(*qerl.mxfp4_quantize(d.weight(N, K))), *d.lora(N, K, r)))
        s.x = {K: d.bf16(M, K) for _, _, K in lin}
        s.ws = qerl.Workspace(max(lib.mxfp4_lora_linear_native_workspace_bytes(M, N, K, r) for _, N, K in lin))
        return s
    if kind == "backward":
        s.w = {n: qerl.nvfp4_prepack_t(*qerl.nvfp4_quantize(d.weight(N, K))) for n, N, K in lin}
        s.ab = {n: d.lora(N, K, r) for n, N, K in lin}
        # the linears' inputs as the forward pass left them; gradients small beside them
        s.x = {"qkv": d.bf16(M, case["hidden"]), "o": d.bf16(M, case["hidden"]), "mlp": d.bf16(M, case["hidden"]), "down": d.bf16(M, case["inter"])}
        s.dy = {n: d.bf16(M, N, std=0.02) for n, N, K in lin}
        return s
    # decode, prefill
    h = case["hidden"]
    s.layers = []
    for _ in range(case.get("layers", 1)):
        w = {n: (qerl.nvfp4_prepack(*qerl.nvfp4_quantize(d.weight(N, K))), *d.lora(N, K, r)) for n, N, K in lin}
        s.layers.append(dict(w=w, gain_in=d.gain(h), gain_post=d.gain(h),
                             hidden=d.bf16(M, h), attn=d.bf16(M, h), mid=d.bf16(M, h),
                             out={n: torch.empty((M, N), dtype=torch.bfloat16, device="cuda") for n, N, K in lin if n not in ("gate", "up")}))
    s.noise = torch.empty((2 * len(s.layers) * h,), dtype=torch.float32, device="cuda")
    for i, L in enumerate(s.layers):
        L["z_in"], L["z_post"] = s.noise[2 * i * h:(2 * i + 1) * h], s.noise[(2 * i + 1) * h:(2 * i + 2) * h]
    s.seed = seed
    s.ws_qkv = qerl.Workspace(qerl.aqn_rmsnorm_nvfp4_lora_linear_group_workspace_bytes(M, h, [h, case["kv"], case["kv"]], [r] * 3))
    s.ws_o = qerl.Workspace(qerl.nvfp4_lora_linear_workspace_bytes(M, h, h, r))
    s.ws_mlp = qerl.Workspace(lib.aqn_rmsnorm_nvfp4_lora_mlp_workspace_bytes(M, h, case["inter"], h, r, r, r))
    s.outputs = [t for L in s.layers for t in L["out"].values()]
    if kind == "decode":
        _layers_pass(s)              # everything loaded before the recording
        torch.cuda.synchronize()
        s.graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s.graph):
            _layers_pass(s)
    return s


def _layers_pass(s):
    qerl.aqn_noise_fill(s.noise.numel(), qerl.aqn_sigma(1, 10, 1e-2, 5e-4), s.seed, 0, out=s.noise)
    for L in s.layers:
        w, out = L["w"], L["out"]
        ws, As, Bs = zip(*(w[n] for n in ("q", "k", "v")))
        qerl.aqn_rmsnorm_nvfp4_lora_linear_group(L["hidden"], L["gain_in"], L["z_in"], EPS, ws, As, Bs, [s.scale] * 3,
                                                 workspace=s.ws_qkv, outs=[out[n] for n in ("q", "k", "v")])
        wo, Ao, Bo = w["o"]
        qerl.nvfp4_lora_linear_packed(L["attn"], wo, Ao, Bo, s.scale, workspace=s.ws_o, out=out["o"])
        (wg, wu, wd), As, Bs = zip(*(w[n] for n in ("gate", "up", "down")))
        qerl.aqn_rmsnorm_nvfp4_lora_mlp(L["mid"], L["gain_post"], L["z_post"], EPS, wg, wu, wd, As, Bs, (s.scale,) * 3,
                                        workspace=s.ws_mlp, out=out["down"])


def run(s):
    if s.kind == "linear":
        return qerl.nvfp4_lora_linear_packed(s.x, s.w, s.A, s.B, s.scale, workspace=s.ws)
    if s.kind == "decode":
        s.graph.replay()
        return s.outputs
    if s.kind == "prefill":
        _layers_pass(s)
        return s.outputs
    if s.kind == "quantize":
        got = []
        for W in s.weights:
            codes, scales, ts = qerl.nvfp4_quantize(W)
            got.append((codes, scales, ts, qerl.nvfp4_prepack(codes, scales, ts).packed))
        return got
    if s.kind == "mx":
        return {n: qerl.mxfp4_lora_linear_native(s.x[w.K], w, A, B, s.scale, workspace=s.ws) for n, w, A, B in s.lin}
    got = []
    for key, names in (("down", ("down",)), ("mlp", ("gate", "up")), ("o", ("o",)), ("qkv", ("q", "k", "v"))):
        As, Bs = zip(*(s.ab[n] for n in names))
        if len(names) == 1:
            got.append(qerl.nvfp4_lora_linear_backward(s.x[key], s.dy[names[0]], s.w[names[0]], As[0], Bs[0], s.scale))
        else:
            got.append(qerl.nvfp4_lora_linear_backward_group(s.x[key], [s.dy[n] for n in names], [s.w[n] for n in names], As, Bs,
                                                             [s.scale] * len(names)))
    return got


def work(case):
    kind, M, r = case["kind"], case.get("M", 0), case.get("r", 0)
    lin = _linears(case)
    params = sum(N * K for _, N, K in lin)
    ranks = sum(r * (N + K) for _, N, K in lin)
    if kind == "quantize":
        # bf16 in; codes, scales and the packed tiles out
        return {"bytes": params * (2 + 2 * 0.5625), "flops": 0}
    if kind == "linear":
        _, N, K = lin[0]
        return {"bytes": params * 0.5625 + 2 * ranks + 2 * M * (N + K), "flops": 2 * M * (params + ranks)}
    h, kv, i = case["hidden"], case["kv"], case["inter"]
    if kind == "mx":
        return {"bytes": params * 0.53125 + 2 * ranks + 2 * M * (h + i + sum(N for _, N, _ in lin)), "flops": 2 * M * (params + ranks)}
    if kind == "backward":
        io = 2 * M * (2 * (3 * h + i) + sum(N for _, N, _ in lin))      # x and dX of the four inputs, every dY
        # dX; dY B and its product with A; x A^T; dA and dB
        return {"bytes": params * 0.5625 + 2 * ranks + 4 * ranks + io, "flops": 2 * M * (params + sum(r * (2 * N + 3 * K) for _, N, K in lin))}
    n = case.get("layers", 1)
    # the three inputs and q, k, v, o, down; gains, noise written and read once
    io = 2 * M * (3 * h + 3 * h + 2 * kv) + 2 * h * (2 + 4 + 4)
    return {"bytes": n * (params * 0.5625 + 2 * ranks + io), "flops": n * 2 * M * (params + ranks)}


def tolerance(case):
    # The passes against their composition in fp64 with the same bf16 roundings between the operators: rel 1.6e-3..1.7e-3
    # everywhere (the outputs' rounding to bf16), max 4e-3, up to 9e-3 for down's output behind the rounded SiLU(gate) * up.
    if case["kind"] == "quantize":
        return "exact"
    return {"rel": 6.5e-3, "max": 3.5e-2}
