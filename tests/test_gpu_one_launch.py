"""The persistent one-launch kernel of the composed calls (up to 16 tokens) where they still take it: a feed-forward block whose down
projection has a bias, and a workspace of the size that this launch alone needs where the separate launches need more.  The
other calls of these entry points are covered by test_gpu_block.py; which launches a call makes is checked on the host."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2510_11696_amd as qerl
from oracle import nvfp4_oracle as oracle
from paper_2510_11696_amd import binding
from tests.gpu_util import check_linear, smallest_workspace
from tests.test_gpu_block import _bf16, _member, _norm_inputs, _ref
from tests.test_gpu_graph import _replays_match

pytestmark = pytest.mark.gpu


def _mlp_with_bias(x, gain, Z, gate, up, down, ws, out):
    """aqn_rmsnorm_nvfp4_lora_mlp with a bias on down, which the binding does not offer."""
    H, I = x.shape[1], gate["N"]
    descs = [binding._make_desc(m["pw"], m["Ad"], m["Bd"], 2.0, y, b, k)[0]
             for m, y, b, k in ((gate, None, None, H), (up, None, None, H), (down, out, down["bd"], I))]
    binding._check("aqn_rmsnorm_nvfp4_lora_mlp", qerl.load_library().aqn_rmsnorm_nvfp4_lora_mlp(
        x.data_ptr(), x.shape[0], H, H, gain.data_ptr(), Z.data_ptr() if Z is not None else None, 1e-6,
        *(ctypes.byref(d) for d in descs), ws.ptr, ws.nbytes, torch.cuda.current_stream().cuda_stream))


@pytest.mark.parametrize("M", [1, 5, 8, 9, 13, 16])
@pytest.mark.parametrize("H,I,rs,sigma", [
    (512, 1024, (16, 16, 16), 1e-2),
    (3584, 2368, (32, 32, 32), 1e-2),        # 74 gate / up tile pairs; down's K is not a multiple of 128
    (5120, 1728, (64, 64, 64), 5e-4),        # rows longer than one K-range at 16 tokens
    (2048, 4096, (0, 0, 0), None),           # no adapters, no noise: no producers
    (1024, 640, (8, 0, 64), 1e-2),           # mixed ranks
    (8192, 3584, (16, 16, 16), 5e-3),        # stages that need different LDS areas
])
def test_feed_forward_block_with_a_bias(M, H, I, rs, sigma):
    print("one launch, mlp with bias", M, H, I, rs, sigma, flush=True)
    xin, gain, Z, xn = _norm_inputs(M, H, 1800 + M, sigma)
    gate, up, down = _member(I, H, rs[0], 7000 + M), _member(I, H, rs[1], 7100 + M), _member(H, I, rs[2], 7200 + M, True)
    act = oracle.silu_mul(_bf16(_ref(gate, xn, 2.0)), _bf16(_ref(up, xn, 2.0))).astype(np.float32)
    ws = qerl.Workspace(qerl.load_library().aqn_rmsnorm_nvfp4_lora_mlp_workspace_bytes(M, H, I, H, *rs))
    x, g, z = xin.cuda(), gain.cuda(), Z.cuda() if Z is not None else None
    y, again = (torch.empty((M, H), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    _mlp_with_bias(x, g, z, gate, up, down, ws, y)
    _mlp_with_bias(x, g, z, gate, up, down, ws, again)
    torch.cuda.synchronize()
    assert qerl.workspace_status(ws) == 0
    check_linear(y, _ref(down, act, 2.0), ("one launch, mlp with bias", M, H, I, rs), slack=4e-3)
    assert torch.equal(y, again), "second run on the same workspace differs"


@pytest.mark.parametrize("M", [9, 13, 16])
@pytest.mark.parametrize("H,Ns,rs,sigma,bias", [
    (2048, (16384,), (16,), 1e-2, True),
    (1040, (20000, 72), (0, 64), None, False),    # K not a multiple of 128; a member without adapter
    (1536, (8200, 8200, 40), (8, 32, 24), 5e-4, True),
])
def test_wide_groups_on_the_smallest_workspace(M, H, Ns, rs, sigma, bias):
    print("one launch, group", M, H, Ns, rs, flush=True)
    xin, gain, Z, xn = _norm_inputs(M, H, 1900 + M, sigma)
    mem = [_member(N, H, r, 7300 + 10 * i + M, bias) for i, (N, r) in enumerate(zip(Ns, rs))]
    x, g, z = xin.cuda(), gain.cuda(), Z.cuda() if Z is not None else None

    def call(ws):
        return qerl.aqn_rmsnorm_nvfp4_lora_linear_group(x, g, z, 1e-6, [m["pw"] for m in mem], [m["Ad"] for m in mem], [m["Bd"] for m in mem],
                                                        [2.0] * len(mem), workspace=ws, biases=[m["bd"] for m in mem])
    need = qerl.aqn_rmsnorm_nvfp4_lora_linear_group_workspace_bytes(M, H, list(Ns), list(rs))
    small = smallest_workspace(call, need)
    assert small.nbytes < need                   # the separate launches do not fit
    sizes = [need, (need + small.nbytes) // 512 * 256, small.nbytes]
    for ws in [qerl.Workspace(n) for n in sizes[:2]] + [small]:
        outs = [o.clone() for o in call(ws)]
        again = call(ws)
        torch.cuda.synchronize()
        assert qerl.workspace_status(ws) == 0
        for i, (m, o) in enumerate(zip(mem, outs)):
            check_linear(o, _ref(m, xn, 2.0), ("one launch, group", i, M, H, Ns, rs, ws.nbytes))
        assert all(torch.equal(p, q) for p, q in zip(outs, again)), "second run on the same workspace differs"


@pytest.mark.parametrize("M", [1, 9, 16])
def test_the_one_launch_replays_like_eager(M):
    """Its stage boundary, hand-over words and K-range counters live in the workspace and are re-armed by the launch itself."""
    print("one launch, graph", M, flush=True)
    H, I, r = 2048, 2816, 32
    xin, gain, Z, _ = _norm_inputs(M, H, 2000 + M, 1e-2)
    gate, up, down = _member(I, H, r, 7400), _member(I, H, r, 7410), _member(H, I, r, 7420, True)
    x, g, z = xin.cuda(), gain.cuda(), Z.cuda()
    ws = qerl.Workspace(qerl.load_library().aqn_rmsnorm_nvfp4_lora_mlp_workspace_bytes(M, H, I, H, r, r, r))
    y = torch.empty((M, H), dtype=torch.bfloat16, device="cuda")
    _replays_match(lambda: _mlp_with_bias(x, g, z, gate, up, down, ws, y), lambda: [y])
    assert qerl.workspace_status(ws) == 0


class _Guarded:
    """A workspace of exactly `nbytes` with a guard behind it."""

    def __init__(self, nbytes):
        self.inner = qerl.Workspace(nbytes + (1 << 16))
        self.ptr, self.nbytes = self.inner.ptr, nbytes
        self.inner.buf[nbytes:] = 0xA5

    def intact(self):
        return bool((self.inner.buf[self.nbytes:] == 0xA5).all())


@pytest.mark.parametrize("M", [1, 7, 8, 9, 16])
@pytest.mark.parametrize("H,I,rs", [(512, 1024, (16, 16, 16)), (2048, 5504, (64, 64, 64)), (9216, 2048, (16, 0, 8)), (1024, 20000, (0, 0, 0)),
                                    (3584, 9472, (32, 32, 32))])
def test_composed_calls_stay_inside_the_workspace_they_ask_for(M, H, I, rs):
    """The bytes behind the workspace stay as they are, and the outputs are those of a larger one."""
    print("composed call, guarded workspace", M, H, I, rs, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(M + I)
    mk = lambda *s, std=1.0: (torch.randn(s, generator=gen, device="cuda") * std).to(torch.bfloat16)

    def member(N, K, r):
        codes = torch.randint(0, 256, (N, K // 2), dtype=torch.uint8, device="cuda", generator=gen)
        scales = torch.randint(0x30, 0x48, (N, K // 16), dtype=torch.uint8, device="cuda", generator=gen)
        return qerl.nvfp4_prepack(codes, scales, torch.tensor([2e-4], device="cuda")), mk(r, K, std=0.1) if r else None, mk(N, r, std=0.02) if r else None
    gate, up, down = member(I, H, rs[0]), member(I, H, rs[1]), member(H, I, rs[2])
    x, gain = mk(M, H), mk(H, std=0.05) + 1
    lib = qerl.load_library()
    calls = [
        (lib.aqn_rmsnorm_nvfp4_lora_mlp_workspace_bytes(M, H, I, H, *rs),
         lambda ws: [qerl.aqn_rmsnorm_nvfp4_lora_mlp(x, gain, None, 1e-6, gate[0], up[0], down[0], (gate[1], up[1], down[1]), (gate[2], up[2], down[2]),
                                                     (2.0,) * 3, workspace=ws)]),
        (qerl.aqn_rmsnorm_nvfp4_lora_linear_group_workspace_bytes(M, H, [I, I], list(rs[:2])),
         lambda ws: qerl.aqn_rmsnorm_nvfp4_lora_linear_group(x, gain, None, 1e-6, [gate[0], up[0]], [gate[1], up[1]], [gate[2], up[2]], [2.0] * 2, workspace=ws)),
    ]
    for need, call in calls:
        ws = _Guarded(need)
        outs = [o.clone() for o in call(ws)]
        want = call(qerl.Workspace(need + (64 << 20)))
        torch.cuda.synchronize()
        assert ws.intact()
        assert all(torch.equal(p, q) for p, q in zip(outs, want))
        assert all(torch.isfinite(p.float()).all() for p in outs)
