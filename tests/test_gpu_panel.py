"""GPU parity of the 9..128-token kernels (linear_panel.hip) at the sizes where their plan changes: edges of token tiles, row
tiles, units and stages, each way of cutting the units into pieces, ranks beyond one chunk, rows in several launches, outputs
and without 8-byte stores."""

import numpy as np
import pytest
import torch

import paper_2510_11696_amd as qerl
import qerl_synth as qs
from oracle import nvfp4_oracle as oracle
from tests.gpu_util import check_linear
from tests.test_gpu_block import _bf16, _member, _norm_inputs, _ref

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [9, 16, 17, 32, 33, 64, 65, 96, 97, 128])
@pytest.mark.parametrize("K,Ns,rs,bias", [
    (512, (129, 64), (16, 0), True),        # a ragged row tile, one row past a unit; a member without adapter
    (1168, (1000, 40, 31), (32, 8, 64), False),   # K: ten K-tiles, the last of 16 inputs; stages that end on half a slab
    (4352, (320,), (72,), True),            # more than 64 ranks, more than one piece per unit
    (16, (8200,), (8,), False),             # one K-tile: the second half of the stage is beyond K
])
def test_edges_of_the_plan(M, K, Ns, rs, bias):
    print("panel case", M, K, Ns, rs, bias, flush=True)
    x = qs.activations(M, K, 50 + M)
    ms = [_member(N, K, r, 60 + 3 * i + M, bias) for i, (N, r) in enumerate(zip(Ns, rs))]
    ws = qerl.Workspace(qerl.nvfp4_lora_linear_workspace_bytes(M, sum(Ns), K, sum(rs)))
    # rows of x further apart than K; the first output at an odd leading dimension (no 8-byte stores), with canaries
    xs = torch.full((M, K + 24), 7.0, dtype=torch.bfloat16, device="cuda")
    xs[:, :K] = x.cuda()
    wide = torch.full((M, Ns[0] + 3), -5.0, dtype=torch.bfloat16, device="cuda")
    outs = [wide[:, :Ns[0]]] + [torch.empty((M, N), dtype=torch.bfloat16, device="cuda") for N in Ns[1:]]
    call = lambda: qerl.nvfp4_lora_linear_packed_group(xs[:, :K], [m["pw"] for m in ms], [m["Ad"] for m in ms], [m["Bd"] for m in ms],
                                                       [2.0] * len(ms), workspace=ws, outs=outs, biases=[m["bd"] for m in ms])
    got = [o.clone() for o in call()]
    for i, m in enumerate(ms):
        check_linear(got[i], _ref(m, x.float().numpy(), 2.0), ("panel", i, M, K, Ns, rs))
    assert torch.all(wide[:, Ns[0]:] == -5.0)
    assert all(torch.equal(a, b) for a, b in zip(call(), got))


@pytest.mark.parametrize("M", [129, 192, 193, 256, 300, 640, 1000])
@pytest.mark.parametrize("K,Ns,rs", [
    (512, (129, 64), (16, 0)),
    (2064, (520, 40), (40, 64)),
])
def test_several_token_blocks(M, K, Ns, rs):
    """More than 128 tokens on few rows: blocks of three or four token tiles, the last one partly beyond M."""
    print("panel token blocks", M, K, Ns, rs, flush=True)
    x = qs.activations(M, K, 70 + M)
    ms = [_member(N, K, r, 80 + 3 * i + M, True) for i, (N, r) in enumerate(zip(Ns, rs))]
    call = lambda: qerl.nvfp4_lora_linear_packed_group(x.cuda(), [m["pw"] for m in ms], [m["Ad"] for m in ms], [m["Bd"] for m in ms],
                                                       [2.0] * len(ms), biases=[m["bd"] for m in ms])
    got = call()
    for i, m in enumerate(ms):
        check_linear(got[i], _ref(m, x.float().numpy(), 2.0), ("token blocks", i, M, K, Ns, rs))
    assert all(torch.equal(a, b) for a, b in zip(call(), got))


@pytest.mark.parametrize("M,N,K,r", [
    (16, 40000, 512, 16),     # more units than workgroups
    (40, 36864, 768, 16),     # equal pieces of the line of units (pieces that end inside a unit)
    (30, 24576, 1536, 8),     # the same at two workgroups per CU
    (128, 55296, 384, 8),     # whole units of 256 rows
    (70, 53248, 256, 8),      # the same, three token tiles
    (128, 70016, 128, 8),     # the sums of all rows do not fit the workspace: the GEMM
    (33, 140032, 128, 8),     # the same up to 64 tokens: several pairs of launches
    (100, 40000, 768, 8),     # few stages in units of 256 rows: one round of the chip where units of 128 would take two
    (16, 33024, 512, 8),      # the sums do not fit at 9..16 tokens: the decode kernels
])
def test_wide_launches(M, N, K, r):
    _wide(M, N, K, r)


@pytest.mark.parametrize("M", [9, 16, 17, 33, 65, 128])
@pytest.mark.parametrize("N,K", [
    (8200, 512),              # whole units of 128 rows: one launch stores the outputs
    (1000, 272),              # units of 64 rows up to 64 tokens, a ragged last tile
    (70016, 384),             # more units than CUs; from 33 tokens on units of 256 rows
    (4096, 2048),             # units in several pieces: two launches (up to 16 tokens the streaming kernel)
])
def test_linears_without_adapters(M, N, K):
    _wide(M, N, K, 0)


def test_outputs_without_adapters_in_one_launch_at_odd_strides():
    """The first launch stores the outputs of a group: a bias, a leading dimension that allows no 8-byte stores, a ragged member."""
    for M in (9, 50, 128):
        K, Ns = 1168, (1000, 33)
        x = qs.activations(M, K, 50 + M)
        ms = [_member(N, K, 0, 60 + 3 * i + M, i == 0) for i, N in enumerate(Ns)]
        wide = torch.full((M, Ns[0] + 3), -5.0, dtype=torch.bfloat16, device="cuda")
        outs = [wide[:, :Ns[0]], torch.empty((M, Ns[1]), dtype=torch.bfloat16, device="cuda")]
        qerl.nvfp4_lora_linear_packed_group(x.cuda(), [m["pw"] for m in ms], [None] * 2, [None] * 2, [0.0] * 2, outs=outs, biases=[m["bd"] for m in ms])
        for i, m in enumerate(ms):
            check_linear(outs[i], _ref(m, x.float().numpy(), 2.0), ("panel, no adapter", i, M))
        assert torch.all(wide[:, Ns[0]:] == -5.0)


def _wide(M, N, K, r):
    print("panel wide case", M, N, K, r, flush=True)
    gen = torch.Generator().manual_seed(M + N)
    codes = torch.randint(0, 256, (N, K // 2), dtype=torch.uint8, generator=gen)
    scales = torch.randint(0x20, 0x50, (N, K // 16), dtype=torch.uint8, generator=gen)
    ts = torch.tensor([0.01], dtype=torch.float32)
    A, B = qs.lora_pair(N, K, r, 5) if r else (None, None)
    x = qs.activations(M, K, 6)
    pw = qerl.nvfp4_prepack(codes.cuda(), scales.cuda(), ts.cuda())
    y = qerl.nvfp4_lora_linear_packed(x.cuda(), pw, A.cuda() if r else None, B.cuda() if r else None, 2.0)
    rows = np.unique(np.concatenate([np.arange(0, N, 997), np.arange(0, N, 128), np.arange(127, N, 128), [N - 1]]))
    ref = oracle.nvfp4_lora_linear(x.float().numpy(), codes.numpy()[rows], scales.numpy()[rows], float(ts), A.float().numpy() if r else None,
                                   B.float().numpy()[rows] if r else None, 2.0)
    check_linear(y[:, torch.from_numpy(rows).cuda()].contiguous(), ref, ("panel wide", M, N, K, r))


@pytest.mark.parametrize("M", [9, 16, 40, 100, 128])
@pytest.mark.parametrize("N,K", [(96, 16), (160, 272), (129, 1168), (64, 2064), (4100, 144)])
def test_infinities_in_the_last_inputs_of_a_row(M, N, K):
    """K no multiple of a stage: what stands beyond it is padding and takes no part, so an infinity among a token's last inputs gives
    infinities with the weights' signs (and NaN at zero weights), and the other tokens keep their values."""
    print("panel, infinities", M, N, K, flush=True)
    x, m = qs.activations(M, K, 150 + M), _member(N, K, 0, 155)
    clean = qerl.nvfp4_lora_linear_packed(x.cuda(), m["pw"])
    rows = torch.arange(0, M, 3)
    x[rows, K - 1 - rows % 8] = torch.where(rows % 2 == 0, float("inf"), float("-inf")).to(torch.bfloat16)
    y = qerl.nvfp4_lora_linear_packed(x.cuda(), m["pw"]).cpu().float()
    w = oracle.nvfp4_dequantize(m["codes"], m["scales"], m["ts"])
    with np.errstate(invalid="ignore"):
        want = torch.from_numpy((x[rows, K - 1 - rows % 8].double().numpy()[:, None] * w[:, (K - 1 - rows % 8).numpy()].T).astype(np.float32))
    assert torch.equal(torch.isnan(y[rows]), torch.isnan(want))
    assert torch.equal(torch.nan_to_num(y[rows], nan=0.0, posinf=1.0, neginf=-1.0), torch.nan_to_num(want, nan=0.0, posinf=1.0, neginf=-1.0))
    keep = torch.ones(M, dtype=torch.bool)
    keep[rows] = False
    assert torch.equal(y[keep], clean.cpu().float()[keep])


@pytest.mark.parametrize("M", [9, 16])
@pytest.mark.parametrize("N,K,r", [(256, 1024, 512), (32, 1024, 296), (1, 16, 1096)])
def test_ranks_whose_sums_exceed_the_workspace(M, N, K, r):
    """9..16 tokens and few rows: x A^T's parts alone take more than the workspace's area, and the decode kernels take the call."""
    print("panel, large rank", M, N, K, r, flush=True)
    x, m = qs.activations(M, K, 90 + M), _member(N, K, r, 95 + M)
    y = qerl.nvfp4_lora_linear_packed(x.cuda(), m["pw"], m["Ad"], m["Bd"], 2.0)
    check_linear(y, _ref(m, x.float().numpy(), 2.0), ("large rank", M, N, K, r))


@pytest.mark.parametrize("M", [9, 16, 33, 100])
@pytest.mark.parametrize("H,I,r", [(1024, 2736, 16), (512, 400, 72), (512, 4000, 64)])
def test_feed_forward_block_with_the_gated_second_launch(M, H, I, r):
    if r > 64 and M <= 16:
        pytest.skip("up to 16 tokens this entry point takes ranks up to 64")
    print("panel mlp case", M, H, I, r, flush=True)
    xin, gain, Z, xn = _norm_inputs(M, H, 11, 1e-2)
    g, u, d = _member(I, H, r, 12), _member(I, H, r, 15), _member(H, I, r, 18)
    act = _bf16(oracle.silu_mul(_bf16(_ref(g, xn, 2.0)), _bf16(_ref(u, xn, 2.0))))
    ref = _ref(d, act, 2.0)
    lib = qerl.load_library()
    need = lib.aqn_rmsnorm_nvfp4_lora_mlp_workspace_bytes(M, H, I, H, r, r, r)

    def call(ws):
        return qerl.aqn_rmsnorm_nvfp4_lora_mlp(xin.cuda(), gain.cuda(), Z.cuda(), 1e-6, g["pw"], u["pw"], d["pw"],
                                               [m["Ad"] for m in (g, u, d)], [m["Bd"] for m in (g, u, d)], (2.0,) * 3,
                                               workspace=ws)
    ws = qerl.Workspace(need)
    y = call(ws)
    check_linear(y, ref, ("panel mlp", M, H, I, r), slack=4e-3)
    assert torch.equal(call(ws), y)
