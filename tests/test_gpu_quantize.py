"""GPU parity: nvfp4_quantize / nvfp4_dequantize are bit-exact against the oracle."""
import numpy as np
import pytest
import torch

import paper_2510_11696_amd as qerl
from oracle import nvfp4_oracle as oracle
from tests import cases
from tests.gpu_util import quantize_both, to_gpu_bf16

pytestmark = pytest.mark.gpu


def _assert_same(gpu, ref, what):
    codes, scales, ts = gpu
    rcodes, rscales, rts = ref
    assert np.float32(ts.item()) == rts, (what, ts.item(), rts)
    assert np.array_equal(scales.cpu().numpy(), rscales), what
    assert np.array_equal(codes.cpu().numpy(), rcodes), what


@pytest.mark.parametrize("N,K", [(8, 128), (3, 32), (33, 272), (1, 16)])
def test_quantize_adversarial_cases_bit_exact(N, K):
    for name, W in cases.quantizer_cases(N, K, seed=100 + N).items():
        print("case", name, N, K, flush=True)
        gpu, ref = quantize_both(W)
        _assert_same(gpu, ref, name)
        # Eq. 6 on the GPU reproduces the oracle's fp32 dequantisation bit for bit
        Wh = qerl.nvfp4_dequantize(*gpu).cpu().numpy()
        assert np.array_equal(Wh.view(np.uint32), oracle.nvfp4_dequantize(*ref).view(np.uint32)), name


@pytest.mark.parametrize("N,K", [(512, 3584), (2048, 2048), (100, 18944)])
def test_quantize_model_shapes_bit_exact(N, K):
    W = cases.gaussian(N, K, seed=N + K)
    gpu, ref = quantize_both(W)
    _assert_same(gpu, ref, (N, K))


def test_quantize_order_sensitive_scale_chain():
    from tests.test_oracle_quantize import ORDER_SENSITIVE
    for amax, bamax in ORDER_SENSITIVE:
        W = np.zeros((1, 32), dtype=np.float32)
        W[0, 5] = -amax
        W[0, 20] = bamax
        gpu, ref = quantize_both(W)
        _assert_same(gpu, ref, (amax, bamax))


def test_quantize_strided_rows_and_empty():
    W = cases.gaussian(16, 256, seed=5)
    big = torch.zeros((16, 512), dtype=torch.bfloat16, device="cuda")
    big[:, :256] = to_gpu_bf16(W)
    big[:, 256:] = 99.0                      # must not be read as part of the tensor
    codes, scales, ts = qerl.nvfp4_quantize(big[:, :256])
    _assert_same((codes, scales, ts), oracle.nvfp4_quantize(W), "strided")
    codes, scales, ts = qerl.nvfp4_quantize(torch.empty((0, 64), dtype=torch.bfloat16, device="cuda"))
    assert ts.item() == 1.0 and codes.numel() == 0


def test_quantize_is_deterministic():
    W = to_gpu_bf16(cases.gaussian(256, 1024, seed=77))
    a = qerl.nvfp4_quantize(W)
    for _ in range(5):
        b = qerl.nvfp4_quantize(W)
        assert all(torch.equal(p, q) for p, q in zip(a, b))


@pytest.mark.parametrize("amax", [1.0, 0.0546875, 3.0e4, 2.0e-20, 1.0e-30])
def test_quantize_every_bf16_below_the_block_maximum(amax):
    """Sixteenths of every binade a code can come from, around all rounding boundaries, under several block maxima:
    the codes taken from w * (1 / d) equal those of the divisions, next to a boundary and away from it."""
    top = torch.tensor([amax], dtype=torch.bfloat16).view(torch.int16).item()
    rows = []
    for bmax in (top, top - 1, top - 37, top - 128 * 3 - 5, top - 128 * 9 - 77):
        mags = np.arange(max(bmax - 128 * 6, 0), bmax + 1, dtype=np.int64)
        mags = np.concatenate([mags, np.zeros(-len(mags) % 15, dtype=np.int64)]).reshape(-1, 15)
        blocks = np.concatenate([np.full((len(mags), 1), bmax), mags], axis=1)
        blocks[:, 1::2] |= 0x8000
        rows.append(blocks)
    bits = np.concatenate(rows)
    bits = np.concatenate([np.tile(np.int64(top), (1, 16)), bits])
    W = (bits.astype(np.uint32) << 16).view(np.float32).reshape(1, -1)
    gpu, ref = quantize_both(W)
    _assert_same(gpu, ref, amax)


@pytest.mark.parametrize("N,K,ldw", [(1, 16, 16), (255, 16 * 129, 16 * 129), (257, 16 * 129, 16 * 131), (1111, 16 * 480, 16 * 480),
                                     (700, 16 * 800, 16 * 800 + 8)])
def test_quantize_remainders_of_the_two_passes(N, K, ldw):
    """Less than one load per thread, several steps of either pass and a last one that is partly empty; rows with and
    without a gap behind them."""
    W = cases.gaussian(N, K, seed=N)
    big = torch.full((N, ldw), 9.0, dtype=torch.bfloat16, device="cuda")
    big[:, :K] = to_gpu_bf16(W)
    _assert_same(qerl.nvfp4_quantize(big[:, :K]), oracle.nvfp4_quantize(W), (N, K, ldw))


@pytest.mark.parametrize("N,K", [(1, 16), (33, 272), (64, 640), (100, 1104), (32, 64 * 9)])
def test_prepack_of_unaligned_codes_and_scales_is_the_same(N, K):
    gen = torch.Generator().manual_seed(N * K)
    codes = torch.randint(0, 256, (N, K // 2), generator=gen, dtype=torch.uint8).cuda()
    scales = torch.randint(0, 127, (N, K // 16), generator=gen, dtype=torch.uint8).cuda()
    ts = torch.ones(1, device="cuda")
    want = qerl.nvfp4_prepack(codes, scales, ts).packed

    def shifted(t, by):
        flat = torch.empty(t.numel() + 16, dtype=torch.uint8, device="cuda")
        flat[by:by + t.numel()] = t.flatten()
        return flat[by:by + t.numel()].view(t.shape)

    for cs, ss in ((0, 1), (8, 2), (4, 0), (1, 3)):
        assert torch.equal(qerl.nvfp4_prepack(shifted(codes, cs), shifted(scales, ss), ts).packed, want), (cs, ss)
