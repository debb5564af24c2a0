"""MXFP4 variant on the GPU: quantisers and dequantiser bit-exact, packed layout, and the linear on the
block-scaled matrix instruction against the oracle's product of the two quantised operands."""
import numpy as np
import pytest
import torch

import paper_2510_11696_amd as qerl
import qerl_synth as qs
from oracle import mx_oracle as mx
from tests import cases
from tests.gpu_util import check_linear

pytestmark = pytest.mark.gpu


def _bf16(a):
    return torch.from_numpy(np.asarray(a, dtype=np.float32)).to(torch.bfloat16)


@pytest.mark.parametrize("N,K", [(48, 512), (5, 32), (100, 18944), (512, 3584)])
def test_mxfp4_quantize_bit_exact(N, K):
    print("mx quantize case", N, K, flush=True)
    tensors = {"gaussian": cases.gaussian(N, K, seed=N + K)}
    if N * K <= 48 * 512:
        tensors.update(cases.quantizer_cases(N, K, seed=7))
    for name, W in tensors.items():
        W = _bf16(W)
        codes, scales = qerl.mxfp4_quantize(W.cuda())
        ref_c, ref_s = mx.mxfp4_quantize(W.float().numpy())
        assert np.array_equal(scales.cpu().numpy(), ref_s), name
        assert np.array_equal(codes.cpu().numpy(), ref_c), name
        What = qerl.mxfp4_dequantize(codes, scales).cpu().numpy().astype(np.float64)
        assert np.array_equal(What, mx.mxfp4_dequantize(ref_c, ref_s).astype(np.float32).astype(np.float64)), name


def test_mx_quantize_special_blocks_and_strided_rows():
    rows = np.zeros((6, 64), dtype=np.float32)
    rows[0, :4] = [6.0, 2.5, 3.5, -5.0]                 # ties
    rows[1, 32:36] = [3.9, -0.0, 1e-30, 7.0]            # saturation inside the block; signed zero; underflow
    rows[2, :2] = [2.0 ** 100, -2.0 ** 96]              # large exponents
    rows[3, :2] = [2.0 ** -120, 2.0 ** -126]            # scale byte near its lower clamp
    rows[4, :] = 448.0
    rows[5, 0] = 500.0                                   # MXFP8: clamps to 448
    W = _bf16(rows)
    wide = torch.zeros((6, 96), dtype=torch.bfloat16)
    wide[:, :64] = W
    for src in (W.cuda(), wide.cuda()[:, :64]):          # contiguous and strided rows
        c, s = qerl.mxfp4_quantize(src)
        rc, rs = mx.mxfp4_quantize(W.float().numpy())
        assert np.array_equal(c.cpu().numpy(), rc) and np.array_equal(s.cpu().numpy(), rs)
        c8, s8 = qerl.mxfp8_quantize(src)
        rc8, rs8 = mx.mxfp8_quantize(W.float().numpy())
        assert np.array_equal(c8.cpu().numpy(), rc8) and np.array_equal(s8.cpu().numpy(), rs8)
    assert qerl.mxfp4_quantize(torch.empty((0, 64), dtype=torch.bfloat16, device="cuda"))[0].numel() == 0


@pytest.mark.parametrize("M,K", [(1, 32), (8, 3584), (32, 5120), (7, 18944)])
def test_mxfp8_activation_quantize_bit_exact(M, K):
    x = qs.activations(M, K, 600 + M)
    c, s = qerl.mxfp8_quantize(x.cuda())
    rc, rs = mx.mxfp8_quantize(x.float().numpy())
    assert np.array_equal(s.cpu().numpy(), rs)
    assert np.array_equal(c.cpu().numpy(), rc)


@pytest.mark.parametrize("M,K", [(1, 32), (3, 512), (9, 544), (130, 1056), (2051, 5120)])
def test_mxfp8_quantize_of_any_bits_with_and_without_wide_loads(M, K):
    """Rows that 16-byte loads may read and rows offset by four bytes go to different kernels: the same bytes, over all bf16 bit
    patterns (infinities and NaNs too), and the oracle's where the values are finite."""
    print("mxfp8 any bits", M, K, flush=True)
    g = torch.Generator().manual_seed(M + K)
    bits = torch.randint(0, 1 << 16, (M, K), generator=g, dtype=torch.int32)
    near = torch.randint(0, 256, (M, K // 32, 1), generator=g, dtype=torch.int32)       # most blocks: exponents that lie close together
    exp = (near - torch.randint(0, 20, (M, K // 32, 32), generator=g, dtype=torch.int32)).clamp(0, 254).reshape(M, K)
    bits = torch.where((torch.arange(K) // 32 % 4 != 3)[None, :], (bits & 0x807f) | (exp << 7), bits)
    x = bits.to(torch.int16).view(torch.bfloat16)
    wide = torch.zeros((M, K + 8), dtype=torch.bfloat16, device="cuda")
    wide[:, 2:K + 2] = x.cuda()
    c, s = qerl.mxfp8_quantize(x.cuda())
    co, so = qerl.mxfp8_quantize(wide[:, 2:K + 2])
    assert torch.equal(s, so) and torch.equal(c, co)
    finite = torch.isfinite(x.float().reshape(M, K // 32, 32)).all(-1)
    xf = torch.where(finite.repeat_interleave(32, 1), x.float(), torch.zeros(()))
    rc, rs = mx.mxfp8_quantize(xf.numpy())
    f = finite.numpy()
    assert np.array_equal(s.cpu().numpy()[f], rs[f])
    assert np.array_equal(c.cpu().numpy().reshape(M, K // 32, 32)[f], rc.reshape(M, K // 32, 32)[f])


@pytest.mark.parametrize("M,K,r", [(255, 544, 16), (256, 32, 8), (257, 1056, 72), (700, 13824, 64), (2051, 2592, 128)])
def test_mx_lora_linear_quantises_x_like_the_plain_one(M, K, r):
    """From 256 tokens the launch of the down-projection quantises x too.  With B = 0 the adapter adds zeros: the same bytes as the
    linear without one, which quantises in a launch of its own; on rows with a stride and a second pass on the same workspace too."""
    print("mx lora quantise", M, K, r, flush=True)
    N = 96
    wide = qs.activations(M, K + 8, 40 + M).cuda()
    w = qerl.mxfp4_prepack(*qerl.mxfp4_quantize(qs.activations(N, K, 41).cuda()))
    A, B = qs.activations(r, K, 42).cuda(), torch.zeros((N, r), dtype=torch.bfloat16, device="cuda")
    wk = qerl.Workspace(qerl.load_library().mxfp4_lora_linear_native_workspace_bytes(M, N, K, r))
    for x in (wide[:, :K], wide[:, 8:].contiguous()):
        ref = qerl.mxfp4_linear_native(x, w)
        assert torch.equal(qerl.mxfp4_lora_linear_native(x, w, A, B, 2.0, workspace=wk), ref)


def _pack_reference(codes, scales):
    """Tiles of 32 rows x 256 inputs, 4352 bytes: step j (64 inputs) holds, for lane l = (n = l % 32, g = l // 32),
    the 16 code bytes of inputs 64 j + 32 g .. + 31 of row n at j * 1024 + l * 16 and their scale byte at 4096 + 4 l + j."""
    N, K = codes.shape[0], codes.shape[1] * 2
    nt, kt = -(-N // 32), -(-K // 256)
    cp = np.zeros((nt * 32, kt * 128), dtype=np.uint8); cp[:N, :K // 2] = codes
    sp = np.zeros((nt * 32, kt * 8), dtype=np.uint8); sp[:N, :K // 32] = scales
    out = np.zeros((nt, kt, 4352), dtype=np.uint8)
    for a in range(nt):
        for b in range(kt):
            for j in range(4):
                for lane in range(64):
                    n, g = a * 32 + lane % 32, lane // 32
                    k0 = b * 256 + 64 * j + 32 * g
                    out[a, b, j * 1024 + lane * 16: j * 1024 + lane * 16 + 16] = cp[n, k0 // 2: k0 // 2 + 16]
                    out[a, b, 4096 + 4 * lane + j] = sp[n, k0 // 32]
    return out.reshape(-1)


@pytest.mark.parametrize("N,K", [(32, 128), (40, 320), (100, 64), (64, 1024)])
def test_mxfp4_prepack_is_the_documented_permutation(N, K):
    rng = np.random.default_rng(N + K)
    codes = rng.integers(0, 256, size=(N, K // 2)).astype(np.uint8)
    scales = rng.integers(0, 255, size=(N, K // 32)).astype(np.uint8)
    pw = qerl.mxfp4_prepack(torch.from_numpy(codes).cuda(), torch.from_numpy(scales).cuda())
    assert np.array_equal(pw.packed.cpu().numpy(), _pack_reference(codes, scales))


def _problem(M, N, K, seed):
    W = _bf16(cases.gaussian(N, K, seed))
    x = qs.activations(M, K, seed + 1)
    codes, scales = mx.mxfp4_quantize(W.float().numpy())
    pw = qerl.mxfp4_prepack(torch.from_numpy(codes).cuda(), torch.from_numpy(scales).cuda())
    return x, codes, scales, pw


def test_native_linear_reads_dequantised_columns_for_one_hot_rows():
    """x = rows of the identity (exact in MXFP8): y[m, :] is column k_m of the dequantised weights, for k_m
    in both halves of a 64-input step, across steps, tiles and the padded tail."""
    N, K = 96, 320
    _, codes, scales, pw = _problem(1, N, K, 11)
    ks = [0, 1, 31, 32, 33, 63, 64, 127, 128, 200, 319]
    x = torch.zeros((len(ks), K), dtype=torch.bfloat16)
    for m, k in enumerate(ks):
        x[m, k] = 1.0
    y = qerl.mxfp4_linear_native(x.cuda(), pw).float().cpu().numpy()
    What = mx.mxfp4_dequantize(codes, scales)
    want = torch.from_numpy(What[:, ks].T.astype(np.float32)).to(torch.bfloat16).float().numpy()
    assert np.array_equal(y, want)


@pytest.mark.parametrize("M,N,K", [
    (1, 64, 128), (3, 40, 320), (8, 512, 3584), (8, 3584, 3584), (8, 96, 18944),   # the last: K split over ranges of workgroups
    (16, 1000, 2112), (32, 130, 5120), (9, 33, 27648),
    # more than 32 tokens: the GEMM (x quantised by a launch of its own); ragged token blocks, row tiles and a half step of K
    (33, 64, 128), (64, 130, 320), (130, 1000, 2112), (300, 96, 96), (200, 3584, 3584), (513, 40, 32), (1100, 5120, 1024),
])
def test_native_linear_is_the_product_of_the_quantised_operands(M, N, K):
    """Products of FP8 and FP4 values are exact and the sums are fp32: the result is held to the same gate as the
    NVFP4 linear (2^-8 |y| + 1e-3 row maximum), against the oracle's float64 product of the two quantised operands."""
    print("mx linear case", M, N, K, flush=True)
    x, codes, scales, pw = _problem(M, N, K, 100 + M + N)
    y = qerl.mxfp4_linear_native(x.cuda(), pw)
    torch.cuda.synchronize()
    check_linear(y, mx.mx_linear_native(x.float().numpy(), codes, scales), ("mx native", M, N, K))
    again = qerl.mxfp4_linear_native(x.cuda(), pw)
    assert torch.equal(y, again)


@pytest.mark.parametrize("M,N,K,r,with_bias", [
    (1, 64, 128, 8, True), (3, 40, 320, 16, False), (8, 512, 3584, 32, True), (8, 96, 18944, 64, True),   # K split over ranges
    (16, 1000, 2112, 32, False), (32, 130, 5120, 128, True), (9, 33, 27648, 24, True), (5, 3584, 3584, 0, True),
    (33, 64, 128, 8, True), (64, 130, 320, 32, False), (130, 1000, 2112, 64, True), (300, 96, 96, 40, True),
    (200, 3584, 3584, 32, True), (1100, 5120, 1024, 128, True), (513, 40, 32, 0, True),
])
def test_native_linear_with_lora_and_bias(M, N, K, r, with_bias):
    """Eq. (2) on the native product: the adapter reads bf16 x; the sum is held to the linear's gate against the
    oracle's float64 composition.  Twice through one workspace (the K-parts' counters are left at zero), bit-equal;
    without adapter and bias the entry point gives the plain native linear's bits."""
    print("mx lora linear case", M, N, K, r, with_bias, flush=True)
    x, codes, scales, pw = _problem(M, N, K, 300 + M + N + r)
    rng = np.random.default_rng(1000 + M + r)
    A = _bf16(rng.standard_normal((r, K)).astype(np.float32) / np.sqrt(K)) if r else None
    B = _bf16(rng.standard_normal((N, r)).astype(np.float32) * 0.05) if r else None
    bias = _bf16(rng.standard_normal(N).astype(np.float32) * 0.1) if with_bias else None
    ws = qerl.Workspace(qerl.load_library().mxfp4_lora_linear_native_workspace_bytes(M, N, K, r))
    cu = lambda t: None if t is None else t.cuda()
    y = qerl.mxfp4_lora_linear_native(x.cuda(), pw, cu(A), cu(B), 1.5, cu(bias), workspace=ws)
    torch.cuda.synchronize()
    nf = lambda t: None if t is None else t.float().numpy()
    check_linear(y, mx.mx_lora_linear_native(x.float().numpy(), codes, scales, nf(A), nf(B), 1.5, nf(bias)), ("mx lora", M, N, K, r))
    again = qerl.mxfp4_lora_linear_native(x.cuda(), pw, cu(A), cu(B), 1.5, cu(bias), workspace=ws)
    assert torch.equal(y, again)
    plain = qerl.mxfp4_lora_linear_native(x.cuda(), pw, workspace=ws)
    assert torch.equal(plain, qerl.mxfp4_linear_native(x.cuda(), pw))


def test_native_lora_branch_reads_the_unquantised_activations():
    """A rank-8 adapter whose first row copies one activation into one output: the difference to the plain linear is
    that activation itself (1.0625: MXFP8 with the scale of a Gaussian block would make it 1 or 1.125), for few tokens and for the GEMM."""
    N, K = 64, 256
    for M in (4, 40):
        x, codes, scales, pw = _problem(M, N, K, 55 + M)
        x = x.clone()
        x[:, 5] = 1.0625
        A = torch.zeros((8, K), dtype=torch.bfloat16); A[0, 5] = 1.0
        B = torch.zeros((N, 8), dtype=torch.bfloat16); B[2, 0] = 1.0
        base = qerl.mxfp4_linear_native(x.cuda(), pw).float().cpu().numpy().astype(np.float64)
        y = qerl.mxfp4_lora_linear_native(x.cuda(), pw, A.cuda(), B.cuda(), 1.0)
        want = mx.mx_lora_linear_native(x.float().numpy(), codes, scales, A.float().numpy(), B.float().numpy(), 1.0)
        check_linear(y, want, ("lora reads x", M))
        d = y.float().cpu().numpy() - base
        assert not d[:, [0, 1, 3, 4, 5]].any() and np.all(np.abs(d[:, 2] - 1.0625) < 2.0 ** -6)


def test_native_lora_linear_rejects_what_it_cannot_run():
    lib = qerl.load_library()
    assert lib.mxfp4_lora_linear_native_workspace_bytes(8, 64, 128, 136) == 0
    x, codes, scales, pw = _problem(4, 64, 128, 3)
    A = torch.zeros((12, 128), dtype=torch.bfloat16).cuda(); B = torch.zeros((64, 12), dtype=torch.bfloat16).cuda()
    ws = qerl.Workspace(lib.mxfp4_lora_linear_native_workspace_bytes(4, 64, 128, 16))
    with pytest.raises(qerl.QerlError):
        qerl.mxfp4_lora_linear_native(x.cuda(), pw, A, B, 1.0, workspace=ws)       # rank not a multiple of 8
    small = qerl.Workspace(256)
    with pytest.raises(qerl.QerlError):
        qerl.mxfp4_lora_linear_native(x.cuda(), pw, workspace=small)


def test_how_far_the_native_path_is_from_the_weight_only_result():
    """Not a parity claim: the measured cost of rounding activations to MXFP8 on Gaussian inputs, relative to
    each output row's root mean square (the weight-only result is what the paper's kernels compute)."""
    M, N, K = 8, 3584, 3584
    x, codes, scales, pw = _problem(M, N, K, 4242)
    y = qerl.mxfp4_linear_native(x.cuda(), pw).float().cpu().numpy().astype(np.float64)
    ref = mx.mx_linear_weight_only(x.float().numpy(), codes, scales)
    rel_rms = np.sqrt(((y - ref) ** 2).mean(axis=1)) / np.sqrt((ref ** 2).mean(axis=1))
    rel_max = np.abs(y - ref).max(axis=1) / np.abs(ref).max(axis=1)
    print("native vs weight-only: rms error / row rms =", rel_rms.max(), " max error / row max =", rel_max.max(), flush=True)
    assert rel_rms.max() < 0.05 and rel_max.max() < 0.05
    assert rel_max.max() > 2e-3      # and it is not the weight-only result: the activation rounding is visible


def test_native_linear_quantises_awkward_activations_like_the_oracle():
    """Activations with ties, values beyond the largest element after scaling, block-subnormal and zero entries,
    signed zeros and an all-zero block go through the kernel's own MXFP8 conversion: same result as the oracle's."""
    N, K = 64, 256
    _, codes, scales, pw = _problem(1, N, K, 77)
    x = np.zeros((6, K), dtype=np.float32)
    x[0, :8] = [448.0, 208.0, 240.0, 17.0, 19.0, 1.0 / 512, 3.0 / 1024, -0.0]     # ties at 3 mantissa bits; block subnormals
    x[1, 32:40] = [500.0, -499.0, 464.0, 460.0, 1e-3, -1e-3, 2.0 ** -7, 2.0 ** -9]   # clamps to 448; tiny next to large
    x[2, 64:96] = np.linspace(-3.0, 3.0, 32)
    x[3, :] = 2.0 ** -60
    x[4, 128:132] = [2.0 ** 40, -2.0 ** 36, 2.0 ** 33, 2.0 ** 30]
    xt = _bf16(x)
    y = qerl.mxfp4_linear_native(xt.cuda(), pw)
    check_linear(y, mx.mx_linear_native(xt.float().numpy(), codes, scales), ("awkward activations",))

