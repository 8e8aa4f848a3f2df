"""Convolution kernels at the sizes where their dispatch changes, against the CPU oracle: every
direction, the fused forward and input-gradient epilogues, channel-slice views, and workspaces of
the smallest accepted size."""
import ctypes
import zlib

import numpy as np
import pytest
import torch

import oracle
from paper_1605_08695_amd import ops
from paper_1605_08695_amd._lib import load
from tests.gpu_parity import assert_close, f64, say

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _mk(shape, dtype, rng, scale=1.0):
    return torch.from_numpy(rng.standard_normal(shape) * scale).to(dtype).to(DEV)


def _check_all(name, dtype, N, H, W, C, K, KH, KW, s, pads, wide=0):
    """Forward + bias + ReLU, filter gradient, input gradient (beta 0 and 1) and its fused ReLU
    backward of one convolution; ``wide`` > 0 makes y / dy and x / dx channel slices."""
    say("conv path case", name, dtype)
    rng = np.random.default_rng(zlib.crc32(name.encode()))
    xb = torch.from_numpy(np.maximum(rng.standard_normal((N, H, W, C + wide)), 0.0)).to(dtype).to(DEV)
    x = xb[..., wide:]
    w = _mk((KH, KW, C, K), dtype, rng, np.sqrt(2.0 / (KH * KW * C)))
    bias = torch.from_numpy(rng.standard_normal(K) * 0.5).to(torch.float32).to(DEV)
    pre = oracle.conv2d_fwd(f64(x), f64(w), (s, s), pads)
    yb = torch.full(pre.shape[:3] + (K + wide,), 7.0, dtype=dtype, device=DEV)
    y = ops.conv2d_fwd_bias_relu(x, w, bias, s, pads, y=yb[..., wide:])
    torch.cuda.synchronize()
    assert_close(f64(y), oracle.bias_relu_fwd(pre, f64(bias)), dtype, label="fwd")
    assert bool(torch.all(yb[..., :wide] == 7.0))
    dy = _mk(pre.shape[:3] + (K + wide,), dtype, rng)[..., wide:]
    dw = ops.conv2d_bwd_filter(x, dy, (KH, KW), s, pads)
    torch.cuda.synchronize()
    assert_close(f64(dw), oracle.conv2d_bwd_filter(f64(x), f64(dy), (KH, KW), (s, s), pads), torch.float32, dtype,
                 label="filter gradient")
    for beta in (0.0, 1.0):
        db_ = torch.full((N, H, W, C + wide), 0.5, dtype=dtype, device=DEV)
        dx = db_[..., wide:]
        old = f64(dx)
        ops.conv2d_bwd_input(dy, w, dx, s, pads, beta=beta)
        dpb = torch.full((N, H, W, C + wide), 0.5, dtype=dtype, device=DEV)
        dp, db = ops.conv2d_bwd_input_relu_bwd(dy, w, x, dpb[..., wide:], s, pads, beta=beta)
        torch.cuda.synchronize()
        g = oracle.conv2d_bwd_input(f64(dy), f64(w), tuple(x.shape), (s, s), pads, dx=old, beta=beta)
        assert_close(f64(dx), g, dtype, label="input gradient beta=%g" % beta)
        ref_dp, ref_db = oracle.bias_relu_bwd(f64(x), g)
        assert_close(f64(dp), ref_dp, dtype, label="fused dpre beta=%g" % beta)
        assert_close(f64(db), ref_db, torch.float32, dtype, label="fused db beta=%g" % beta)
        assert bool(torch.all(db_[..., :wide] == 0.5)) and bool(torch.all(dpb[..., :wide] == 0.5))


# N, H, W, C, K, KH, KW, stride, pads, extra channels of the buffers
F32_CASES = [
    # few blocks: 32 x 32 tiles
    ("f32_c4_k4", 1, 5, 7, 4, 4, 3, 3, 1, (1, 1, 1, 1), 0),
    ("f32_c12_k20", 2, 9, 8, 12, 20, 3, 3, 1, (1, 1, 1, 1), 4),             # multiples of 4, not of 8
    ("f32_c96_k100_s2", 2, 15, 14, 96, 100, 3, 3, 2, (0, 0, 0, 0), 0),      # remainders, stride phases
    ("f32_c64_k68", 3, 8, 11, 64, 68, 1, 3, 1, (0, 0, 1, 1), 8),            # remainders, channel slices
    ("f32_c160_k32_tail", 1, 13, 5, 160, 32, 5, 1, 1, (2, 2, 0, 0), 0),     # 65 pixels: one past two tiles
    ("f32_1x1_k1_tile", 1, 8, 8, 32, 64, 1, 1, 1, (0, 0, 0, 0), 0),         # one reduction tile
    ("f32_2tiles", 1, 8, 8, 40, 32, 1, 1, 1, (0, 0, 0, 0), 0),              # two, the second partial
    # 256 blocks and more: 64 x 64 tiles with a channel and a pixel remainder, forward (124 out of K) and input
    # gradient (124 out of C), and 32 x 64 ones (100 channels fill little of a second 64), in channel slices
    ("f32_64x64_k124", 6, 39, 37, 40, 124, 3, 3, 1, (1, 1, 1, 1), 4),
    ("f32_64x64_c124", 6, 39, 37, 124, 40, 3, 3, 1, (1, 1, 1, 1), 12),
    ("f32_32x64_k100", 3, 39, 37, 36, 100, 3, 3, 1, (1, 1, 1, 1), 8),
    ("f32_32x64_c100", 3, 39, 37, 100, 36, 3, 3, 1, (1, 1, 1, 1), 4),
    ("f32_c6_k10", 2, 6, 5, 6, 10, 3, 3, 1, (1, 1, 1, 1), 0),               # register-staged kernel
]


@pytest.mark.parametrize("case", F32_CASES, ids=[c[0] for c in F32_CASES])
def test_conv_f32_paths(case):
    name, N, H, W, C, K, KH, KW, s, pads, wide = case
    _check_all(name, torch.float32, N, H, W, C, K, KH, KW, s, pads, wide)


BF16_CASES = [
    # 64 x 64 tiles with three LDS stages: one, two, three and four reduction tiles, remainders
    ("b64_k1", 1, 9, 9, 64, 72, 1, 1, 1, (0, 0, 0, 0), 0),
    ("b64_k2", 1, 8, 8, 104, 64, 1, 1, 1, (0, 0, 0, 0), 8),
    ("b64_k3", 2, 7, 5, 64, 40, 1, 3, 1, (0, 0, 1, 1), 0),
    ("b64_k4_s2", 2, 11, 9, 24, 96, 3, 3, 2, (1, 1, 1, 1), 0),
    # more than one round of 128 x 128 blocks: 160- and 192-row tiles, forward and input gradient
    ("rows160", 7, 100, 100, 16, 128, 1, 1, 1, (0, 0, 0, 0), 0),
    ("rows160_dx", 7, 100, 100, 128, 16, 1, 1, 1, (0, 0, 0, 0), 0),
    ("rows192", 9, 100, 100, 24, 128, 1, 1, 1, (0, 0, 0, 0), 0),
    ("rows192_dx", 9, 100, 100, 128, 24, 1, 1, 1, (0, 0, 0, 0), 0),
]


@pytest.mark.parametrize("case", BF16_CASES, ids=[c[0] for c in BF16_CASES])
def test_conv_bf16_paths(case):
    name, N, H, W, C, K, KH, KW, s, pads, wide = case
    _check_all(name, torch.bfloat16, N, H, W, C, K, KH, KW, s, pads, wide)


# stride phases renumbered by themselves: with no taps in three of four, with 4, 2, 2 and 1, and 9, 6, 6
# and 4, over block counts that are not multiples of the 8 XCDs, aligned and padded channels
PHASE_CASES = [
    ("phases_1x1_s2", torch.bfloat16, 20, 61, 61, 136, 64, 1, 1, 2, (0, 0, 0, 0), 8),
    ("phases_3x3_s2", torch.bfloat16, 9, 45, 46, 72, 40, 3, 3, 2, (1, 0, 1, 0), 0),
    ("phases_5x5_s2", torch.bfloat16, 24, 57, 57, 64, 8, 5, 5, 2, (2, 2, 2, 2), 0),
    ("phases_1x3_s3", torch.bfloat16, 7, 40, 50, 96, 32, 1, 3, 3, (0, 0, 1, 1), 0),
    ("phases_f32_3x3_s2", torch.float32, 6, 41, 41, 36, 20, 3, 3, 2, (1, 1, 1, 1), 0),
    ("phases_pad_c37_s2", torch.bfloat16, 9, 45, 46, 37, 72, 3, 3, 2, (1, 1, 1, 1), 3),
]


@pytest.mark.parametrize("case", PHASE_CASES, ids=[c[0] for c in PHASE_CASES])
def test_conv_stride_phases(case):
    name, dtype, N, H, W, C, K, KH, KW, s, pads, wide = case
    _check_all(name, dtype, N, H, W, C, K, KH, KW, s, pads, wide)


# channel counts that are not multiples of a 16-byte chunk: padded copies in the workspace and the
# element-wise epilogue (one or both counts odd, strided phases, channel slices at odd offsets, 64-
# and 128-channel tiles)
PAD_CASES = [
    ("pad_c21_k64", torch.bfloat16, 12, 33, 31, 21, 64, 3, 3, 1, (1, 1, 1, 1), 0),
    ("pad_c64_k37", torch.bfloat16, 5, 41, 25, 64, 37, 3, 3, 1, (1, 1, 1, 1), 0),
    ("pad_c45_k131_s2", torch.bfloat16, 16, 29, 30, 45, 131, 3, 3, 2, (1, 0, 1, 0), 0),
    ("pad_c99_k203_slices", torch.bfloat16, 6, 23, 21, 99, 203, 1, 3, 1, (0, 0, 1, 1), 5),
    ("pad_c250_k250_wide", torch.bfloat16, 9, 64, 64, 250, 250, 1, 1, 1, (0, 0, 0, 0), 0),
    ("pad_small", torch.bfloat16, 1, 9, 11, 9, 70, 3, 3, 1, (1, 1, 1, 1), 0),
    ("pad_f32_c30_k65", torch.float32, 6, 33, 31, 30, 65, 3, 3, 1, (1, 1, 1, 1), 0),
    ("pad_f32_c64_k7_s2", torch.float32, 36, 35, 33, 64, 7, 5, 5, 2, (2, 2, 2, 2), 3),
]


@pytest.mark.parametrize("case", PAD_CASES, ids=[c[0] for c in PAD_CASES])
def test_conv_padded_channels(case):
    name, dtype, N, H, W, C, K, KH, KW, s, pads, wide = case
    x = torch.empty((N, H, W, C), dtype=dtype, device=DEV)
    # (the query asks for the padded copies; their filter alone is more than nothing)
    assert ops.conv2d_workspace_bytes(0, x, K, KH, KW, s, pads) >= KH * KW * C * K * x.element_size()
    _check_all(name, dtype, N, H, W, C, K, KH, KW, s, pads, wide)


@pytest.mark.parametrize("dtype,C,K", [(torch.bfloat16, 45, 131), (torch.bfloat16, 64, 37), (torch.float32, 30, 66)])
def test_conv_padded_channels_deferred_bias(dtype, C, K):
    """The fused input gradient over padded copies with its bias partials left for a later sum: the
    partials lie in the workspace it was given, and their sum has the bits of the immediate form."""
    rng = np.random.default_rng(C)
    N, H, W, p = 5, 23, 21, (1, 1, 1, 1)
    y = torch.from_numpy(np.maximum(rng.standard_normal((N, H, W, C)), 0.0)).to(dtype).to(DEV)
    w, dy = _mk((3, 3, C, K), dtype, rng, 0.05), _mk((N, H, W, K), dtype, rng)
    need = ops.conv2d_workspace_bytes(3, y, K, 3, 3, 1, p)
    assert need >= 9 * C * K * y.element_size()                             # (the padded filter at least)
    dp, db = ops.conv2d_bwd_input_relu_bwd(dy, w, y, torch.empty_like(y), 1, p)
    ws = torch.empty((need + 15) // 16 * 16, dtype=torch.uint8, device=DEV)
    dp2, job = ops.conv2d_bwd_input_relu_bwd(dy, w, y, torch.empty_like(y), 1, p, ws=ws, defer=True)
    assert ws.data_ptr() <= job.part and job.part + job.rows * C * 4 <= ws.data_ptr() + need
    db2 = torch.full((C,), 3.0, device=DEV)
    ops.bias_grad_finish([(job, db2)])
    torch.cuda.synchronize()
    assert torch.equal(dp, dp2) and torch.equal(db, db2)


# short reductions over large tensors: gathered (or, fp32 with whole chunks, register-staged) instead
SHORT_CASES = [
    ("short_c33_k64", torch.bfloat16, 30, 33, 31, 33, 64, 1, 1, 1, (0, 0, 0, 0), 0),
    ("short_c64_k9", torch.bfloat16, 30, 33, 31, 64, 9, 1, 1, 1, (0, 0, 0, 0), 0),
    ("short_f32_c42_k10", torch.float32, 30, 33, 31, 42, 10, 1, 1, 1, (0, 0, 0, 0), 3),
    ("short_f32_c100_k32_s2", torch.float32, 44, 31, 31, 100, 32, 1, 1, 2, (0, 0, 0, 0), 0),
    ("few_pixels_c75_k88", torch.bfloat16, 1, 5, 5, 75, 88, 3, 3, 1, (0, 0, 0, 0), 0),
    ("phase_c35_k66_s2", torch.bfloat16, 34, 31, 31, 35, 66, 1, 1, 2, (0, 0, 0, 0), 3),
    ("phase_f32_c35_k33_s2", torch.float32, 5, 31, 31, 35, 33, 1, 1, 2, (0, 0, 0, 0), 0),
    ("large_f32_c81_k12", torch.float32, 30, 59, 59, 81, 12, 1, 1, 1, (0, 0, 0, 0), 0),
    ("large_f32_c165_k4_s2", torch.float32, 30, 59, 59, 165, 4, 1, 1, 2, (0, 0, 0, 0), 0),
]


@pytest.mark.parametrize("case", SHORT_CASES, ids=[c[0] for c in SHORT_CASES])
def test_conv_short_reductions(case):
    name, dtype, N, H, W, C, K, KH, KW, s, pads, wide = case
    _check_all(name, dtype, N, H, W, C, K, KH, KW, s, pads, wide)


def test_conv_padded_channels_least_workspace():
    """Without the workspace that the padded copies need (none is required here) the same shapes run
    on the register-staged kernel."""
    lib = load()
    rng = np.random.default_rng(8)
    x, w = _mk((12, 33, 31, 21), torch.bfloat16, rng), _mk((3, 3, 21, 64), torch.bfloat16, rng, 0.1)
    y = torch.empty((12, 33, 31, 64), dtype=torch.bfloat16, device=DEV)
    rc = lib.tfk_conv2d_fwd(ops._ptr(x), ops.nhwc(x), ops._ptr(w), 64, ops.window(3, 3, 1, (1, 1, 1, 1)), 1, ops._ptr(y),
                            ops.nhwc(y), None, 0, ops._stream(None))
    assert rc == 0
    torch.cuda.synchronize()
    assert_close(f64(y), oracle.conv2d_fwd(f64(x), f64(w), 1, (1, 1, 1, 1)), torch.bfloat16, label="no workspace")


def _relu_bwd_with_workspace(dy, w, y, nbytes):
    lib = load()
    ws = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
    dp, db = torch.empty_like(y), torch.empty(y.shape[3], dtype=torch.float32, device=DEV)
    rc = lib.tfk_conv2d_bwd_input_relu_bwd(
        ops._ptr(dy), ops.nhwc(dy), ops._ptr(w), ops.window(3, 3, 1, (1, 1, 1, 1)), ops._dt(y), ops._ptr(y),
        ops._ptr(dp), ops.nhwc(y), ctypes.c_float(0.0), ops._ptr(db), ops._ptr(ws), nbytes, ops._stream(None))
    assert rc == 0
    torch.cuda.synchronize()
    return dp, db


@pytest.mark.parametrize("dtype,least", [
    (torch.float32, lambda y: ops.bias_relu_bwd_workspace_bytes(y)),
    # 64 x 128 tiles: two rows of partials per block (more than the unfused pair's here)
    (torch.bfloat16, lambda y: max(ops.bias_relu_bwd_workspace_bytes(y), 2 * (-(-y[..., 0].numel() // 128)) * y.shape[3] * 4)),
], ids=["f32", "bf16"])
def test_conv_relu_bwd_least_workspace(dtype, least):
    """A workspace that holds the partials of the unfused pair (fp32) or of 64 x 128 tiles (bf16),
    but not those of the tiles the rule takes, is accepted and gives the same gradient (the bias
    gradient up to the order of its fp32 sums)."""
    rng = np.random.default_rng(5)
    N, H, W, C, K = 8, 28, 28, 96, 64
    y = torch.from_numpy(np.maximum(rng.standard_normal((N, H, W, C)), 0.0)).to(dtype).to(DEV)
    w, dy = _mk((3, 3, C, K), dtype, rng, 0.05), _mk((N, H, W, K), dtype, rng)
    want = ops.conv2d_workspace_bytes(3, y, K, 3, 3, 1, (1, 1, 1, 1))
    assert least(y) <= want
    a, b = _relu_bwd_with_workspace(dy, w, y, want), _relu_bwd_with_workspace(dy, w, y, least(y))
    assert torch.equal(a[0], b[0])
    # N H W = 6272 terms of one fp32 sum each side: 2 * 6272 * 2^-24 of the sum of magnitudes at most
    bound = 2 * N * H * W * 2.0 ** -24 * f64(a[0].abs()).sum(axis=(0, 1, 2))
    assert np.all(np.abs(f64(a[1]) - f64(b[1])) <= bound)


# standalone ReLU backward: partial grids of two blocks per CU (with blocks that get no pixel), of 16
# pixels a block, of one block, and a channel slice
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "f32"])
@pytest.mark.parametrize("P,C,wide", [(8200, 64, 64), (8193, 24, 72), (2304, 768, 768), (2560, 1664, 1664), (37, 72, 72),
                                      (1, 1000, 1000), (9001, 13, 13)])
def test_relu_bwd_partial_grid(P, C, wide, dtype):
    rng = np.random.default_rng(P + C)
    y = torch.from_numpy(np.maximum(rng.standard_normal((1, 1, P, wide)), 0.0)).to(dtype).to(DEV)[..., :C]
    full = _mk((1, 1, P, wide), dtype, rng)
    dy = full[..., :C]
    for yy in (y, None):
        dp, db = ops.bias_relu_bwd(yy, dy, dpre=torch.empty_like(full)[..., :C])
        torch.cuda.synchronize()
        ref_dp, ref_db = oracle.bias_relu_bwd(f64(y) if yy is not None else np.ones(y.shape), f64(dy))
        assert np.array_equal(f64(dp), ref_dp)
        # a sum of P fp32 terms in any order: at most P 2^-24 of the sum of magnitudes
        assert np.all(np.abs(f64(db) - ref_db) <= P * 2.0 ** -24 * np.abs(ref_dp).sum(axis=(0, 1, 2)) + 1e-30)


# first layers (at most 4 channels) on the band kernels: few bands (spread over the workgroups), staged
# columns shifted by one for 16-byte copies (odd left pad, even width), odd widths, one output row, two
# channel blocks, and filter gradients of two and three tap groups
FIRST_CASES = [
    ("first_3x3s1_evenw", 3, 44, 46, 3, 64, 3, 1, (1, 1, 1, 1)),
    ("first_3x3s1_oddw", 2, 21, 33, 3, 128, 3, 1, (1, 1, 1, 1)),
    ("first_3x3s2_valid", 5, 35, 41, 3, 32, 3, 2, (0, 0, 0, 0)),
    ("first_7x7s2_p3", 2, 60, 64, 3, 64, 7, 2, (3, 3, 3, 3)),
    ("first_7x7s2_p3_oddw", 1, 31, 45, 3, 48, 7, 2, (3, 3, 3, 3)),
    ("first_one_row", 1, 3, 250, 4, 64, 3, 1, (0, 0, 1, 1)),
    ("first_wide", 1, 6, 520, 3, 16, 3, 1, (1, 1, 1, 1)),
    ("first_many_bands", 90, 24, 24, 1, 16, 3, 1, (1, 1, 1, 1)),
    # two channel blocks, bands of less than the LDS allows; more bands than workgroups; longer runs than that
    ("first_two_blocks", 5, 33, 35, 3, 112, 11, 1, (5, 5, 5, 5)),
    ("first_runs", 70, 21, 30, 4, 32, 5, 1, (2, 2, 2, 2)),
    ("first_few_groups", 80, 15, 15, 4, 128, 7, 2, (3, 3, 3, 3)),
    # 3 x 3 filter gradients on either side of 64 reduction steps per CU
    ("first_3x3_steps_below", 20, 118, 110, 3, 80, 3, 1, (1, 1, 1, 1)),
    ("first_3x3_steps_above", 20, 120, 110, 3, 80, 3, 1, (1, 1, 1, 1)),
]


# (in place also one pixel into its buffer: a multiple of 8 bytes, not of 16)
@pytest.mark.parametrize("rgbx", [0, 1, 2], ids=["copied", "in_place", "in_place_8"])
@pytest.mark.parametrize("case", FIRST_CASES, ids=[c[0] for c in FIRST_CASES])
def test_first_layer_paths(case, rgbx):
    name, N, H, W, C, K, k, s, pads = case
    say("first layer", name, rgbx)
    rng = np.random.default_rng(zlib.crc32(name.encode()))
    if rgbx:
        x = _mk((N * H * W + rgbx - 1, 4), torch.bfloat16, rng)[rgbx - 1:].view(N, H, W, 4)[..., :C]
        assert x.data_ptr() % 16 == 8 * (rgbx - 1)
    else:
        x = _mk((N, H, W, C), torch.bfloat16, rng)
    w = _mk((k, k, C, K), torch.bfloat16, rng, np.sqrt(2.0 / (k * k * C)))
    bias = torch.from_numpy(rng.standard_normal(K) * 0.5).to(torch.float32).to(DEV)
    y = ops.conv2d_fwd_bias_relu(x, w, bias, s, pads)
    plain = ops.conv2d_fwd(x, w, s, pads)
    torch.cuda.synchronize()
    pre = oracle.conv2d_fwd(f64(x), f64(w), (s, s), pads)
    assert_close(f64(plain), pre, torch.bfloat16, label="fwd")
    assert_close(f64(y), oracle.bias_relu_fwd(pre, f64(bias)), torch.bfloat16, label="fwd + bias + relu")
    dy = _mk(pre.shape, torch.bfloat16, rng)
    dw = torch.full((k, k, C, K), 3.0, device=DEV)
    ops.conv2d_bwd_filter(x, dy, (k, k), s, pads, dw=dw)
    torch.cuda.synchronize()
    assert_close(f64(dw), oracle.conv2d_bwd_filter(f64(x), f64(dy), (k, k), (s, s), pads), torch.float32, torch.bfloat16,
                 label="filter gradient")


# one or two channels whose fold (strides, pads and width divisible by 4 or 8) is narrower than 4 channels
@pytest.mark.parametrize("N,H,W,C,K,k,s,pads", [(19, 108, 20, 2, 64, 5, 4, (0, 0, 0, 0)), (2, 64, 64, 1, 16, 8, 8, (0, 0, 0, 0)),
                                                (3, 33, 40, 1, 32, 5, 4, (4, 1, 4, 0))])
def test_first_layer_narrow_fold(N, H, W, C, K, k, s, pads):
    """The queried workspace (the band kernel) and the least that is accepted (the fold: its copy of x and
    its filter): both give the oracle's outputs and leave what follows the workspace alone."""
    say("first layer, narrow fold", N, H, W, C, K, k, s)
    lib = load()
    rng = np.random.default_rng(C)
    x, w = _mk((N, H, W, C), torch.bfloat16, rng), _mk((k, k, C, K), torch.bfloat16, rng, 0.2)
    ref = oracle.conv2d_fwd(f64(x), f64(w), (s, s), pads)
    F = max(f for f in (1, 2, 4, 8) if 8 // f >= C and s % f == 0 and pads[2] % f == 0 and W % f == 0)
    up = lambda b: -(-b // 256) * 256
    least = up(N * H * W * (8 // F) * 2) + up(k * -(-k // F) * 8 * K * 2)
    queried = ops.conv2d_workspace_bytes(0, x, K, k, k, s, pads)
    assert 8 // F < 4 and queried > least
    for nbytes in (queried, least):
        ws = torch.full((nbytes + 4096,), 0x5a, dtype=torch.uint8, device=DEV)
        y = torch.empty(ref.shape, dtype=torch.bfloat16, device=DEV)
        rc = lib.tfk_conv2d_fwd(ops._ptr(x), ops.nhwc(x), ops._ptr(w), K, ops.window(k, k, s, pads), 1, ops._ptr(y), ops.nhwc(y),
                                ops._ptr(ws), nbytes, ops._stream(None))
        assert rc == 0
        torch.cuda.synchronize()
        assert_close(f64(y), ref, torch.bfloat16, label="%d bytes" % nbytes)
        assert bool((ws[nbytes:] == 0x5a).all())


def _kernels_of(call):
    """Kernel launches of one call, from a stream capture of it."""
    lib = load()
    for name in ("hipStreamBeginCapture", "hipStreamEndCapture", "hipGraphGetNodes", "hipGraphDestroy"):
        getattr(lib, name).restype = ctypes.c_int
    s = torch.cuda.Stream()
    call(s)                                  # (outside the capture once: code objects load)
    torch.cuda.synchronize()
    st, graph, n = ctypes.c_void_p(s.cuda_stream), ctypes.c_void_p(), ctypes.c_size_t(0)
    assert lib.hipStreamBeginCapture(st, ctypes.c_int(1)) == 0            # (thread-local mode)
    try:
        call(s)
    finally:
        assert lib.hipStreamEndCapture(st, ctypes.byref(graph)) == 0
    assert lib.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    assert lib.hipGraphDestroy(graph) == 0
    return n.value


# one round of two 128-row blocks per CU with the pool in the kernel; more rounds, counted in 128-row tiles
# whatever tile the convolution alone takes (VGG-16's conv10 + pool4 and conv7 + pool3 at small batches)
@pytest.mark.parametrize("N,H,C,K,ps,pk,kernels", [(128, 13, 256, 256, 2, 3, 1), (12, 56, 128, 256, 2, 2, 2), (24, 28, 256, 512, 2, 2, 2),
                                                   (20, 28, 256, 512, 2, 2, 1)])
def test_pool_in_the_convolution_for_one_round(N, H, C, K, ps, pk, kernels):
    rng = np.random.default_rng(2)
    x, w = _mk((N, H, H, C), torch.bfloat16, rng), _mk((3, 3, C, K), torch.bfloat16, rng, 0.03)
    bias = torch.zeros(K, device=DEV)
    y = torch.empty((N, H, H, K), dtype=torch.bfloat16, device=DEV)
    o = (H - pk) // ps + 1
    py = torch.empty((N, o, o, K), dtype=torch.bfloat16, device=DEV)
    taps = torch.empty((N, o, o, K), dtype=torch.uint8, device=DEV)
    assert ops.conv2d_workspace_bytes(0, x, K, 3, 3, 1, (1, 1, 1, 1)) == 0

    def call(s):
        ops.conv2d_fwd_bias_relu_maxpool(x, w, bias, 1, (1, 1, 1, 1), (pk, pk), ps, (0, 0, 0, 0), y=y, py=py, taps=taps, stream=s)
    assert _kernels_of(call) == kernels
    ref_y = ops.conv2d_fwd_bias_relu(x, w, bias, 1, (1, 1, 1, 1))
    ref_py, ref_taps = ops.maxpool_fwd(ref_y, (pk, pk), ps, (0, 0, 0, 0), taps=True)
    torch.cuda.synchronize()
    assert torch.equal(y, ref_y) and torch.equal(py, ref_py) and torch.equal(taps, ref_taps)
