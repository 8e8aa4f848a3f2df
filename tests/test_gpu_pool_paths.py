"""Max-pool kernels over strips of rows (3x3, stride 1, bf16, uint8 taps, enough work) against the CPU
oracle: values and taps bit for bit, gradients against the int32-index form's kernels too."""
import numpy as np
import pytest
import torch

import oracle
from paper_1605_08695_amd import ops
from tests.gpu_parity import assert_close, f64, say

pytestmark = pytest.mark.gpu
DEV = "cuda"

# N, H, W, C, pads: row counts on both sides of a multiple of the strip, one row, VALID and uneven pads
CASES = [
    (48, 29, 31, 72, (1, 1, 1, 1)),
    (104, 28, 28, 40, (1, 1, 1, 1)),
    (176, 7, 9, 256, (1, 1, 1, 1)),
    (64, 22, 35, 80, (0, 0, 0, 0)),
    (640, 1, 20, 64, (1, 1, 1, 1)),
    (64, 13, 33, 96, (2, 1, 0, 2)),
]
STRIPS = 3 << 15                                     # fewer strips run the one-output kernels


def _data(kind, shape, rng):
    if kind == "relu":
        return np.maximum(rng.standard_normal(shape), 0.0)
    if kind == "ties":
        return np.maximum(np.round(rng.standard_normal(shape) * 2), 0.0)
    a = np.maximum(rng.standard_normal(shape), 0.0)                       # "special"
    pick = rng.random(shape)
    a[pick < 0.002] = np.nan
    a[(pick > 0.5) & (pick < 0.502)] = -0.0
    a[(pick > 0.6) & (pick < 0.601)] = -1.5
    a[(pick > 0.7) & (pick < 0.71)] = np.inf
    a[(pick > 0.8) & (pick < 0.81)] = 1e-40
    return a


@pytest.mark.parametrize("kind", ["relu", "ties", "special"])
@pytest.mark.parametrize("case", CASES, ids=["x".join(map(str, c[:4])) for c in CASES])
def test_pool_strips(case, kind):
    N, H, W, C, pads = case
    say("pool strips", case, kind)
    rng = np.random.default_rng(3)
    # (the forward reads and writes channel slices)
    x = torch.from_numpy(_data(kind, (N, H, W, C + 8), rng)).to(torch.bfloat16).to(DEV)[..., 8:]
    oh, ow = H + pads[0] + pads[1] - 2, W + pads[2] + pads[3] - 2
    assert N * -(-oh // 4) * ow * (C // 8) >= STRIPS and N * -(-H // 4) * W * (C // 8) >= STRIPS
    yb = torch.full((N, oh, ow, C + 16), 7.0, dtype=torch.bfloat16, device=DEV)
    y8, taps = ops.maxpool_fwd(x, (3, 3), 1, pads, y=yb[..., 8:8 + C], taps=True)
    y, am = ops.maxpool_fwd(x, (3, 3), 1, pads)
    torch.cuda.synchronize()
    assert bool((yb[..., :8] == 7.0).all()) and bool((yb[..., 8 + C:] == 7.0).all())
    ref_y, ref_am = oracle.maxpool_fwd(f64(x), (3, 3), 1, pads)
    for got in (y8, y):
        assert np.array_equal(f64(got), ref_y, equal_nan=True)
        assert np.array_equal(np.signbit(f64(got)), np.signbit(ref_y))
    n, oh, ow, c = np.indices(ref_am.shape, dtype=np.int32)
    t = taps.cpu().numpy().astype(np.int32)
    dense = ((n * H + oh - pads[0] + t // 3) * W + ow - pads[2] + t % 3) * C + c
    assert np.array_equal(dense, ref_am) and np.array_equal(am.cpu().numpy(), ref_am)
    # gradients in and out of channel slices
    wide = torch.from_numpy(rng.standard_normal(y8.shape[:3] + (C + 16,))).to(torch.bfloat16).to(DEV)
    dy = wide[..., 8:8 + C]
    for beta in (0.0, 1.0):
        old = torch.from_numpy(rng.standard_normal((N, H, W, C + 8))).to(torch.bfloat16).to(DEV)
        a, b = old.clone(), old.clone()
        ops.maxpool_bwd(dy, taps, a[..., 8:], (3, 3), 1, pads, beta=beta)
        ops.maxpool_bwd(dy, am, b[..., 8:], (3, 3), 1, pads, beta=beta)
        torch.cuda.synchronize()
        assert torch.equal(a, b)
        ref = oracle.maxpool_bwd(f64(dy), ref_am, (N, H, W, C), dx=f64(old[..., 8:]), beta=beta)
        assert_close(f64(a[..., 8:]), ref, torch.bfloat16, label="gradient beta=%g" % beta)
