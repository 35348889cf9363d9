"""1-D fp32 layers in one kernel on the bf16 matrix cores, against the fp64
direct oracle where the kernel can go wrong: filters, tiles and channels that
leave remainders in the 16-filter blocks, filter groups, 32-tile workgroups and
16-channel steps, even and odd step counts, rows whose 16-byte loads begin
before the tensor or end past it, padding wider than the region, odd widths,
tensors that are only 4-byte aligned, every (m, r), either axis.

The explicit three stages round differently, so a result that differs from
theirs shows that AUTO ran this kernel; on the smallest layers, where they are
faster (10.9 against 9.4 to 14 us), AUTO's result is theirs.  Tolerance: the gate of
the 1-D paths, and the three stages' 2-norm error, which a wrong third term exceeds
some hundred times (1.05 of it is allowed)."""
import numpy as np
import pytest

import gpu_helpers as h
from test_gpu_bf3_values import err2
from oracle import direct
from paper_1903_01521_amd import binding as B

pytestmark = pytest.mark.gpu

# (N, C, H, W, K, pad, m, r)
SHAPES = [
    (60, 16, 14, 14, 16, 3, 2, 7),      # one step
    (3, 33, 37, 101, 50, 3, 2, 7),      # odd sizes, 3 steps
    (2, 20, 57, 58, 130, 0, 4, 5),      # no padding, two filter groups, the last with one block
    (100, 17, 9, 20, 40, 9, 6, 3),      # regions wholly outside the image
    (200, 17, 9, 1, 16, 7, 2, 7),       # one column: regions that begin rows before the tensor
    (1200, 13, 7, 3, 7, 2, 4, 5),       # images smaller than a tile row
    (64, 48, 28, 29, 272, 1, 6, 3),     # three filter groups, several rounds of workgroups
    (40, 420, 28, 28, 500, 1, 6, 3),    # 27 steps
    (30, 491, 25, 29, 500, 2, 4, 5),    # 31 steps
]
SMALL = [
    (1, 16, 14, 14, 16, 3, 2, 7),
    (2, 17, 9, 20, 40, 9, 6, 3),
    (2, 17, 9, 1, 16, 7, 2, 7),
    (5, 13, 7, 3, 7, 2, 4, 5),
    (2, 48, 24, 24, 112, 1, 6, 3),
    (9, 48, 8, 16, 96, 3, 2, 7),
]


def _run(x, g, pad, m, r, axis, flags, shift=0):
    N, C, H, W = x.shape
    K = g.shape[0]
    ax = B.WINO_AXIS_W if axis == "w" else B.WINO_AXIS_H
    Ho, Wo = (H, W + 2 * pad - r + 1) if axis == "w" else (H + 2 * pad - r + 1, W)
    U = h.empty_bytes(B.wino_filter_bytes_1d(C, K, m, r))
    B.check(B.wino_filter_transform_1d(h.dev(g), U, C, K, m, r))
    wsb = B.wino_workspace_bytes_1d(N, C, H, W, K, pad, m, r, ax, flags)
    ws, yb = h.empty_bytes(wsb), h.empty_bytes(4 * (N * K * Ho * Wo + shift))
    ws.fill_(float("nan"))
    yb.fill_(float("nan"))
    xb = h.dev(np.concatenate([np.full(shift, np.nan, np.float32), x.ravel()]))
    B.check(B.wino_conv2d_1d(xb[shift:], U, yb[shift:], N, C, H, W, K, pad, m, r, ax, flags, ws, wsb))
    return h.host(yb)[shift:].reshape(N, K, Ho, Wo)


def _case(shape, axis):
    N, C, H, W, K, pad, m, r = shape
    if axis == "h":
        H, W = W, H
    rng = np.random.default_rng(sum(shape))
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    g = (rng.standard_normal((K, C, r)) * np.sqrt(2.0 / (r * C))).astype(np.float32)
    pads = ((0, 0), (0, 0), (0, 0), (pad, pad)) if axis == "w" else ((0, 0), (0, 0), (pad, pad), (0, 0))
    g4 = g[:, :, None, :] if axis == "w" else g[:, :, :, None]
    return x, g, np.maximum(direct.conv2d(np.pad(x, pads), np.ascontiguousarray(g4), 0), 0.0)


@pytest.mark.parametrize("axis", ["w", "h"])
@pytest.mark.parametrize("shape", SHAPES + SMALL, ids=lambda s: "x".join(map(str, s)))
def test_bf3_1d_edges(shape, axis):
    print(f"bf3 1-D shape={shape} axis={axis}", flush=True)
    pad, m, r = shape[5:]
    x, g, ref = _case(shape, axis)
    y = _run(x, g, pad, m, r, axis, B.WINO_FLAG_RELU)
    assert np.all(np.isfinite(y))
    err = h.normwise_err(y, ref)
    staged = _run(x, g, pad, m, r, axis, B.WINO_FLAG_RELU | B.WINO_ALGO_STAGED)
    print(f"  normwise err {err:.2e}, three stages {h.normwise_err(staged, ref):.2e}", flush=True)
    print(f"  2-norm err {err2(y, ref):.2e}, three stages {err2(staged, ref):.2e}", flush=True)
    assert err <= 1e-3 and err2(y, ref) <= 1.05 * err2(staged, ref)
    assert np.array_equal(y, staged) == (shape in SMALL), "which layers run in one kernel"
    assert np.array_equal(y, _run(x, g, pad, m, r, axis, B.WINO_FLAG_RELU, shift=1))   # 4-byte aligned tensors
