"""Deep fp32 layers as three stages with the GEMMs on the bf16 matrix cores (the
filters and the transformed input stored as three bf16 terms), against the fp64
direct oracle at the edges of the kernel's tiles: filters, tiles and channels
that leave remainders in the 128-filter, 128-tile and 16-channel blocks, step
counts of every residue of the kernel's unrolled loop, NCHW and channel-last
tensors (by tile rows, and by region for other channel counts and widths).

A layer runs this path when AUTO asks for exactly its workspace.  Tolerances:
the gates of the fp32 paths, and the 2-norm error of the explicit three stages,
which a wrong third term on either side exceeds some hundred times (AUTO's is
0.85-0.95 of theirs; 1.05 is allowed)."""
import numpy as np
import pytest

import gpu_helpers as h
from test_gpu_bf3 import wide_inputs
from test_gpu_bf3_values import err2
from oracle import direct
from paper_1903_01521_amd import binding as B

pytestmark = pytest.mark.gpu

TOL = {2: 1e-4, 4: 1e-3}


def workspace(T, P, C, K):
    KB, PB, C16 = -(-K // 16), -(-P // 16), -(-C // 16)
    up = lambda v: -(-v // 256) * 256
    return up(KB * C16 * T * 1536) + up(PB * C16 * T * 1536) + PB * KB * T * 1024


# (N, C, H, W, K, m, layouts): steps 29, 31, 23, 29, 34, 24, 26, 27, every residue of 6;
# whole and ragged tiles
SHAPES_2D = [
    (16, 456, 28, 28, 512, 4, "both"),
    (12, 491, 27, 25, 390, 4, "nchw"),
    (16, 362, 30, 26, 500, 4, "both"),      # C % 4 != 0: channel-last by region
    (32, 456, 14, 14, 500, 2, "both"),
    (48, 536, 13, 15, 500, 2, "both"),
    (32, 380, 14, 14, 500, 2, "both"),
    (16, 410, 28, 28, 512, 4, "both"),
    (32, 425, 14, 15, 490, 2, "both"),
]

# (N, C, H, W, K, pad, m, r): 5x5 filters and other paddings, steps 13, 36, 26, 17, 36, 24, 25
SHAPES_R = [
    (13, 205, 12, 11, 476, 2, 2, 5),
    (33, 565, 10, 10, 161, 2, 2, 5),
    (10, 410, 28, 28, 182, 1, 2, 5),
    (16, 270, 14, 14, 300, 2, 2, 5),
    (22, 566, 27, 26, 259, 0, 4, 3),
    (33, 378, 17, 17, 312, 0, 2, 3),
    (20, 400, 19, 18, 390, 2, 2, 3),
]


def _inputs(N, C, H, W, K, R, S, seed):
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    g = (rng.standard_normal((K, C, R, S)) * np.sqrt(2.0 / (R * S * C))).astype(np.float32)
    return x, g


def _check(y, ref, tol, staged=None):
    assert np.all(np.isfinite(y))
    err = h.normwise_err(y, ref)
    print(f"  normwise err {err:.2e}", flush=True)
    assert err <= tol
    if staged is not None:
        e, e3 = err2(y, ref), err2(staged, ref)
        print(f"  2-norm err {e:.2e}, three stages {e3:.2e}", flush=True)
        assert e <= 1.05 * e3


@pytest.mark.parametrize("shape", SHAPES_2D, ids=lambda s: "x".join(map(str, s)))
def test_g3_edges(shape):
    N, C, H, W, K, m, layouts = shape
    print(f"g3 shape={shape}", flush=True)
    x, g = _inputs(N, C, H, W, K, 3, 3, sum(shape[:6]))
    ref = np.maximum(direct.conv2d(x, g, 1), 0.0)
    U = h.filter_transform(g, m)
    P = N * -(-H // m) * -(-W // m)
    for nhwc in (False, True) if layouts == "both" else (False,):
        size = B.wino_workspace_bytes_nhwc if nhwc else B.wino_workspace_bytes
        run = B.wino_conv2d_nhwc if nhwc else B.wino_conv2d
        wsb = size(N, C, H, W, K, 1, m, B.WINO_FLAG_RELU)
        assert wsb == workspace((m + 2) ** 2, P, C, K), "the layer runs on the bf16 matrix cores"
        ws, y = h.empty_bytes(wsb), h.empty_bytes(4 * N * K * H * W)
        ws.fill_(float("nan"))
        y.fill_(float("nan"))
        xd = h.dev(np.ascontiguousarray(x.transpose(0, 2, 3, 1)) if nhwc else x)
        B.check(run(xd, U, y, N, C, H, W, K, 1, m, B.WINO_FLAG_RELU, ws, wsb))
        nchw = lambda a: a.reshape(N, H, W, K).transpose(0, 3, 1, 2) if nhwc else a.reshape(N, K, H, W)
        out = nchw(h.host(y))
        flags = B.WINO_FLAG_RELU | B.WINO_ALGO_STAGED
        wsb = size(N, C, H, W, K, 1, m, flags)
        B.check(run(xd, U, y, N, C, H, W, K, 1, m, flags, h.empty_bytes(wsb), wsb))
        _check(out, ref, TOL[m], nchw(h.host(y)))


@pytest.mark.parametrize("shift", [0, 1], ids=["aligned", "4-byte"])
@pytest.mark.parametrize("shape", SHAPES_R, ids=lambda s: "x".join(map(str, s)))
def test_g3_filters_and_paddings(shape, shift):
    # shift: x and y one float off 16-byte alignment
    N, C, H, W, K, pad, m, r = shape
    print(f"g3 shape={shape} shift={shift}", flush=True)
    x, g = _inputs(N, C, H, W, K, r, r, sum(shape))
    ref = direct.conv2d(x, g, pad)
    Ho, Wo = ref.shape[2:]
    U = h.empty_bytes(B.wino_filter_bytes_r(C, K, m, r))
    B.check(B.wino_filter_transform_r(h.dev(g), U, C, K, m, r))
    xd = h.dev(np.concatenate([np.full(shift, np.nan, np.float32), x.ravel()]))[shift:]
    P = N * -(-Ho // m) * -(-Wo // m)
    out = []
    for flags in (0, B.WINO_ALGO_STAGED):
        wsb = B.wino_workspace_bytes_r(N, C, H, W, K, pad, m, r, flags)
        if not flags:
            assert wsb == workspace((m + r - 1) ** 2, P, C, K), "the layer runs on the bf16 matrix cores"
        ws, y = h.empty_bytes(wsb), h.empty_bytes(4 * (N * K * Ho * Wo + shift))
        B.check(B.wino_conv2d_r(xd, U, y[shift:], N, C, H, W, K, pad, m, r, flags, ws, wsb))
        out.append(h.host(y)[shift:].reshape(N, K, Ho, Wo))
    _check(out[0], ref, 1e-3 if r == 5 else TOL[m], out[1])


@pytest.mark.parametrize("side", ["u", "v"])
@pytest.mark.parametrize("nhwc", [False, True], ids=["nchw", "nhwc"])
def test_g3_exact_on_wide_integers(nhwc, side):
    # one operand needs three terms, the other fits one: nothing is dropped
    N, C, H, W, K, m, _ = SHAPES_2D[4]
    print(f"g3 wide integers nhwc={nhwc} side={side}", flush=True)
    x, g = wide_inputs(N, C, H, W, K, side)
    U = h.filter_transform(g, m)
    size = B.wino_workspace_bytes_nhwc if nhwc else B.wino_workspace_bytes
    wsb = size(N, C, H, W, K, 1, m, 0)
    y = h.empty_bytes(4 * N * K * H * W)
    xd = h.dev(np.ascontiguousarray(x.transpose(0, 2, 3, 1)) if nhwc else x)
    B.check((B.wino_conv2d_nhwc if nhwc else B.wino_conv2d)(xd, U, y, N, C, H, W, K, 1, m, 0, h.empty_bytes(wsb), wsb))
    out = h.host(y)
    out = out.reshape(N, H, W, K).transpose(0, 3, 1, 2) if nhwc else out.reshape(N, K, H, W)
    assert np.array_equal(out.astype(np.float64), direct.conv2d(x, g, 1))


def test_g3_without_its_workspace():
    # less workspace than the path needs: the layer runs as before
    N, C, H, W, K, m, _ = SHAPES_2D[3]
    print(f"g3 fallback shape={SHAPES_2D[3]}", flush=True)
    x, g = _inputs(N, C, H, W, K, 3, 3, 1)
    U = h.filter_transform(g, m)
    xd, y = h.dev(x), h.empty_bytes(4 * N * K * H * W)
    for wsb in (0, B.wino_workspace_bytes(N, C, H, W, K, 1, m, B.WINO_ALGO_SPLIT)):
        y.fill_(float("nan"))
        B.check(B.wino_conv2d(xd, U, y, N, C, H, W, K, 1, m, 0, h.empty_bytes(wsb) if wsb else None, wsb))
        _check(h.host(y).reshape(N, K, H, W), direct.conv2d(x, g, 1), TOL[m])
