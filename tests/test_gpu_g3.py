"""Deep fp32 layers as three stages with the GEMMs on the bf16 matrix cores (the
filters and the transformed input stored as three bf16 terms), against the fp64
direct oracle at the edges of the kernel's tiles: filters, tiles and channels
that leave remainders in the 128-filter, 128-tile and 16-channel blocks, step
counts of every residue of the kernel's unrolled loop, NCHW and channel-last
tensors (by tile rows, and by region for other channel counts and widths).

A layer runs this path when AUTO asks for exactly its workspace.  Tolerances:
the gates of the fp32 paths."""
import numpy as np
import pytest

import gpu_helpers as h
from oracle import direct
from paper_1903_01521_amd import binding as B

pytestmark = pytest.mark.gpu

TOL = {2: 1e-4, 4: 1e-3}


def workspace(T, P, C, K):
    KB, PB, C16 = -(-K // 16), -(-P // 16), -(-C // 16)
    up = lambda v: -(-v // 256) * 256
    return up(KB * C16 * T * 1536) + up(PB * C16 * T * 1536) + PB * KB * T * 1024


# (N, C, H, W, K, m, layouts): steps 29, 31, 23, 29, 34; whole and ragged tiles
SHAPES_2D = [
    (16, 456, 28, 28, 512, 4, "both"),
    (12, 491, 27, 25, 390, 4, "nchw"),
    (16, 362, 30, 26, 500, 4, "both"),      # C % 4 != 0: channel-last by region
    (32, 456, 14, 14, 500, 2, "both"),
    (48, 536, 13, 15, 500, 2, "both"),
]


def _inputs(N, C, H, W, K, R, S, seed):
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    g = (rng.standard_normal((K, C, R, S)) * np.sqrt(2.0 / (R * S * C))).astype(np.float32)
    return x, g


def _check(y, ref, tol):
    assert np.all(np.isfinite(y))
    err = h.normwise_err(y, ref)
    print(f"  normwise err {err:.2e}", flush=True)
    assert err <= tol


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
        out = h.host(y)
        out = out.reshape(N, H, W, K).transpose(0, 3, 1, 2) if nhwc else out.reshape(N, K, H, W)
        _check(out, ref, TOL[m])


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
