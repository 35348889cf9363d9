"""Large fp32 layers on the bf16 matrix cores (every fp32 operand split exactly
into three bf16 terms), against the fp64 direct oracle at the edges of the
kernel's tiles: filters, channels and tiles that leave remainders in the
64-filter groups, 16-channel steps and 32- or 64-tile blocks, odd widths (the
last tile's columns past the image), images of which several share a block of
tiles, a single channel step, and F(4x4,3x3), F(2x2,3x3), F(2x2,5x5).

In place of the fused kernel AUTO asks for exactly the filters' split as
workspace, 6 bytes per element of U with the channels in whole steps of 16, which
shows that this kernel runs; in place of the split algorithm it asks for that
algorithm's workspace, and a result that differs from that algorithm's shows it.

Tolerances: the gates of the fp32 paths.  The split drops products below
2^-21 of |u v| (2^-24 on average), inside fp32 rounding, so that the 2-norm error
is no larger than the explicit fp32 algorithm's (1.05 of it is allowed; a wrong
third term exceeds it some hundred times); on integers whose terms fit 16 bits
nothing is dropped and the result is the oracle's exactly, nor where one side has
more bits and the other fits 8."""
import numpy as np
import pytest

import gpu_helpers as h
from test_gpu_bf3_values import err2
from oracle import direct
from paper_1903_01521_amd import binding as B

pytestmark = pytest.mark.gpu

TOL = {2: 1e-4, 4: 1e-3}


def split_bytes(C, K, m, r):
    return -(-K // 16) * -(-C // 16) * (m + r - 1) ** 2 * 1536


# (N, C, H, W, K, m, r)
SHAPES = [
    (33, 64, 56, 56, 64, 4, 3),     # whole tiles, 4 steps, half a 32-tile block at the end
    (70, 77, 29, 27, 50, 4, 3),     # odd: 8 x 7 tiles, blocks across images, C and K ragged
    (300, 61, 13, 14, 64, 4, 3),    # small images: 4 x 4 tiles, a block holds two
    (20, 45, 112, 110, 49, 4, 3),   # one filter in the last block
    (30, 40, 28, 28, 144, 2, 3),    # F(2x2): whole tiles
    (31, 37, 27, 25, 140, 2, 3),    # odd
    (16, 48, 35, 35, 64, 2, 5),     # 5x5, odd
    (41, 39, 34, 36, 60, 2, 5),     # 5x5, whole tiles
    (16, 100, 27, 25, 144, 2, 3),   # in place of the split algorithm
    (48, 100, 27, 25, 144, 4, 3),
]


def _conv(x, g, m, r, flags=0, with_fp32=False):
    N, C, H, W = x.shape
    K = g.shape[0]
    pad = r // 2
    U = h.empty_bytes(B.wino_filter_bytes_r(C, K, m, r))
    B.check(B.wino_filter_transform_r(h.dev(g), U, C, K, m, r))
    wsb = B.wino_workspace_bytes_r(N, C, H, W, K, pad, m, r, flags)
    ws, xd = h.empty_bytes(wsb), h.dev(x)

    def run(flags):
        y = h.empty_bytes(4 * N * K * H * W)
        B.check(B.wino_conv2d_r(xd, U, y, N, C, H, W, K, pad, m, r, flags, ws, wsb))
        return h.host(y).reshape(N, K, H, W)

    def run_at(shift):                       # x and y off 16-byte alignment by floats
        xs = h.dev(np.concatenate([np.full(shift, np.nan, np.float32), x.ravel()]))[shift:]
        y = h.empty_bytes(4 * (N * K * H * W + shift))
        B.check(B.wino_conv2d_r(xs, U, y[shift:], N, C, H, W, K, pad, m, r, flags, ws, wsb))
        return h.host(y)[shift:].reshape(N, K, H, W)

    y = run(flags)
    st, algo, _ = B.wino_plan_r(N, C, H, W, K, pad, m, r, flags)
    assert st == B.WINO_OK
    y32 = run(flags | algo)
    if algo == B.WINO_ALGO_SPLIT:
        assert not np.array_equal(y, y32), "the layer runs on the bf16 matrix cores"
    else:
        assert wsb == split_bytes(C, K, m, r), "the layer runs on the bf16 matrix cores"
    assert np.array_equal(y, run_at(1))
    return (y, y32) if with_fp32 else y


def _reference(x, g, r):
    return direct.conv2d(x, g, r // 2)


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_bf3_edges(shape):
    N, C, H, W, K, m, r = shape
    print(f"bf3 shape={shape}", flush=True)
    rng = np.random.default_rng(sum(shape))
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    g = (rng.standard_normal((K, C, r, r)) * np.sqrt(2.0 / (r * r * C))).astype(np.float32)
    y, y32 = _conv(x, g, m, r, B.WINO_FLAG_RELU, with_fp32=True)
    ref = np.maximum(_reference(x, g, r), 0.0)
    assert np.all(np.isfinite(y))
    err = h.normwise_err(y, ref)
    print(f"  normwise err {err:.2e}, 2-norm {err2(y, ref):.2e}, fp32 {err2(y32, ref):.2e}", flush=True)
    assert err <= (1e-3 if r == 5 else TOL[m])
    assert err2(y, ref) <= 1.05 * err2(y32, ref)
    assert np.array_equal(y, _conv(x, g, m, r, B.WINO_FLAG_RELU))      # bitwise run to run


@pytest.mark.parametrize("shape", [SHAPES[1], SHAPES[5]], ids=lambda s: "x".join(map(str, s)))
def test_bf3_exact_on_integers(shape):
    # |V| <= 100 (m = 4) and |U| <= 576 * 9 / 16: both below 2^16, so no third
    # term is dropped, and every sum is an integer below 2^24.
    N, C, H, W, K, m, r = shape
    print(f"bf3 integers shape={shape}", flush=True)
    rng = np.random.default_rng(5)
    x = rng.integers(-1, 2, (N, C, H, W)).astype(np.float32)
    g = (rng.integers(-1, 2, (K, C, r, r)) * (576 if m == 4 else 4)).astype(np.float32)
    assert np.array_equal(_conv(x, g, m, r).astype(np.float64), _reference(x, g, r))


def wide_inputs(N, C, H, W, K, side):
    """Integers of F(2x2,3x3) whose transformed filters (side "u") or inputs ("v")
    need three terms, with every sum below 2^24 in units of its last bit."""
    rng = np.random.default_rng(9)
    odd = lambda shape, top: ((2 * rng.integers(0, top // 2, shape) + 1) * rng.choice([-1, 1], shape)).astype(np.float32)
    x, g = np.zeros((N, C, H, W), np.float32), np.zeros((K, C, 3, 3), np.float32)
    if side == "u":
        # |U| < 9 * 2^15; a region's four pixels of every third row and column, each in one
        # channel: |M| < 2^20.2, their nine in an output < 2^23.4
        g[:] = 4 * odd(g.shape, 1 << 15)
        i, j = np.meshgrid(range(0, H, 3), range(0, W, 3), indexing="ij")
        for n in range(N):
            x[n, rng.integers(0, C, i.shape), i, j] = rng.choice([-1, 1], i.shape)
    else:
        # |V| < 2^18, U in 0, 1, 2, 4 from one tap in each of two channels: an output's
        # nine |M| add up to at most 2 * 16 * 2^18
        x[:] = odd(x.shape, 1 << 16)
        for k in range(K):
            for c in rng.choice(C, 2, replace=False):
                g[k, c, rng.integers(3), rng.integers(3)] = 4 * rng.choice([-1, 1])
    return x, g


@pytest.mark.parametrize("side", ["u", "v"])
@pytest.mark.parametrize("shape", [SHAPES[4], SHAPES[5]], ids=lambda s: "x".join(map(str, s)))
def test_bf3_exact_on_wide_integers(shape, side):
    N, C, H, W, K, m, r = shape
    print(f"bf3 wide integers shape={shape} side={side}", flush=True)
    x, g = wide_inputs(N, C, H, W, K, side)
    assert np.array_equal(_conv(x, g, m, r).astype(np.float64), _reference(x, g, r))


@pytest.mark.parametrize("scale", [1e-25, 1e25])
def test_bf3_range(scale):
    # the split keeps fp32's exponent range: scaled inputs give scaled results
    N, C, H, W, K, m, r = SHAPES[2]
    print(f"bf3 scale={scale}", flush=True)
    rng = np.random.default_rng(6)
    x = (rng.standard_normal((N, C, H, W)) * scale).astype(np.float32)
    g = (rng.standard_normal((K, C, r, r)) * np.sqrt(2.0 / (9 * C))).astype(np.float32)
    assert h.normwise_err(_conv(x, g, m, r), _reference(x, g, r)) <= TOL[m]


@pytest.mark.parametrize("shape", [SHAPES[4], SHAPES[6], (13, 205, 12, 11, 476, 2, 5)], ids=["bf3", "bf3_5x5", "gemm3"])
def test_workspace_not_16_byte_aligned(shape):
    # counts as none: the fused kernel, which needs none
    N, C, H, W, K, m, r = shape
    print(f"bf3 unaligned workspace shape={shape}", flush=True)
    st, algo, _ = B.wino_plan_r(N, C, H, W, K, r // 2, m, r, 0)
    assert st == B.WINO_OK and algo == B.WINO_ALGO_FUSED
    rng = np.random.default_rng(10)
    x = h.dev(rng.standard_normal((N, C, H, W)))
    g = h.dev(rng.standard_normal((K, C, r, r)) * np.sqrt(2.0 / (r * r * C)))
    U = h.empty_bytes(B.wino_filter_bytes_r(C, K, m, r))
    B.check(B.wino_filter_transform_r(g, U, C, K, m, r))
    wsb = B.wino_workspace_bytes_r(N, C, H, W, K, r // 2, m, r, 0)
    assert wsb > 0
    ws, out = h.empty_bytes(wsb + 16), []
    for flags, w, n in ((0, ws[1:], wsb), (algo, None, 0), (0, ws[4:], wsb)):
        y = h.empty_bytes(4 * N * K * H * W)
        B.check(B.wino_conv2d_r(x, U, y, N, C, H, W, K, r // 2, m, r, flags, w, n))
        out.append(h.host(y))
    assert np.array_equal(out[0], out[1]) and not np.array_equal(out[2], out[1])


@pytest.mark.parametrize("shape", [SHAPES[4], SHAPES[8]], ids=["fused", "split"])
def test_bf3_without_its_workspace(shape):
    # a byte less than AUTO asks for: the fused kernel
    N, C, H, W, K, m, r = shape
    print(f"bf3 without workspace shape={shape}", flush=True)
    st, algo, _ = B.wino_plan_r(N, C, H, W, K, r // 2, m, r, 0)
    assert st == B.WINO_OK and algo == (B.WINO_ALGO_FUSED if shape == SHAPES[4] else B.WINO_ALGO_SPLIT)
    rng = np.random.default_rng(7)
    x = h.dev(rng.standard_normal((N, C, H, W)))
    g = h.dev(rng.standard_normal((K, C, r, r)) * np.sqrt(2.0 / (r * r * C)))
    U = h.empty_bytes(B.wino_filter_bytes_r(C, K, m, r))
    B.check(B.wino_filter_transform_r(g, U, C, K, m, r))
    wsb = B.wino_workspace_bytes_r(N, C, H, W, K, r // 2, m, r, 0)
    ws = h.empty_bytes(wsb)
    out = {}
    for name, flags, w, n in (("exact", 0, ws, wsb), ("short", 0, ws, wsb - 1), ("none", 0, None, 0),
                              ("fused", B.WINO_ALGO_FUSED, None, 0)):
        y = h.empty_bytes(4 * N * K * H * W)
        B.check(B.wino_conv2d_r(x, U, y, N, C, H, W, K, r // 2, m, r, flags, w, n))
        out[name] = h.host(y)
    assert np.array_equal(out["short"], out["fused"]) and np.array_equal(out["none"], out["fused"])
    assert not np.array_equal(out["exact"], out["fused"])


@pytest.mark.parametrize("shape", [(16, 11, 35, 35, 160, 2, 3), (8, 11, 112, 112, 160, 2, 3), (32, 11, 17, 17, 160, 2, 5),
                                   (64, 11, 35, 35, 64, 4, 3)], ids=lambda s: "x".join(map(str, s)))
def test_few_channels_run_on_fp32(shape):
    # below 12 channels the dropped products are as large as the fp32 kernels'
    # own rounding: AUTO is the fp32 algorithm that wino_plan_r names
    N, C, H, W, K, m, r = shape
    print(f"few channels shape={shape}", flush=True)
    rng = np.random.default_rng(8)
    x = h.dev(rng.standard_normal((N, C, H, W)))
    g = h.dev(rng.standard_normal((K, C, r, r)) * np.sqrt(2.0 / (r * r * C)))
    U = h.empty_bytes(B.wino_filter_bytes_r(C, K, m, r))
    B.check(B.wino_filter_transform_r(g, U, C, K, m, r))
    st, algo, _ = B.wino_plan_r(N, C, H, W, K, r // 2, m, r, 0)
    assert st == B.WINO_OK
    out = []
    for flags in (0, algo):
        wsb = B.wino_workspace_bytes_r(N, C, H, W, K, r // 2, m, r, flags)
        y = h.empty_bytes(4 * N * K * H * W)
        B.check(B.wino_conv2d_r(x, U, y, N, C, H, W, K, r // 2, m, r, flags, h.empty_bytes(wsb), wsb))
        out.append(h.host(y))
    assert np.array_equal(*out)
