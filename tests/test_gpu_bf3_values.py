"""Values at the ends of fp32's range on the kernels that split their operands in
three bf16 terms (AUTO's k_bf3, k_gemm3 and k_bf3_1d): infinities and NaN in x
and in the filters, with and without ReLU, against the three stages on fp32
MFMA.  Where those give an infinity, a NaN or (ReLU of a NaN) a zero, so must
AUTO; the other values agree within the gates of the fp32 paths."""
import numpy as np
import pytest
import torch

import gpu_helpers as h
from oracle import direct
from paper_1903_01521_amd import binding as B

pytestmark = pytest.mark.gpu

# name: (entry, N, C, H, W, K, pad, m, r), the layers of the kernels' edge tests
LAYERS = {
    "bf3_f4": ("2d", 33, 64, 56, 56, 64, 1, 4, 3),
    "bf3_f4_ragged": ("2d", 70, 77, 29, 27, 50, 1, 4, 3),
    "bf3_f2": ("2d", 31, 37, 27, 25, 140, 1, 2, 3),
    "bf3_5x5": ("2d", 16, 48, 35, 35, 64, 2, 2, 5),
    "g3_f2": ("2d", 48, 536, 13, 15, 500, 1, 2, 3),
    "g3_f4": ("2d", 12, 491, 27, 25, 390, 1, 4, 3),
    "g3_nhwc": ("nhwc", 16, 456, 28, 28, 512, 1, 4, 3),
    "1d_w": ("w", 3, 33, 37, 101, 50, 3, 2, 7),
    "1d_h": ("h", 2, 20, 58, 57, 130, 2, 4, 5),
}


def make(name, seed=11):
    entry, N, C, H, W, K, pad, m, r = LAYERS[name]
    gen = torch.Generator(device=h.DEV).manual_seed(seed)
    x = torch.randn((N, H, W, C) if entry == "nhwc" else (N, C, H, W), generator=gen, device=h.DEV)
    taps = (r,) if entry in "wh" else (r, r)
    g = torch.randn((K, C) + taps, generator=gen, device=h.DEV) * (2.0 / (C * np.prod(taps))) ** 0.5
    return x, g


def run(name, x, g, flags):
    """The layer's y as [N][K][Ho][Wo], and the workspace it asked for."""
    entry, N, C, H, W, K, pad, m, r = LAYERS[name]
    if entry in "wh":
        axis = {"w": B.WINO_AXIS_W, "h": B.WINO_AXIS_H}[entry]
        U = h.empty_bytes(B.wino_filter_bytes_1d(C, K, m, r))
        B.check(B.wino_filter_transform_1d(g, U, C, K, m, r))
        wsb = B.wino_workspace_bytes_1d(N, C, H, W, K, pad, m, r, axis, flags)
        Ho, Wo = H + (2 * pad - r + 1) * (entry == "h"), W + (2 * pad - r + 1) * (entry == "w")
    else:
        U = h.empty_bytes(B.wino_filter_bytes_r(C, K, m, r))
        B.check(B.wino_filter_transform_r(g, U, C, K, m, r))
        wsb = B.wino_workspace_bytes_nhwc(N, C, H, W, K, pad, m, flags) if entry == "nhwc" else \
            B.wino_workspace_bytes_r(N, C, H, W, K, pad, m, r, flags)
        Ho, Wo = H + 2 * pad - r + 1, W + 2 * pad - r + 1
    assert wsb < 2**63
    ws, y = h.empty_bytes(wsb), h.empty_bytes(4 * N * K * Ho * Wo)
    if entry in "wh":
        st = B.wino_conv2d_1d(x, U, y, N, C, H, W, K, pad, m, r, axis, flags, ws, wsb)
    elif entry == "nhwc":
        st = B.wino_conv2d_nhwc(x, U, y, N, C, H, W, K, pad, m, flags, ws, wsb)
    else:
        st = B.wino_conv2d_r(x, U, y, N, C, H, W, K, pad, m, r, flags, ws, wsb)
    B.check(st)
    y = h.host(y)
    return y.reshape(N, Ho, Wo, K).transpose(0, 3, 1, 2) if entry == "nhwc" else y.reshape(N, K, Ho, Wo)


def same(name, x, g, flags):
    tol = 1e-4 if LAYERS[name][7:] == (2, 3) else 1e-3
    y, ref = run(name, x, g, flags), run(name, x, g, flags | B.WINO_ALGO_STAGED)
    assert not np.array_equal(y, ref, equal_nan=True), "AUTO runs on the bf16 matrix cores"
    for what in (np.isnan, np.isposinf, np.isneginf):
        assert np.array_equal(what(y), what(ref)), (what.__name__, what(y).sum(), what(ref).sum())
    ok = np.isfinite(ref)
    assert np.abs(y[ok] - ref[ok]).max() <= tol * np.abs(ref[ok]).max()
    return ref


@pytest.mark.parametrize("relu", [0, B.WINO_FLAG_RELU], ids=["plain", "relu"])
@pytest.mark.parametrize("name", LAYERS)
def test_nonfinite_inputs(name, relu):
    print(f"non-finite inputs {name} relu={relu}", flush=True)
    x, g = make(name)
    n, a, b = x.shape[:3]
    x[0, a // 2, b // 3, 7] = float("inf")
    x[n - 1, 0, 0, 0] = -float("inf")
    x[n - 1, a - 1, b - 1, -1] = float("inf")      # the tensor's last element
    x[n // 2, 1, 2, 3] = float("nan")
    x[1, a - 2, b - 2, 5] = 3.0e38                 # overflows in the transforms and sums
    ref = same(name, x, g, relu)
    if LAYERS[name][0] in "wh" or LAYERS[name][7:] == (2, 3):
        assert np.isposinf(ref).any()              # not only NaN
    if not relu:
        assert np.isnan(ref).any()


@pytest.mark.parametrize("name", LAYERS)
def test_nonfinite_filters(name):
    print(f"non-finite filters {name}", flush=True)
    x, g = make(name)
    flat = g.view(g.shape[0], -1)
    flat[0, 1] = float("inf")
    flat[g.shape[0] // 2, 4] = float("nan")
    flat[-1, -1] = -float("inf")                   # the last filter's last tap
    flat[1, 2] = 3.0e38
    assert not np.isfinite(same(name, x, g, 0)).all()


def err2(y, ref):
    d = y.astype(np.float64) - ref
    return float(np.sqrt((d * d).sum() / (ref * ref).sum()))


# powers of two that x and the filters are scaled by: the smallest that keep every
# output a normal number, U below 2^-126, values past 2^112 and sums past 2^96
SCALES = [(0, 0), (-110, 0), (-120, 0), (0, -110), (0, -118), (60, -118), (-124, 60), (110, -30), (100, 0)]


@pytest.mark.parametrize("name", ["bf3_f4", "bf3_f2", "bf3_5x5", "g3_f2", "g3_nhwc", "1d_w", "1d_h"])
def test_small_and_large_scales(name):
    # AUTO's 2-norm error is no larger than the three stages' (measured 0.86-0.89
    # of it at scale 1; 1.05 leaves room for values that scaling made subnormal),
    # at every scale of the inputs.
    entry, _, _, _, _, _, pad, m, r = LAYERS[name][:9]
    x0, g0 = make(name)
    xd = x0.permute(0, 3, 1, 2) if entry == "nhwc" else x0
    g4 = g0[:, :, None] if entry == "w" else g0[..., None] if entry == "h" else g0
    pads = ((0, 0), (0, 0), (0 if entry == "w" else pad,) * 2, (0 if entry == "h" else pad,) * 2)
    ref0 = direct.conv2d(np.pad(h.host(xd), pads), np.ascontiguousarray(h.host(g4)), 0)
    for sx, sg in SCALES:
        x, g = x0 * 2.0 ** sx, g0 * 2.0 ** sg
        ref = ref0 * 2.0 ** (sx + sg)
        e, e3 = err2(run(name, x, g, 0), ref), err2(run(name, x, g, B.WINO_ALGO_STAGED), ref)
        print(f"  {name} x 2^{sx} g 2^{sg}: {e:.2e}, three stages {e3:.2e}", flush=True)
        assert e <= 1.05 * e3
