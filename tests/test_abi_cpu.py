"""The C-ABI library loads, exports what include/wino.h declares, and rejects
invalid arguments before any HIP call (CPU only: no call here reaches a kernel)."""
import pytest

from paper_1903_01521_amd import binding as B

# A non-null address that is never dereferenced: every call using it carries
# another invalid argument that validation rejects first.
FAKE = 0x1000


def test_library_exports_every_declared_symbol():
    names = B.header_functions()
    assert len(names) >= 12
    so = B.lib()
    for n in names:
        assert hasattr(so, n), n


def test_version_and_status_strings():
    assert B.wino_version() >= 100
    for st in (B.WINO_OK, B.WINO_ERR_INVALID_ARG, B.WINO_ERR_UNSUPPORTED, B.WINO_ERR_WORKSPACE,
               B.WINO_ERR_HIP):
        assert B.wino_status_string(st) and B.wino_status_string(st) != "unknown status"
    assert B.wino_status_string(12345) == "unknown status"


@pytest.mark.parametrize("m,T", [(2, 16), (4, 36)])
def test_filter_bytes(m, T):
    assert B.wino_filter_bytes(64, 64, m) == 4 * T * 64 * 64
    assert B.wino_filter_bytes(3, 20, m) == 4 * T * 4 * 32       # C padded to 4, K to 16
    assert B.wino_filter_bytes(0, 8, m) == 0
    assert B.wino_filter_bytes(8, 0, m) == 0
    assert B.wino_filter_bytes(8, 8, 3) == 0


def test_transform_domain_sizes():
    # N=1, 112x112, pad 1, m=4: 28x28 tiles = 784 -> 49 blocks of 16.
    assert B.wino_input_tf_bytes(1, 64, 112, 112, 1, 4) == 4 * 49 * 16 * 36 * 64
    assert B.wino_gemm_out_bytes(1, 64, 112, 112, 1, 4) == 4 * 49 * 4 * 36 * 256
    # ragged: 57x57 -> 15x15 = 225 tiles -> 15 blocks
    assert B.wino_input_tf_bytes(1, 48, 57, 57, 1, 4) == 4 * 15 * 12 * 36 * 64
    assert B.wino_input_tf_bytes(1, 8, 2, 2, 0, 4) == 0         # Ho < 1


def test_workspace_bytes():
    assert B.wino_workspace_bytes(1, 64, 112, 112, 64, 1, 4, B.WINO_ALGO_FUSED) == 0
    staged = B.wino_workspace_bytes(1, 64, 112, 112, 64, 1, 4, B.WINO_ALGO_STAGED)
    assert staged >= B.wino_input_tf_bytes(1, 64, 112, 112, 1, 4) + B.wino_gemm_out_bytes(1, 64, 112, 112, 1, 4)
    assert B.wino_workspace_bytes(1, 64, 112, 112, 64, 1, 3, 0) == 2**64 - 1
    # split: the blocked V, blocks of 16 consecutive tiles (28 x 28 tiles -> 49 blocks),
    # channel quads rounded up to a multiple of 4 (16 here; C = 20: 5 -> 8 quads, 2 x 15 x 15 tiles -> 29 blocks)
    assert B.wino_workspace_bytes(1, 64, 112, 112, 64, 1, 4, B.WINO_ALGO_SPLIT) == 4 * 49 * 16 * 36 * 64
    assert B.wino_workspace_bytes(2, 20, 30, 30, 64, 1, 2, B.WINO_ALGO_SPLIT) == 4 * 29 * 8 * 16 * 64
    assert B.wino_workspace_bytes(1, 3, 112, 112, 64, 1, 4, B.WINO_ALGO_LOWC) == 0
    assert B.wino_workspace_bytes(1, 64, 112, 112, 64, 1, 4, B.WINO_ALGO_LOWC) == 2**64 - 1   # C > 4
    assert B.wino_workspace_bytes(1, 64, 112, 112, 64, 1, 4, 0x500) == 2**64 - 1


def test_workspace_bytes_on_the_bf16_matrix_cores():
    # In place of the fused kernel: the filters' split, 6 bytes per element of U
    # with the channels in whole steps of 16.  In place of the split algorithm:
    # that algorithm's workspace.
    N, C, H, W, K, m = 33, 64, 56, 56, 64, 4
    assert B.wino_plan_r(N, C, H, W, K, 1, m, 3, 0)[1] == B.WINO_ALGO_FUSED
    assert B.wino_workspace_bytes(N, C, H, W, K, 1, m, 0) == 6 * 36 * 64 * 64
    N, C, H, W, K, m = 64, 256, 56, 56, 256, 4
    assert B.wino_plan_r(N, C, H, W, K, 1, m, 3, 0)[1] == B.WINO_ALGO_SPLIT
    assert B.wino_workspace_bytes(N, C, H, W, K, 1, m, 0) == \
        B.wino_workspace_bytes(N, C, H, W, K, 1, m, B.WINO_ALGO_SPLIT) > 6 * 36 * 256 * 256


@pytest.mark.parametrize("N, C, H, W, K, pad, m, r", [
    (18, 144, 29, 63, 448, 1, 2, 5),      # 421 us, on the bf16 matrix cores 456
    (23, 112, 67, 67, 464, 0, 2, 5),      # 1109, 1196
    (1, 336, 161, 161, 160, 0, 2, 5),     # 337, 366
    (60, 502, 16, 18, 372, 2, 2, 3),      # 289, 331
    (58, 480, 25, 26, 245, 0, 2, 3),      # 327, 362
])
def test_auto_stays_on_fp32_where_it_is_faster(N, C, H, W, K, pad, m, r):
    # AUTO asks for the workspace of the fp32 algorithm that wino_plan_r names
    st, algo, slices = B.wino_plan_r(N, C, H, W, K, pad, m, r, 0)
    assert st == B.WINO_OK and slices == 1
    assert B.wino_workspace_bytes_r(N, C, H, W, K, pad, m, r, 0) == \
        B.wino_workspace_bytes_r(N, C, H, W, K, pad, m, r, algo)


GOOD = dict(N=1, C=4, H=8, W=8, K=4, pad=1, m=4)


def _conv(x=FAKE, U=FAKE, y=FAKE + 0x100000, flags=0, ws=None, wsb=0, **kw):
    a = dict(GOOD)
    a.update(kw)
    return B.wino_conv2d(x, U, y, a["N"], a["C"], a["H"], a["W"], a["K"], a["pad"], a["m"],
                         flags, ws, wsb, None)


@pytest.mark.parametrize("kw,status", [
    (dict(x=None), B.WINO_ERR_INVALID_ARG),
    (dict(U=None), B.WINO_ERR_INVALID_ARG),
    (dict(y=None), B.WINO_ERR_INVALID_ARG),
    (dict(N=0), B.WINO_ERR_INVALID_ARG),
    (dict(C=-1), B.WINO_ERR_INVALID_ARG),
    (dict(H=0), B.WINO_ERR_INVALID_ARG),
    (dict(W=0), B.WINO_ERR_INVALID_ARG),
    (dict(K=0), B.WINO_ERR_INVALID_ARG),
    (dict(pad=-1), B.WINO_ERR_INVALID_ARG),
    (dict(H=2, pad=0), B.WINO_ERR_INVALID_ARG),             # Ho = 0
    (dict(m=3), B.WINO_ERR_UNSUPPORTED),
    (dict(m=6), B.WINO_ERR_UNSUPPORTED),
    (dict(flags=0x80000000), B.WINO_ERR_UNSUPPORTED),        # unknown flag bit
    (dict(flags=0x500), B.WINO_ERR_UNSUPPORTED),             # unknown algorithm
    (dict(flags=B.WINO_ALGO_LOWC, C=5), B.WINO_ERR_UNSUPPORTED),   # low-C kernel needs C <= 4
    (dict(flags=B.WINO_ALGO_SPLIT), B.WINO_ERR_WORKSPACE),   # split needs its workspace
    (dict(flags=B.WINO_ALGO_FUSED | B.WINO_CSPLIT(3)), B.WINO_ERR_UNSUPPORTED),
    (dict(flags=B.WINO_ALGO_FUSED | B.WINO_CSPLIT(8)), B.WINO_ERR_UNSUPPORTED),  # m=4: 2 x 8 > 8 waves
    (dict(flags=B.WINO_BLOCK_1x16 | B.WINO_BLOCK_4x4), B.WINO_ERR_UNSUPPORTED),  # two block shapes
    (dict(flags=B.WINO_ALGO_STAGED), B.WINO_ERR_WORKSPACE),  # no workspace
    (dict(flags=B.WINO_ALGO_STAGED, ws=FAKE + 0x900000, wsb=16), B.WINO_ERR_WORKSPACE),
    (dict(y=FAKE), B.WINO_ERR_INVALID_ARG),                  # y aliases x
    (dict(y=FAKE + 64), B.WINO_ERR_INVALID_ARG),             # y overlaps x
    (dict(N=1 << 20, C=1 << 10, H=1 << 10, W=1 << 10), B.WINO_ERR_INVALID_ARG),   # size overflow
    # an image of 1 GiB of input: past the fused kernel's 32-bit offsets
    (dict(C=256, H=1024, W=1024, K=16, y=FAKE + (1 << 42)), B.WINO_ERR_UNSUPPORTED),
    # 512 MiB images: the staged input transform's blocks span two of them
    (dict(C=128, H=1024, W=1024, K=16, y=FAKE + (1 << 42), flags=B.WINO_ALGO_STAGED), B.WINO_ERR_UNSUPPORTED),
])
def test_conv2d_rejects(kw, status):
    assert _conv(**kw) == status


def test_stage_entry_points_reject():
    assert B.wino_filter_transform(None, FAKE, 4, 4, 4) == B.WINO_ERR_INVALID_ARG
    assert B.wino_filter_transform(FAKE, None, 4, 4, 4) == B.WINO_ERR_INVALID_ARG
    assert B.wino_filter_transform(FAKE, FAKE + 0x10000, 0, 4, 4) == B.WINO_ERR_INVALID_ARG
    assert B.wino_filter_transform(FAKE, FAKE + 0x10000, 4, 4, 5) == B.WINO_ERR_UNSUPPORTED
    assert B.wino_filter_transform(FAKE, FAKE + 4, 4, 4, 4) == B.WINO_ERR_INVALID_ARG    # overlap
    assert B.wino_input_transform(None, FAKE, 1, 4, 8, 8, 1, 4) == B.WINO_ERR_INVALID_ARG
    assert B.wino_input_transform(FAKE, FAKE + 0x100000, 1, 4, 8, 8, -2, 4) == B.WINO_ERR_INVALID_ARG
    assert B.wino_input_transform(FAKE, FAKE + 0x100000, 1, 4, 8, 8, 1, 7) == B.WINO_ERR_UNSUPPORTED
    assert B.wino_input_transform(FAKE, FAKE + (1 << 42), 2, 128, 1024, 1024, 1, 4) == B.WINO_ERR_UNSUPPORTED
    assert B.wino_workspace_bytes(2, 128, 1024, 1024, 16, 1, 4, B.WINO_ALGO_STAGED) == 2**64 - 1
    assert B.wino_batched_gemm(FAKE, None, FAKE, 1, 4, 8, 8, 4, 1, 4) == B.WINO_ERR_INVALID_ARG
    assert B.wino_batched_gemm(FAKE, FAKE, FAKE + 8, 1, 4, 8, 8, 4, 1, 4) == B.WINO_ERR_INVALID_ARG
    assert B.wino_output_transform(None, FAKE, 1, 4, 8, 8, 1, 4) == B.WINO_ERR_INVALID_ARG
    assert B.wino_output_transform(FAKE, FAKE + 0x1000000, 1, 4, 8, 8, 1, 4, 0x100) == B.WINO_ERR_UNSUPPORTED
    assert B.wino_output_transform(FAKE, FAKE + 0x1000000, 0, 4, 8, 8, 1, 4) == B.WINO_ERR_INVALID_ARG
    assert B.wino_maxpool2x2(FAKE, None, 1, 1, 4, 4) == B.WINO_ERR_INVALID_ARG
    assert B.wino_maxpool2x2(FAKE, FAKE + 0x10000, 1, 1, 1, 4) == B.WINO_ERR_INVALID_ARG
    assert B.wino_maxpool2x2(FAKE, FAKE + 4, 1, 1, 4, 4) == B.WINO_ERR_INVALID_ARG     # overlap


def test_5x5_sizes_and_rejections():
    # F(2x2,5x5): T = 36, so U has the F(4x4,3x3) size for the same (C, K).
    assert B.wino_filter_bytes_r(3, 20, 2, 5) == 4 * 36 * 4 * 32
    assert B.wino_filter_bytes_r(3, 20, 2, 3) == B.wino_filter_bytes(3, 20, 2)
    assert B.wino_filter_bytes_r(3, 20, 4, 5) == 0                 # F(4x4,5x5): not supported
    assert B.wino_filter_bytes_r(3, 20, 2, 7) == 0
    # 35x35, pad 2 -> 35x35 output, 18x18 tiles = 324 -> 21 blocks; V + M of the staged path
    ws = B.wino_workspace_bytes_r(1, 48, 35, 35, 64, 2, 2, 5, B.WINO_ALGO_STAGED)
    v = 4 * 21 * 12 * 36 * 64
    assert ws == (v + 255) // 256 * 256 + 4 * 21 * 4 * 36 * 256
    # the fused kernel (the planner's choice) needs none; two row groups of 18
    # positions per unit, so at most 4 channel parts
    for flags in (0, B.WINO_ALGO_FUSED, B.WINO_BLOCK_4x4, B.WINO_CSPLIT(2), B.WINO_ALGO_FUSED | B.WINO_CSPLIT(4)):
        assert B.wino_workspace_bytes_r(1, 48, 35, 35, 64, 2, 2, 5, flags) == 0
    for flags in (B.WINO_ALGO_SPLIT, B.WINO_ALGO_LOWC, B.WINO_CSPLIT(8)):
        assert B.wino_workspace_bytes_r(1, 48, 35, 35, 64, 2, 2, 5, flags) == 2**64 - 1
    assert B.wino_workspace_bytes_r(1, 4, 3, 3, 4, 0, 2, 5, 0) == 2**64 - 1        # Ho < 1
    # the 3x3 calls are the r = 3 case
    assert B.wino_workspace_bytes_r(1, 64, 112, 112, 64, 1, 4, 3, B.WINO_ALGO_STAGED) == \
        B.wino_workspace_bytes(1, 64, 112, 112, 64, 1, 4, B.WINO_ALGO_STAGED)


def test_5x5_entry_points_reject():
    y = FAKE + 0x100000
    assert B.wino_filter_transform_r(None, FAKE, 4, 4, 2, 5) == B.WINO_ERR_INVALID_ARG
    assert B.wino_filter_transform_r(FAKE, FAKE + 0x10000, 4, 4, 4, 5) == B.WINO_ERR_UNSUPPORTED
    assert B.wino_filter_transform_r(FAKE, FAKE + 4 * 25, 4, 4, 2, 5) == B.WINO_ERR_INVALID_ARG  # overlap
    conv = lambda **kw: B.wino_conv2d_r(kw.get("x", FAKE), FAKE + 0x800000, kw.get("y", y), 1, 4, 8, 8, 4,
                                        kw.get("pad", 2), kw.get("m", 2), kw.get("r", 5), kw.get("flags", 0),
                                        kw.get("ws"), kw.get("wsb", 0), None)
    assert conv(flags=B.WINO_ALGO_STAGED) == B.WINO_ERR_WORKSPACE  # the three stages need V and M
    assert conv(flags=B.WINO_ALGO_SPLIT) == B.WINO_ERR_UNSUPPORTED
    assert conv(flags=B.WINO_ALGO_LOWC) == B.WINO_ERR_UNSUPPORTED
    assert conv(flags=B.WINO_CSPLIT(8)) == B.WINO_ERR_UNSUPPORTED
    assert conv(r=7) == B.WINO_ERR_UNSUPPORTED
    assert conv(m=4) == B.WINO_ERR_UNSUPPORTED
    assert conv(pad=-1) == B.WINO_ERR_INVALID_ARG
    assert B.wino_conv2d_r(FAKE, FAKE + 0x800000, y, 1, 4, 3, 3, 4, 0, 2, 5, 0, None, 0, None) == \
        B.WINO_ERR_INVALID_ARG                                     # Ho = -1
    assert conv(y=FAKE + 64) == B.WINO_ERR_INVALID_ARG             # y overlaps x


def test_1d_sizes_and_rejections():
    W_, H_ = B.WINO_AXIS_W, B.WINO_AXIS_H
    assert B.wino_filter_bytes_1d(3, 20, 6, 3) == 4 * 8 * 4 * 32
    assert B.wino_filter_bytes_1d(3, 20, 2, 7) == 4 * 8 * 4 * 32
    assert B.wino_filter_bytes_1d(3, 20, 4, 3) == 0                  # not a supported variant
    # 1x7 on 17x17, pad 3 along W: 17 x 17 output, 17 x 9 tiles = 153 -> 10 blocks
    ws = B.wino_workspace_bytes_1d(1, 192, 17, 17, 160, 3, 2, 7, W_, 0)
    assert ws == (4 * 10 * 48 * 8 * 64 + 255) // 256 * 256 + 4 * 10 * 10 * 8 * 256
    assert B.wino_workspace_bytes_1d(1, 192, 17, 17, 160, 3, 2, 7, H_, 0) == ws   # 9 x 17 tiles, same count
    assert B.wino_workspace_bytes_1d(1, 192, 17, 17, 160, 3, 2, 7, 3, 0) == 2**64 - 1     # unknown axis
    assert B.wino_workspace_bytes_1d(1, 192, 17, 17, 160, 3, 2, 7, W_, B.WINO_ALGO_FUSED) == 2**64 - 1
    assert B.wino_workspace_bytes_1d(1, 4, 5, 5, 4, 0, 2, 7, W_, 0) == 2**64 - 1          # Wo < 1


def test_1d_entry_points_reject():
    y = FAKE + 0x100000
    assert B.wino_filter_transform_1d(None, FAKE, 4, 4, 2, 7) == B.WINO_ERR_INVALID_ARG
    assert B.wino_filter_transform_1d(FAKE, FAKE + 0x10000, 4, 4, 2, 5) == B.WINO_ERR_UNSUPPORTED
    assert B.wino_filter_transform_1d(FAKE, FAKE + 4 * 7, 4, 4, 2, 7) == B.WINO_ERR_INVALID_ARG   # overlap
    conv = lambda **kw: B.wino_conv2d_1d(kw.get("x", FAKE), FAKE + 0x800000, kw.get("y", y), 1, 4, 8, 8, 4,
                                         kw.get("pad", 3), kw.get("m", 2), kw.get("r", 7),
                                         kw.get("axis", B.WINO_AXIS_W), kw.get("flags", 0), None, 0, None)
    assert conv() == B.WINO_ERR_WORKSPACE
    assert conv(axis=0) == B.WINO_ERR_UNSUPPORTED
    assert conv(m=6) == B.WINO_ERR_UNSUPPORTED
    assert conv(flags=B.WINO_ALGO_SPLIT) == B.WINO_ERR_UNSUPPORTED
    assert conv(pad=0, axis=B.WINO_AXIS_H, m=2, r=7) == B.WINO_ERR_WORKSPACE           # Ho = 2: valid
    assert B.wino_conv2d_1d(FAKE, FAKE + 0x800000, y, 1, 4, 5, 5, 4, 0, 2, 7, B.WINO_AXIS_W, 0, None, 0,
                            None) == B.WINO_ERR_INVALID_ARG                           # Wo = -1
    assert conv(y=FAKE + 64) == B.WINO_ERR_INVALID_ARG


def test_nhwc_entry_points():
    staged = B.wino_workspace_bytes(1, 64, 112, 112, 64, 1, 4, B.WINO_ALGO_STAGED)
    assert B.wino_workspace_bytes_nhwc(1, 64, 112, 112, 64, 1, 4, 0) == staged
    assert B.wino_workspace_bytes_nhwc(1, 64, 112, 112, 64, 1, 4, B.WINO_ALGO_FUSED) == 2**64 - 1
    assert B.wino_workspace_bytes_nhwc(1, 64, 112, 112, 64, 1, 3, 0) == 2**64 - 1
    # the split path on channel-last tensors: its blocked V, as for NCHW
    split = B.wino_workspace_bytes(1, 64, 112, 112, 64, 1, 4, B.WINO_ALGO_SPLIT)
    assert B.wino_workspace_bytes_nhwc(1, 64, 112, 112, 64, 1, 4, B.WINO_ALGO_SPLIT) == split
    # AUTO: the three stages below two rounds of split items (here 25 pairs x 1
    # filter group), split at N=64, C=K=256, 56x56 (784 pairs x 4 groups)
    assert B.wino_workspace_bytes_nhwc(1, 64, 112, 112, 64, 1, 4, B.WINO_ALGO_AUTO) == staged
    big_split = B.wino_workspace_bytes(64, 256, 56, 56, 256, 1, 4, B.WINO_ALGO_SPLIT)
    assert B.wino_workspace_bytes_nhwc(64, 256, 56, 56, 256, 1, 4, B.WINO_ALGO_AUTO) == big_split
    assert B.wino_workspace_bytes_nhwc(64, 256, 56, 56, 256, 1, 4, B.WINO_ALGO_STAGED) == \
        B.wino_workspace_bytes(64, 256, 56, 56, 256, 1, 4, B.WINO_ALGO_STAGED)
    # no variant overrides or channel slices on channel-last tensors
    assert B.wino_workspace_bytes_nhwc(64, 256, 56, 56, 256, 1, 4,
                                       B.WINO_ALGO_SPLIT | B.WINO_BLOCK_4x4) == 2**64 - 1
    y = FAKE + 0x100000
    conv = lambda **kw: B.wino_conv2d_nhwc(kw.get("x", FAKE), FAKE + 0x800000, kw.get("y", y), 1, 4, 8, 8, 4,
                                           kw.get("pad", 1), kw.get("m", 4), kw.get("flags", 0), None, 0, None)
    assert conv() == B.WINO_ERR_WORKSPACE
    assert conv(m=3) == B.WINO_ERR_UNSUPPORTED
    assert conv(flags=B.WINO_ALGO_LOWC) == B.WINO_ERR_UNSUPPORTED
    assert conv(pad=-1) == B.WINO_ERR_INVALID_ARG
    assert conv(x=None) == B.WINO_ERR_INVALID_ARG
    assert conv(y=FAKE + 64) == B.WINO_ERR_INVALID_ARG


def test_16bit_operand_entry_points():
    F16, BF16 = B.WINO_PREC_F16, B.WINO_PREC_BF16
    # UH: 2 bytes x T x roundup(C,32) x roundup(K,16)
    assert B.wino_filter_bytes_p(20, 20, 4, F16) == 2 * 36 * 32 * 32
    assert B.wino_filter_bytes_p(20, 20, 2, BF16) == 2 * 16 * 32 * 32
    assert B.wino_filter_bytes_p(37, 5, 4, F16) == 2 * 36 * 64 * 16    # C in 32-channel chunks
    assert B.wino_filter_bytes_p(20, 20, 4, 0) == B.wino_filter_bytes(20, 20, 4)
    assert B.wino_filter_bytes_p(20, 20, 4, 0x30) == 0          # both formats at once
    assert B.wino_filter_bytes_p(20, 20, 3, F16) == 0
    # workspace: VH (8 bytes per lane and position) + fp32 M
    ws = B.wino_workspace_bytes(1, 20, 16, 16, 20, 1, 4, F16)
    vh = 1 * 2 * 36 * 64 * 8                                  # PB = 1 (16 tiles), C16 = 2
    assert ws == (vh + 255) // 256 * 256 + B.wino_gemm_out_bytes(1, 20, 16, 16, 1, 4)
    for flags in (F16 | B.WINO_ALGO_FUSED, F16 | B.WINO_ALGO_LOWC, 0x30):
        assert B.wino_workspace_bytes(1, 20, 16, 16, 20, 1, 4, flags) == 2**64 - 1
    # the split path on 16-bit operands: VH of C16 rounded up to even groups
    # (2 for C = 20: one 32-channel step; 4 for C = 40), no M
    assert B.wino_workspace_bytes(1, 20, 16, 16, 20, 1, 4, BF16 | B.WINO_ALGO_SPLIT) == 1 * 2 * 36 * 64 * 8
    assert B.wino_workspace_bytes(1, 40, 16, 16, 20, 1, 2, F16 | B.WINO_ALGO_SPLIT) == 4 * 4 * 16 * 64 * 8   # 8x8 tiles
    # AUTO: the three stages on small layers, split from two rounds of split
    # items on (N=64, 256 channels, 56x56: 392 tile-block pairs x 4 filter groups)
    assert B.wino_plan_r(1, 20, 16, 16, 20, 1, 4, 3, F16)[1] == B.WINO_ALGO_STAGED
    st, algo, _ = B.wino_plan_r(64, 256, 56, 56, 256, 1, 4, 3, F16)
    assert st == B.WINO_OK and algo == B.WINO_ALGO_SPLIT
    assert B.wino_workspace_bytes(64, 256, 56, 56, 256, 1, 4, F16) == 392 * 2 * 16 * 36 * 64 * 8
    assert B.wino_workspace_bytes_r(1, 20, 16, 16, 20, 2, 2, 5, F16) == 2**64 - 1   # 3x3 only
    assert B.wino_filter_transform_p(None, FAKE, 4, 4, 4, F16) == B.WINO_ERR_INVALID_ARG
    assert B.wino_filter_transform_p(FAKE, FAKE + 0x10000, 4, 4, 4, 0x40) == B.WINO_ERR_UNSUPPORTED
    assert B.wino_filter_transform_p(FAKE, FAKE + 8, 4, 4, 4, F16) == B.WINO_ERR_INVALID_ARG     # overlap
    assert _conv(flags=F16) == B.WINO_ERR_WORKSPACE
    assert _conv(flags=F16 | B.WINO_ALGO_FUSED) == B.WINO_ERR_UNSUPPORTED


def test_mfma_probe_arguments():
    assert B.wino_probe_mfma_f32(1, None) == B.WINO_ERR_INVALID_ARG
    assert B.wino_probe_mfma_f32(0, FAKE) == B.WINO_ERR_INVALID_ARG
    assert B.wino_probe_mfma_f32(2 ** 21 + 1, FAKE) == B.WINO_ERR_INVALID_ARG
    # 2048 waves x iters x 8 chains x (2 * 16 * 16 * 4) FLOPs
    assert B.wino_probe_mfma_f32_flops(1) == 2048 * 8 * 2048
    assert B.wino_probe_mfma_f32_flops(1000) == 1000 * 2048 * 8 * 2048
    assert B.wino_probe_mfma_f32_flops(0) == 0
    assert B.wino_probe_mfma_f32_flops(2 ** 21 + 1) == 0


def test_channel_slice_sizes_and_rejections():
    F = B.WINO_ALGO_FUSED
    # 64 channels = 16 quads in 3 slices of 6 quads: 3 partial outputs
    assert B.wino_workspace_bytes(1, 64, 20, 20, 16, 1, 4, F | B.WINO_CSLICES(3)) == 3 * 16 * 20 * 20 * 4
    # 20 quads in 8 slices of 3: 7 slices hold channels
    assert B.wino_workspace_bytes(1, 80, 20, 20, 16, 1, 4, F | B.WINO_CSLICES(8)) == 7 * 16 * 20 * 20 * 4
    assert B.wino_workspace_bytes(1, 64, 20, 20, 16, 1, 4, F | B.WINO_CSLICES(1)) == 0
    for flags in (B.WINO_CSLICES(2),                          # only with an explicit WINO_ALGO_FUSED
                  B.WINO_ALGO_STAGED | B.WINO_CSLICES(2), B.WINO_ALGO_SPLIT | B.WINO_CSLICES(2),
                  F | B.WINO_CSLICES(9)):
        assert B.wino_workspace_bytes(1, 64, 20, 20, 16, 1, 4, flags) == 2**64 - 1
    assert B.wino_workspace_bytes(1, 8, 20, 20, 16, 1, 4, F | B.WINO_CSLICES(3)) == 2**64 - 1   # 2 quads
    assert B.wino_workspace_bytes_1d(1, 64, 17, 17, 16, 3, 2, 7, B.WINO_AXIS_W, B.WINO_CSLICES(2)) == 2**64 - 1
    # the planner: VGG-16's 512-channel 28x28 layer at batch 1 gets two slices;
    # the bench layer (224 workgroups) and batch-8 ResNet layers get none
    assert B.wino_workspace_bytes(1, 512, 28, 28, 512, 1, 4, 0) == 2 * 512 * 28 * 28 * 4
    assert B.wino_workspace_bytes(1, 512, 14, 14, 512, 1, 2, 0) == 2 * 512 * 14 * 14 * 4
    assert B.wino_workspace_bytes(1, 64, 112, 112, 64, 1, 4, 0) == 0
    assert B.wino_workspace_bytes(8, 128, 28, 28, 128, 1, 4, 0) == 0
    # missing workspace with explicit slices
    y = FAKE + 0x1000000
    assert B.wino_conv2d(FAKE, FAKE + 0x800000, y, 1, 64, 20, 20, 16, 1, 4, F | B.WINO_CSLICES(2), None, 0) == \
        B.WINO_ERR_WORKSPACE


def test_plan_query():
    F = B.WINO_ALGO_FUSED
    assert B.wino_plan_r(1, 64, 112, 112, 64, 1, 4, 3, 0) == (B.WINO_OK, F, 1)
    assert B.wino_plan_r(1, 512, 28, 28, 512, 1, 4, 3, 0) == (B.WINO_OK, F, 2)
    assert B.wino_plan_r(1, 3, 224, 224, 64, 1, 4, 3, 0) == (B.WINO_OK, B.WINO_ALGO_LOWC, 1)
    assert B.wino_plan_r(64, 256, 56, 56, 256, 1, 4, 3, 0) == (B.WINO_OK, B.WINO_ALGO_SPLIT, 1)
    assert B.wino_plan_r(1, 64, 20, 20, 16, 1, 4, 3, B.WINO_ALGO_STAGED) == (B.WINO_OK, B.WINO_ALGO_STAGED, 1)
    assert B.wino_plan_r(1, 80, 20, 20, 16, 1, 4, 3, F | B.WINO_CSLICES(8)) == (B.WINO_OK, F, 7)
    assert B.wino_plan_r(32, 48, 35, 35, 64, 2, 2, 5, 0) == (B.WINO_OK, F, 1)
    assert B.wino_plan_r(1, 64, 20, 20, 16, 1, 3, 3, 0)[0] == B.WINO_ERR_UNSUPPORTED
    assert B.wino_plan_r(0, 64, 20, 20, 16, 1, 4, 3, 0)[0] == B.WINO_ERR_INVALID_ARG
    assert B.lib().wino_plan_r(1, 64, 20, 20, 16, 1, 4, 3, 0, None, None) == B.WINO_ERR_INVALID_ARG


def test_input_offsets_stay_below_2_32():
    """The fused and split kernels read channels past C (or past a slice) as
    zeros because their 32-bit offsets land past the buffer; layers where the
    largest such offset would reach 2^32 (and wrap back inside the image) are
    rejected, or AUTO moves to an algorithm whose offsets fit."""
    F, S, A = B.WINO_ALGO_FUSED, B.WINO_ALGO_SPLIT, B.WINO_ALGO_AUTO
    # fused, m = 4 (16 channels a step): 2^30 + (1 + 3) * 16 * H*W*4 < 2^32  <=>  H*W < 3 * 2^22
    assert B.wino_workspace_bytes(1, 16, 3071, 4096, 16, 1, 4, F) == 0
    assert B.wino_workspace_bytes(1, 16, 3072, 4096, 16, 1, 4, F) == 2**64 - 1
    # fused, m = 2 (32 channels a step): H*W < 3 * 2^21
    assert B.wino_workspace_bytes(1, 16, 2047, 3072, 16, 1, 2, F) == 0
    assert B.wino_workspace_bytes(1, 16, 2048, 3072, 16, 1, 2, F) == 2**64 - 1
    # split (16 channels per input-transform workgroup): 2^30 + 16 * H*W*4 < 2^32
    assert B.wino_workspace_bytes(1, 5, 6143, 8192, 16, 1, 4, S) > 0
    assert B.wino_workspace_bytes(1, 5, 6144, 8192, 16, 1, 4, S) == 2**64 - 1
    assert B.wino_plan_r(1, 3, 9220, 9220, 64, 1, 4, 3, S)[0] == B.WINO_ERR_UNSUPPORTED
    # N=1, C=5, 6400 x 6400, m = 2: the fused kernel's offsets would wrap; AUTO
    # takes split, whose offsets fit, and needs its workspace (no fused fallback)
    assert B.wino_plan_r(1, 5, 6400, 6400, 64, 1, 2, 3, F)[0] == B.WINO_ERR_UNSUPPORTED
    assert B.wino_plan_r(1, 5, 6400, 6400, 64, 1, 2, 3, A) == (B.WINO_OK, S, 1)
    y = FAKE + (1 << 34)
    assert B.wino_conv2d(FAKE, FAKE + (1 << 33), y, 1, 5, 6400, 6400, 64, 1, 2, A, None, 0) == \
        B.WINO_ERR_WORKSPACE
    # 5x5 layers have no split path: AUTO takes the three stages where their
    # offsets fit (two images per block: 2 * 5 * 4000^2 * 4 < 2^30), else rejects
    assert B.wino_plan_r(1, 5, 4000, 4000, 64, 2, 2, 5, F)[0] == B.WINO_ERR_UNSUPPORTED
    assert B.wino_plan_r(1, 5, 4000, 4000, 64, 2, 2, 5, A) == (B.WINO_OK, B.WINO_ALGO_STAGED, 1)
    assert B.wino_plan_r(1, 5, 6400, 6400, 64, 2, 2, 5, A)[0] == B.WINO_ERR_UNSUPPORTED


def test_noalloc_entry_point_rejects():
    """The allocation-free variant validates like wino_conv2d and rejects
    explicit plans whose workspace exceeds its static scratch, before any HIP
    call (CPU only)."""
    y = FAKE + (1 << 33)
    cap = B.WINO_NOALLOC_SCRATCH_BYTES
    assert "WINO_NOALLOC_SCRATCH_BYTES ((size_t)64 << 20)" in open(B.HEADER).read()
    # N=64, C=K=256, 56x56, m=4: V and M of the staged path, or the split path's
    # tile-blocked V, are far past the scratch
    for algo in (B.WINO_ALGO_STAGED, B.WINO_ALGO_SPLIT):
        assert B.wino_workspace_bytes(64, 256, 56, 56, 256, 1, 4, algo) > cap
        assert B.wino_conv2d_noalloc(FAKE, FAKE + (1 << 32), y, 64, 256, 56, 56, 256, 1, 4, algo) == \
            B.WINO_ERR_WORKSPACE
    # invalid arguments as for wino_conv2d
    assert B.wino_conv2d_noalloc(None, FAKE, y, 1, 4, 8, 8, 4, 1, 4) == B.WINO_ERR_INVALID_ARG
    assert B.wino_conv2d_noalloc(FAKE, FAKE + 0x1000, y, 0, 4, 8, 8, 4, 1, 4) == B.WINO_ERR_INVALID_ARG
    assert B.wino_conv2d_noalloc(FAKE, FAKE + 0x1000, y, 1, 4, 8, 8, 4, 1, 3) == B.WINO_ERR_UNSUPPORTED
    assert B.wino_conv2d_noalloc(FAKE, FAKE + 0x1000, y, 1, 4, 8, 8, 4, 1, 4, 0x500) == B.WINO_ERR_UNSUPPORTED
    # x aliasing y
    assert B.wino_conv2d_noalloc(FAKE, FAKE + (1 << 32), FAKE, 1, 4, 8, 8, 4, 1, 4) == B.WINO_ERR_INVALID_ARG
