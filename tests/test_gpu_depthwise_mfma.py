"""The matrix-core depthwise kernels (stride 1) against the fp64 oracle: each of
the four forward tiles at ragged image sizes and channel counts, every filter
size, padding 0 to R-1, and inf / NaN inputs, which must stay in their own
channel; and layers on the vector kernel's side of the rule.  Cases that name a
kernel ask which one the call launches."""
import numpy as np
import pytest

import gpu_util as U
import oracle.oracle as orc
from paper_2102_06725_amd import inputs as I

pytestmark = pytest.mark.gpu

# n, c, h, w, r, pad: ragged layers on either side of the rule
SHAPES = [
    ("w7_5x5", 86, 136, 7, 7, 5, 2),
    ("w8_7x7", 128, 72, 9, 8, 7, 3),
    ("w14_3x3", 171, 136, 14, 14, 3, 1),
    ("w15_5x5", 43, 136, 17, 15, 5, 0),     # padding 0: 13x11 outputs
    ("w16_7x7", 64, 72, 15, 10, 7, 6),      # padding R-1: 21x16 outputs
    ("w28_5x5", 17, 240, 28, 28, 5, 2),
    ("w33_3x3", 19, 72, 29, 33, 3, 1),
    ("w17_7x7", 22, 72, 27, 17, 7, 3),
    ("w40_3x3", 65, 24, 56, 33, 3, 1),
]
BOTH, B16 = (I.F16, I.BF16), (I.BF16,)
# The tiles by their template arguments: 16-channel groups, blocks of pixels,
# columns of a block, output rows of a strip (7x7: half as many, but tile 0).
TILES = [(4, 1, 8, 4), (4, 1, 16, 14), (1, 4, 8, 14), (2, 2, 16, 14)]
TILE_SHAPES = [
    # name, n, c, h, w, r, pad, tile of forward, of backward-data (None: vector kernel), types
    ("w7_5x5", 128, 136, 7, 7, 5, 2, 0, 0, B16),         # 3 blocks of 64 channels, 8 past the end
    ("w7_5x5_c960", 128, 960, 7, 7, 5, 2, 0, 0, BOTH),
    ("w8_7x7", 128, 72, 9, 8, 7, 3, 0, 0, B16),          # two row tiles
    ("w14_3x3", 171, 136, 14, 14, 3, 1, 1, 1, B16),
    ("w13x15_3x3", 200, 264, 13, 15, 3, 1, 1, 1, B16),
    ("w15_5x5", 120, 136, 17, 15, 5, 2, 1, 1, BOTH),     # 3 rows in the second row tile
    ("w15_5x5_p0", 160, 136, 17, 15, 5, 0, 1, 1, B16),   # padding 0: 13x11 outputs
    ("w10_7x7", 150, 136, 14, 10, 7, 3, 1, 1, B16),
    ("w16_7x7", 64, 72, 15, 10, 7, 6, 1, None, B16),     # padding R-1: 21x16 outputs
    ("w28_5x5", 40, 240, 28, 28, 5, 2, 2, 2, BOTH),      # 16 channels x 28 rows
    ("w33_5x5_p4", 60, 72, 27, 33, 5, 4, 2, 2, B16),     # 31x37 outputs
    ("w17_7x7", 22, 72, 27, 17, 7, 3, 2, 2, BOTH),
    ("w29_5x5", 20, 240, 29, 29, 5, 2, 3, 3, B16),       # 32 channels x 14 rows, ragged
    ("w40_5x5", 80, 96, 40, 40, 5, 2, 3, 3, BOTH),
    ("w28x21_7x7", 60, 128, 21, 28, 7, 3, 3, 3, BOTH),
]
BY_NAME = {s[0]: s for s in TILE_SHAPES}
# the LDS-tiled vector kernel is the faster one: few workgroups, badly filled
# tiles, wide or narrow 3x3 images, 3x3 in fp16
VECTOR = [
    ("few_5x5", 86, 136, 7, 7, 5, 2, I.F16),
    ("few_w15_5x5", 43, 136, 17, 15, 5, 0, I.BF16),
    ("w33_3x3", 19, 72, 29, 33, 3, 1, I.BF16),
    ("w40_3x3", 65, 24, 56, 33, 3, 1, I.BF16),
    ("w8_3x3", 200, 264, 9, 8, 3, 1, I.BF16),
    ("w14_3x3_f16", 171, 136, 14, 14, 3, 1, I.F16),
    ("w15_7x7_f16", 47, 464, 15, 15, 7, 3, I.F16),
]


def _assert_tiles(case, fwd, dgrad, passes=("fwd", "dgrad")):
    r = case.layer.r
    for p, tile in (("fwd", fwd), ("dgrad", dgrad)):
        if p not in passes:
            continue
        if tile is None:
            U.assert_runs(case, p, "dwt_fwd_kernel", r)
        else:
            a = list(TILES[tile])
            if r == 7 and tile:
                a[3] //= 2
            U.assert_runs(case, p, "dwm_fwd_kernel", r, *a, p == "dgrad")


def _case(s, layout, dtype):
    name, n, c, h, w, r, pad = s[:7]
    tiled = len(s) > 7
    case = U.Case(I.Layer(name, n, c, h, w, c, r, r, 1, pad, groups=c), layout=layout, dtype=dtype, x_kind="normal",
                  cfg=100, layer_id=20 + TILE_SHAPES.index(s) if tiled else SHAPES.index(s), alpha=0.5)
    if tiled:
        _assert_tiles(case, s[7], s[8])
    return case


@pytest.mark.parametrize("dtype", [I.F16, I.BF16])
@pytest.mark.parametrize("s", SHAPES, ids=[s[0] for s in SHAPES])
def test_depthwise_mfma_parity(nnlib, oracle_lib, s, dtype):
    U.full_parity(_case(s, "nhwc", dtype), passes=("fwd", "dgrad"))


@pytest.mark.parametrize("s,dtype", [(s, t) for s in TILE_SHAPES for t in s[9]],
                         ids=[f"{s[0]}-{t}" for s in TILE_SHAPES for t in s[9]])
def test_depthwise_mfma_tiles(nnlib, oracle_lib, s, dtype):
    U.full_parity(_case(s, "nhwc", dtype), passes=("fwd", "dgrad"))


@pytest.mark.parametrize("s", VECTOR, ids=[s[0] for s in VECTOR])
def test_depthwise_vector_side_of_the_rule(nnlib, oracle_lib, s):
    name, n, c, h, w, r, pad, dtype = s
    case = U.Case(I.Layer(name, n, c, h, w, c, r, r, 1, pad, groups=c), dtype=dtype, x_kind="normal", cfg=100,
                  layer_id=50 + VECTOR.index(s), alpha=0.5)
    _assert_tiles(case, None, None, passes=("fwd",))
    U.full_parity(case, passes=("fwd", "dgrad"))


@pytest.mark.parametrize("s", [SHAPES[5], BY_NAME["w28_5x5"], BY_NAME["w29_5x5"], BY_NAME["w10_7x7"]],
                         ids=["few", "w28_5x5", "w29_5x5", "w10_7x7"])
def test_depthwise_mfma_nchw(nnlib, oracle_lib, s):
    U.full_parity(_case(s, "nchw", I.BF16), passes=("fwd", "dgrad"))


NON_FINITE = [SHAPES[0], SHAPES[2], SHAPES[5], SHAPES[6]] + [
    BY_NAME[n] for n in ("w7_5x5", "w8_7x7", "w14_3x3", "w15_5x5", "w10_7x7", "w28_5x5", "w17_7x7", "w29_5x5",
                         "w28x21_7x7")]


@pytest.mark.parametrize("kind", ["inf", "-inf", "nan"])
@pytest.mark.parametrize("s", NON_FINITE, ids=lambda s: s[0] + ("-tile" if len(s) > 7 else ""))
def test_depthwise_mfma_non_finite(nnlib, oracle_lib, s, kind):
    dtype = s[9][-1] if len(s) > 7 else I.F16
    bits = {I.F16: {"inf": 0x7C00, "-inf": 0xFC00, "nan": 0x7E01},
            I.BF16: {"inf": 0x7F80, "-inf": 0xFF80, "nan": 0x7FC1}}[dtype][kind]
    case = _case(s, "nhwc", dtype)
    t = case.tensors()
    for k in ("x", "dy"):
        flat = t[k].reshape(-1)
        flat[flat.size // 2 + 5] = bits
        flat[-3] = bits
    t["w"].reshape(-1)[7] = bits  # channel 0
    got = U.run_gpu(case, t, ("fwd", "dgrad"))
    x, w, dy = U.nchw_f64(case, t)
    cv = U.oracle_conv(case)
    with np.errstate(invalid="ignore"):
        refs = {"y": cv.fwd(x, w, alpha=case.alpha), "dx": cv.dgrad(dy, w, alpha=case.alpha)}
    for k, ref in refs.items():
        g = U.to_nchw(case, k, got[k])
        assert np.array_equal(np.isnan(g), np.isnan(ref)) and np.array_equal(np.isinf(g), np.isinf(ref)), k
        ok = np.isfinite(ref)
        assert orc.rel_err(g[ok], ref[ok]) <= U.TOL[dtype]


def test_depthwise_mfma_largest_finite_values(nnlib, oracle_lib):
    """The largest finite value does not count as inf."""
    case = _case(BY_NAME["w14_3x3"], "nhwc", I.BF16)
    t = case.tensors()
    t["x"].reshape(-1)[::977] = 0x7F7F
    t["w"].reshape(-1)[:] = I.to_bits(I.from_bits(t["w"].reshape(-1), I.BF16) * 1e-3, I.BF16)
    got = U.run_gpu(case, t, ("fwd",))
    x, w, _ = U.nchw_f64(case, t)
    ref = U.oracle_conv(case).fwd(x, w, alpha=case.alpha)
    assert orc.rel_err(U.to_nchw(case, "y", got["y"]), ref) <= U.TOL[I.BF16]


# backward-weight: at least 96 workgroups of (32 channels, split)
WG_SHAPES = [
    # name, n, c, h, w, r, pad, columns of a block (None: vector kernel)
    ("w8_3x3", 40, 136, 8, 8, 3, 1, 8),        # 8x8 blocks, 5 channel blocks, 8 channels past the end
    ("w5_5x5", 30, 264, 9, 5, 5, 2, 8),        # ragged columns, two row blocks
    ("w14_5x5", 40, 200, 14, 14, 5, 2, 16),    # 16x14 blocks
    ("w17_3x3", 24, 136, 15, 17, 3, 0, None),  # the vector kernel; padding 0: 13x15 outputs
    ("w15_3x3_p0", 120, 136, 15, 13, 3, 0, 16),  # padding 0: 13x11 outputs
    ("w33_5x5", 20, 72, 17, 33, 5, 4, 16),     # padding R-1: 21x37 outputs, ragged both ways
    ("w15_3x3", 90, 136, 15, 15, 3, 1, 16),    # one row past a block
    ("w7_3x3", 100, 136, 7, 7, 3, 1, 8),       # ragged 8x8 blocks
    ("round_5x5", 57, 1152, 14, 14, 5, 2, 16),  # a little over two workgroups per CU: fewer splits
]
WG_BY_NAME = {s[0]: s for s in WG_SHAPES}


def _wg_case(s, dtype=I.F16, layer_id=None, **kw):
    name, n, c, h, w, r, pad, cols = s
    case = U.Case(I.Layer(name, n, c, h, w, c, r, r, 1, pad, groups=c), dtype=dtype, x_kind="normal", cfg=103,
                  layer_id=WG_SHAPES.index(s) if layer_id is None else layer_id, **kw)
    if cols is None:
        U.assert_runs(case, "wgrad", "dwt_wgrad_kernel", r)
    else:
        U.assert_runs(case, "wgrad", "dwm_wgrad_kernel", r, cols)
    return case


@pytest.mark.parametrize("dtype", [I.F16, I.BF16])
@pytest.mark.parametrize("s", WG_SHAPES, ids=[s[0] for s in WG_SHAPES])
def test_depthwise_mfma_backward_weight(nnlib, oracle_lib, s, dtype):
    case = _wg_case(s, dtype, loss_scale=256.0)
    U.full_parity(case, passes=("wgrad",))
    t = case.tensors()
    a, b = (U.run_gpu(case, t, ("wgrad",)) for _ in range(2))
    assert np.array_equal(a["dw_bits"], b["dw_bits"])


def test_depthwise_mfma_backward_weight_non_finite(nnlib, oracle_lib):
    """An inf in one channel of dy leaves the other channels' gradients alone."""
    case = _wg_case(WG_BY_NAME["w14_5x5"])
    c, r = case.layer.c, case.layer.r
    t = case.tensors()
    t["dy"].reshape(-1, c)[777, 33] = 0x7C00
    flag = U.torch().zeros(1, dtype=U.torch().int32, device="cuda")
    g = U.run_gpu(case, t, ("wgrad",), flag=flag)["dw"].reshape(c, r * r)
    x, w_, dy = U.nchw_f64(case, t)
    with np.errstate(invalid="ignore"):
        ref = U.oracle_conv(case).wgrad(x, dy).reshape(c, r * r)
    assert np.array_equal(np.isfinite(g), np.isfinite(ref)) and int(flag.item()) == 1
    ok = np.isfinite(ref)
    assert orc.rel_err(g[ok], ref[ok]) <= U.TOL[I.F16]


@pytest.mark.parametrize("at", ["corner", "last_row", "last_cols"])
@pytest.mark.parametrize("s", [("w24_3x3", 24, 136, 14, 24, 3, 1, None), ("w24_5x5", 24, 136, 14, 24, 5, 2, 16),
                               WG_BY_NAME["w15_3x3"], WG_BY_NAME["w7_3x3"], WG_BY_NAME["w5_5x5"],
                               WG_BY_NAME["w33_5x5"]], ids=lambda s: s[0])
def test_depthwise_mfma_backward_weight_non_finite_input(nnlib, oracle_lib, s, at):
    """An inf in x counts for the taps that read it only: the blocks reach past
    the outputs, where dy has no pixels."""
    case = _wg_case(s, layer_id=s[5])
    L = case.layer
    n, c, h, w, r = L.n, L.c, L.h, L.w, L.r
    pixel = {"corner": (h - 1, w - 1), "last_row": (h - 1, w // 2), "last_cols": (h // 2, w - 2)}[at]
    t = case.tensors()
    t["x"].reshape(n, h, w, c)[n // 2, pixel[0], pixel[1], 35] = 0x7C00
    g = U.run_gpu(case, t, ("wgrad",))["dw"].reshape(c, r * r)
    x, _, dy = U.nchw_f64(case, t)
    with np.errstate(invalid="ignore"):
        ref = U.oracle_conv(case).wgrad(x, dy).reshape(c, r * r)
    assert not np.isfinite(ref[35]).all() and np.isfinite(np.delete(ref, 35, 0)).all()
    assert np.array_equal(np.isfinite(g), np.isfinite(ref))
    ok = np.isfinite(ref)
    assert orc.rel_err(g[ok], ref[ok]) <= U.TOL[I.F16]


def _time(fn, reps=10):
    t = U.torch()
    fn()
    best = float("inf")
    for _ in range(3):
        a, b = (t.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(reps):
            fn()
        b.record()
        t.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / reps)
    return best


def test_depthwise_mfma_overflow_step(nnlib):
    """An overflow of the loss scale is an ordinary event: with every dy inf the
    backward passes take less than three times as long as with finite ones (1.3
    and 1.6 times; without a look at x first the sums of backward-weight, taken
    again term by term, took 90 times as long)."""
    from paper_2102_06725_amd import nnconv as nc
    t = U.torch()
    n, c, h, r = 64, 240, 28, 5
    case = U.Case(I.Layer("ovf", n, c, h, h, c, r, r, 1, r // 2, groups=c))
    _assert_tiles(case, 2, 2)
    U.assert_runs(case, "wgrad", "dwm_wgrad_kernel", r)
    conv = nc.Conv2d(n, c, h, h, c, r, r, stride=1, pad=r // 2, groups=c)
    x, dy, dx = (t.randn(n, h, h, c, device="cuda").half() for _ in range(3))
    w = t.randn(c, r, r, 1, device="cuda").half()
    dw = t.empty(c, r, r, 1, device="cuda")
    flag = t.zeros(1, dtype=t.int32, device="cuda")
    for fn in (lambda: conv.dgrad(dy, w, dx), lambda: conv.wgrad(x, dy, dw, nc.NNCONV_F32, 1.0, 0, flag)):
        keep = dy.clone()
        finite = _time(fn)
        dy.fill_(float("inf"))
        over = _time(fn)
        dy.copy_(keep)
        assert over < 3 * finite, (over, finite)
    assert int(flag.item()) == 1


@pytest.mark.parametrize("where", ["dy", "x", "both"])
@pytest.mark.parametrize("s", [WG_SHAPES[0], WG_SHAPES[1], WG_SHAPES[2]], ids=lambda s: s[0])
def test_depthwise_mfma_backward_weight_many_non_finite(nnlib, oracle_lib, s, where):
    """Infs in a third of the channels of dy, of x, or of both: the non-finite
    sums are the oracle's and no others, and the rest keeps its accuracy."""
    name, n, c, h, w, r, pad, cols = s
    case = _wg_case(s, layer_id=7)
    t = case.tensors()
    rng = np.random.default_rng(11)
    for k in ("x", "dy"):
        if where in (k, "both"):
            a = t[k].reshape(-1, c)
            at = rng.integers(0, a.shape[0], c // 3)
            a[at, np.arange(c // 3) * 3] = 0x7C00
            t[k].reshape(n, -1, w if k == "x" else case.layer.q, c)[-1, -1, :, 1] = 0xFC00  # a whole last row
    g = U.run_gpu(case, t, ("wgrad",))["dw"].reshape(c, r * r)
    x, _, dy = U.nchw_f64(case, t)
    with np.errstate(invalid="ignore"):
        ref = U.oracle_conv(case).wgrad(x, dy).reshape(c, r * r)
    assert np.array_equal(np.isnan(g), np.isnan(ref)) and np.array_equal(np.isinf(g), np.isinf(ref))
    ok = np.isfinite(ref)
    assert orc.rel_err(g[ok], ref[ok]) <= U.TOL[I.F16]
