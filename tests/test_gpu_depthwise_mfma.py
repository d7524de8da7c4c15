"""The matrix-core depthwise kernel (stride 1, from one or two workgroups per
CU up) against the fp64 oracle: each of its four tiles at ragged image sizes
and channel counts, every filter size, padding 0 to R-1, and inf / NaN inputs,
which must stay in their own channel."""
import numpy as np
import pytest

import gpu_util as U
import oracle.oracle as orc
from paper_2102_06725_amd import inputs as I

pytestmark = pytest.mark.gpu

# n, c, h, w, r, pad: workgroups = n * channel blocks * row tiles * column tiles,
# at least 512 for 3x3 and 256 for 5x5 / 7x7
SHAPES = [
    ("w7_5x5", 86, 136, 7, 7, 5, 2),        # 8-wide tile, 3 blocks of 64 channels, 8 past the end
    ("w8_7x7", 128, 72, 9, 8, 7, 3),        # two row tiles
    ("w14_3x3", 171, 136, 14, 14, 3, 1),    # 16-wide tile
    ("w15_5x5", 43, 136, 17, 15, 5, 0),     # padding 0: 13x11 outputs
    ("w16_7x7", 64, 72, 15, 10, 7, 6),      # padding R-1: 21x16 outputs
    ("w28_5x5", 17, 240, 28, 28, 5, 2),     # 16 channels x 28 rows
    ("w33_3x3", 19, 72, 29, 33, 3, 1),      # 32 channels x 14 rows, ragged second tile column
    ("w17_7x7", 22, 72, 27, 17, 7, 3),
    ("w40_3x3", 65, 24, 56, 33, 3, 1),      # 16-channel tile, 24 channels
]


def _case(s, layout, dtype):
    name, n, c, h, w, r, pad = s
    return U.Case(I.Layer(name, n, c, h, w, c, r, r, 1, pad, groups=c), layout=layout, dtype=dtype,
                  x_kind="normal", cfg=100, layer_id=SHAPES.index(s), alpha=0.5)


@pytest.mark.parametrize("dtype", [I.F16, I.BF16])
@pytest.mark.parametrize("s", SHAPES, ids=[s[0] for s in SHAPES])
def test_depthwise_mfma_parity(nnlib, oracle_lib, s, dtype):
    U.full_parity(_case(s, "nhwc", dtype), passes=("fwd", "dgrad"))


def test_depthwise_mfma_nchw(nnlib, oracle_lib):
    U.full_parity(_case(SHAPES[5], "nchw", I.BF16), passes=("fwd", "dgrad"))


@pytest.mark.parametrize("bits", [0x7C00, 0xFC00, 0x7E01], ids=["inf", "-inf", "nan"])
@pytest.mark.parametrize("s", [SHAPES[0], SHAPES[2], SHAPES[5], SHAPES[6]], ids=lambda s: s[0])
def test_depthwise_mfma_non_finite(nnlib, oracle_lib, s, bits):
    case = _case(s, "nhwc", I.F16)
    t = case.tensors()
    for k in ("x", "dy"):
        flat = t[k].reshape(-1)
        flat[flat.size // 2 + 5] = bits
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
        assert orc.rel_err(g[ok], ref[ok]) <= U.TOL[I.F16]


def test_depthwise_mfma_largest_finite_values(nnlib, oracle_lib):
    """The largest finite value does not count as inf."""
    case = _case(SHAPES[2], "nhwc", I.BF16)
    t = case.tensors()
    t["x"].reshape(-1)[::977] = 0x7F7F
    t["w"].reshape(-1)[:] = I.to_bits(I.from_bits(t["w"].reshape(-1), I.BF16) * 1e-3, I.BF16)
    got = U.run_gpu(case, t, ("fwd",))
    x, w, _ = U.nchw_f64(case, t)
    ref = U.oracle_conv(case).fwd(x, w, alpha=case.alpha)
    assert orc.rel_err(U.to_nchw(case, "y", got["y"]), ref) <= U.TOL[I.BF16]


# backward-weight: at least 96 workgroups of (32 channels, split)
WG_SHAPES = [
    ("w8_3x3", 40, 136, 8, 8, 3, 1),       # 8x8 blocks, 5 channel blocks, 8 channels past the end
    ("w5_5x5", 30, 264, 9, 5, 5, 2),       # ragged columns, two row blocks
    ("w14_5x5", 40, 200, 14, 14, 5, 2),    # 16x14 blocks
    ("w17_3x3", 24, 136, 15, 17, 3, 0),    # padding 0: 13x15 outputs
    ("w33_5x5", 20, 72, 17, 33, 5, 4),     # padding R-1: 21x37 outputs, ragged both ways
]


@pytest.mark.parametrize("dtype", [I.F16, I.BF16])
@pytest.mark.parametrize("s", WG_SHAPES, ids=[s[0] for s in WG_SHAPES])
def test_depthwise_mfma_backward_weight(nnlib, oracle_lib, s, dtype):
    name, n, c, h, w, r, pad = s
    L = I.Layer(name, n, c, h, w, c, r, r, 1, pad, groups=c)
    case = U.Case(L, dtype=dtype, loss_scale=256.0, x_kind="normal", cfg=103, layer_id=WG_SHAPES.index(s))
    U.full_parity(case, passes=("wgrad",))
    t = case.tensors()
    a, b = (U.run_gpu(case, t, ("wgrad",)) for _ in range(2))
    assert np.array_equal(a["dw_bits"], b["dw_bits"])


def test_depthwise_mfma_backward_weight_non_finite(nnlib, oracle_lib):
    """An inf in one channel of dy leaves the other channels' gradients alone."""
    name, n, c, h, w, r, pad = WG_SHAPES[2]
    case = U.Case(I.Layer(name, n, c, h, w, c, r, r, 1, pad, groups=c), x_kind="normal", cfg=103, layer_id=2)
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


@pytest.mark.parametrize("pixel", [(13, 23), (12, 15), (8, 22)], ids=["corner", "last_row", "last_cols"])
@pytest.mark.parametrize("r", [3, 5])
def test_depthwise_mfma_backward_weight_non_finite_input(nnlib, oracle_lib, r, pixel):
    """An inf in x counts for the taps that read it only: blocks of 14 rows x 16
    columns reach past the 14x24 outputs, where dy has no pixels."""
    n, c, h, w = 24, 136, 14, 24
    case = U.Case(I.Layer("w24", n, c, h, w, c, r, r, 1, r // 2, groups=c), x_kind="normal", cfg=103, layer_id=r)
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
    U.assert_runs(case, "dgrad", "dwm_fwd_kernel", r)
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
    name, n, c, h, w, r, pad = s
    case = U.Case(I.Layer(name, n, c, h, w, c, r, r, 1, pad, groups=c), x_kind="normal", cfg=103, layer_id=7)
    U.assert_runs(case, "wgrad", "dwm_wgrad_kernel", r)
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
