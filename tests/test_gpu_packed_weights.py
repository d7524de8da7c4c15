"""Fragment packing straight from the caller's weights (the register-weight
halo tiles of backward-data and of both passes of small groups) against the
fp64 oracle: every filter/channel index split of a super-group, several channel
slices, a last block that is not full, both layouts, and an inf or NaN weight,
whose flag the packing raises for the border fix-up."""
import numpy as np
import pytest

import gpu_util as U
import oracle.oracle as orc
from paper_2102_06725_amd import inputs as I
from paper_2102_06725_amd import nnconv as nc

pytestmark = pytest.mark.gpu

SHAPES = [
    # name, n, c, h, w, k, pad, dil, groups, forced tile
    ("c64k64", 2, 64, 9, 10, 64, 1, 1, 1, nc.NNCONV_TILE_HALO_R256x128),
    ("c192k128", 2, 192, 7, 9, 128, 1, 1, 1, nc.NNCONV_TILE_HALO_R256x128),
    ("c256k64", 1, 256, 12, 7, 64, 1, 1, 1, nc.NNCONV_TILE_HALO_R128x256),
    ("c64k192_dil2", 1, 64, 11, 13, 192, 2, 2, 1, nc.NNCONV_TILE_HALO_R256x128),
    ("sg2", 32, 128, 28, 28, 128, 1, 1, 64, None),
    ("sg4", 32, 192, 28, 28, 192, 1, 1, 48, None),
    ("sg8_dil2", 32, 128, 28, 28, 128, 2, 2, 16, None),
    ("sg16", 32, 128, 28, 28, 128, 1, 1, 8, None),
    ("sg32", 32, 128, 28, 28, 128, 1, 1, 4, None),
]


def _case(s, dtype, layout):
    name, n, c, h, w, k, pad, dil, groups, tile = s
    return U.Case(I.Layer(name, n, c, h, w, k, 3, 3, 1, pad, dil, groups), layout=layout, dtype=dtype,
                  x_kind="normal", cfg=96, layer_id=SHAPES.index(s), alpha=1.5)


@pytest.mark.parametrize("layout", ["nhwc", "nchw"])
@pytest.mark.parametrize("dtype", [I.F16, I.BF16])
@pytest.mark.parametrize("s", SHAPES, ids=[s[0] for s in SHAPES])
def test_packed_weights_parity(nnlib, oracle_lib, s, dtype, layout):
    passes = ("fwd", "dgrad") if s[-1] is None else ("dgrad",)
    U.full_parity(_case(s, dtype, layout), passes=passes, tile=s[-1])


@pytest.mark.parametrize("bits", [0x7C00, 0xFC00, 0x7E01], ids=["inf", "-inf", "nan"])
@pytest.mark.parametrize("where", [0, 0.5, 1], ids=["first", "middle", "last"])
@pytest.mark.parametrize("s", SHAPES[:4], ids=[s[0] for s in SHAPES[:4]])
def test_packed_weights_nonfinite(nnlib, oracle_lib, s, where, bits):
    """The non-finite dx are the oracle's and no others: the border pixels
    that the definition gives no such weight stay finite."""
    case = _case(s, I.F16, "nhwc")
    t = case.tensors()
    w = t["w"].reshape(-1)
    w[int(where * (w.size - 1))] = bits
    g = U.to_nchw(case, "dx", U.run_gpu(case, t, ("dgrad",), tile=s[-1])["dx"])
    _, wf, dy = U.nchw_f64(case, t)
    with np.errstate(invalid="ignore", over="ignore"):
        ref = U.oracle_conv(case).dgrad(dy, wf, alpha=case.alpha)
    fin = np.isfinite(ref)
    assert np.array_equal(np.isfinite(g), fin) and not fin.all()
    assert orc.rel_err(g[fin], ref[fin]) <= U.TOL[case.dtype]
