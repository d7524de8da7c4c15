"""The split-reduction tiles (the waves of a workgroup share one small tile),
which forward and backward-data take where the grid is small, against the fp64
oracle: one row or column below, at and above the 32- and 64-wide tiles, fewer
reduction steps than waves, reductions whose 32-element steps mix taps
(channels not a multiple of 32), stride phases of different sizes and without
taps (up to 16 in one launch, beyond that one each), groups, and the
block-diagonal weights of small groups.  The shapes of TILES64 are large enough
for the 64x64 tiles.  Backward-data of the smallest shapes has a kernel of its
own (one launch): those of LONG have reductions too long for it.  Every test asks
which kernel the call launches."""
import numpy as np
import pytest

import gpu_util as U
from paper_2102_06725_amd import inputs as I
from paper_2102_06725_amd import nnconv as nc

pytestmark = pytest.mark.gpu

SHAPES = [
    # name, n, c, h, w, k, r, stride, pad, dil, groups
    ("m31", 1, 64, 1, 31, 32, 1, 1, 0, 1, 1),
    ("m33n40", 1, 64, 3, 11, 40, 1, 1, 0, 1, 1),
    ("m65n72", 1, 128, 5, 13, 72, 3, 1, 1, 1, 1),
    ("two_steps", 2, 64, 4, 4, 64, 1, 1, 0, 1, 1),       # fewer than the waves
    ("one_pixel_long", 1, 1024, 1, 1, 64, 1, 1, 0, 1, 1),
    ("c8", 2, 8, 9, 7, 8, 3, 1, 1, 1, 1),                # 9 chunks of 8 in 3 steps
    ("c16k24", 2, 16, 10, 6, 24, 3, 2, 1, 1, 1),
    ("c40k56", 1, 40, 8, 9, 56, 3, 1, 1, 1, 1),
    ("c96k32_5x5", 1, 96, 7, 7, 32, 5, 1, 2, 1, 1),
    ("dil2", 1, 64, 12, 9, 64, 3, 1, 2, 2, 1),
    ("s2_phases", 1, 64, 13, 11, 128, 3, 2, 1, 1, 1),
    ("s2_tapless", 3, 64, 7, 6, 64, 1, 2, 0, 1, 1),
    ("s3_c24", 1, 24, 10, 11, 16, 3, 3, 1, 1, 1),        # 9 phases: one launch each
    ("groups64", 1, 192, 6, 7, 192, 3, 1, 1, 1, 3),
    ("groups24", 1, 48, 6, 7, 48, 3, 1, 1, 1, 2),
    ("diag4", 1, 128, 9, 9, 128, 3, 1, 1, 1, 32),
    ("diag32_s2", 2, 128, 7, 8, 128, 3, 2, 1, 1, 4),
    ("tiles64_4w", 8, 512, 28, 27, 120, 1, 1, 0, 1, 1),
    ("tiles64_8w", 8, 128, 27, 29, 120, 3, 1, 1, 1, 1),
    # long reductions of backward-data
    ("m33n40_k512", 1, 40, 3, 11, 512, 3, 1, 1, 1, 1),
    ("c8_k520", 2, 8, 9, 7, 520, 3, 1, 1, 1, 1),          # steps across taps
    ("c40_k328", 1, 40, 8, 9, 328, 3, 1, 1, 1, 1),
    ("c72_k1032", 2, 72, 5, 5, 1032, 1, 1, 0, 1, 1),
    ("dil2_k512", 1, 64, 12, 9, 512, 3, 1, 2, 2, 1),
    ("s2_tapless_k1024", 3, 64, 7, 6, 1024, 1, 2, 0, 1, 1),
    ("s2_k264", 1, 64, 13, 11, 264, 3, 2, 1, 1, 1),       # four phases, steps across taps
    ("s3_k264", 1, 24, 10, 11, 264, 3, 3, 1, 1, 1),       # nine
    ("s4_k264", 1, 64, 13, 12, 264, 3, 4, 1, 1, 1),       # sixteen, seven of them without taps
    ("s5_k72", 1, 64, 11, 12, 72, 5, 5, 2, 1, 1),         # 25: one launch each
]
# backward-data of these runs in one launch on the kernel for very small layers
TINY_DGRAD = {"m31", "m33n40", "m65n72", "two_steps", "one_pixel_long", "c8", "c16k24", "c40k56", "dil2", "s2_tapless",
              "s3_c24"}
MIXED_DGRAD = {"tiles64_4w"}  # the mixed-tap tiles are the faster ones
TILES64 = {("tiles64_4w", "fwd"), ("tiles64_8w", "fwd"), ("tiles64_8w", "dgrad")}


def _case(s, dtype, layout="nhwc"):
    name, n, c, h, w, k, r, stride, pad, dil, groups = s
    return U.Case(I.Layer(name, n, c, h, w, k, r, r, stride, pad, dil, groups), layout=layout, dtype=dtype,
                  x_kind="normal", cfg=98, layer_id=SHAPES.index(s), alpha=-0.5)


@pytest.mark.parametrize("dtype", [I.F16, I.BF16])
@pytest.mark.parametrize("s", SHAPES, ids=[s[0] for s in SHAPES])
def test_small_grid_parity(nnlib, oracle_lib, s, dtype):
    case = _case(s, dtype)
    for p in ("fwd", "dgrad"):
        if p == "dgrad" and s[0] in TINY_DGRAD:
            U.assert_runs(case, p, "igemm_tiny_kernel", 1)
        elif p == "dgrad" and s[0] in MIXED_DGRAD:
            U.assert_runs(case, p, "igemm_c64_kernel")
        else:
            U.assert_runs(case, p, "igemm_wk_kernel", *((64, 64) if (s[0], p) in TILES64 else (32, 32)))
    U.full_parity(case, passes=("fwd", "dgrad"))


@pytest.mark.parametrize("stride,launches", [(2, 1), (3, 1), (4, 1), (5, 25)])
def test_stride_phases_share_a_launch(nnlib, oracle_lib, stride, launches):
    """Up to 16 stride phases of backward-data are one launch."""
    case = U.Case(I.Layer("phases", 2, 40, 45, 46, 88, 5, 5, stride, 2), layer_id=30)
    gemms = [k for k in U.kernels(case, "dgrad") if "igemm" in k]
    assert len(gemms) == launches
    U.full_parity(case, passes=("dgrad",))


@pytest.mark.parametrize("s", [SHAPES[2], SHAPES[5], SHAPES[10], SHAPES[15]], ids=lambda s: s[0])
def test_small_grid_is_reproducible(nnlib, s):
    case = _case(s, I.F16)
    t = case.tensors()
    a, b = (U.run_gpu(case, t, ("fwd", "dgrad")) for _ in range(2))
    assert np.array_equal(a["y_bits"], b["y_bits"]) and np.array_equal(a["dx_bits"], b["dx_bits"])


@pytest.mark.parametrize("where", ["x", "w"])
def test_small_grid_block_diagonal_keeps_inf_in_its_half(nnlib, where):
    """An inf reaches at most the 32 channels that share its diagonal block,
    as in the larger block-diagonal tiles."""
    case = _case(SHAPES[15], I.F16)
    U.assert_runs(case, "fwd", "igemm_wk_kernel", 32, 32)
    t = case.tensors()
    t[where].reshape(t[where].shape[0], -1)[0, 0] = 0x7C00  # channel 0 / filter 0
    y = U.run_gpu(case, t, ("fwd",))["y"].reshape(U.shape_of(case, "y"))
    assert not np.all(np.isfinite(y[..., :32])) and np.all(np.isfinite(y[..., 32:]))


# Grids past the split-reduction tiles whose channels per tap are not a
# multiple of 64: the mixed-tap tiles of the 64-element-slice kernel.
MIX_SHAPES = [
    # name, n, c, h, w, k, r, stride, pad, dil, groups; columns and stages of the tile: fwd, dgrad
    ("c40k240", 2, 40, 112, 111, 240, 1, 1, 0, 1, 1, (128, 1), (64, 1)),        # one slice, ragged rows and columns
    ("c240k40", 2, 240, 112, 111, 40, 1, 1, 0, 1, 1, (64, 1), (128, 1)),        # 3.75 slices
    ("c24k72_s2", 3, 24, 120, 121, 72, 3, 2, 1, 1, 1, None, None),              # four phases, chunks across taps
    ("c24k72_s2_n6", 6, 24, 150, 151, 72, 3, 2, 1, 1, 1, (128, 2), (64, 1)),
    ("c8k16_5x5", 2, 8, 150, 151, 16, 5, 1, 2, 1, 1, (64, 1), (64, 1)),         # a tap per chunk, 25 taps
    ("c16k88_s3_n2", 2, 16, 200, 170, 88, 3, 3, 1, 1, 1, None, None),
    ("c16k88_s3", 4, 16, 250, 220, 88, 3, 3, 1, 1, 1, (128, 2), (64, 1)),       # nine phases
    ("c16k88_s4", 4, 16, 250, 220, 88, 3, 4, 1, 1, 1, None, (64, 1)),           # sixteen
    ("c264k72_2stage", 8, 264, 56, 56, 72, 1, 1, 0, 1, 1, (128, 2), (128, 1)),
    ("c72g3", 1, 72, 130, 131, 72, 3, 1, 1, 1, 3, (64, 1), (64, 1)),            # groups of 24
    ("c96g4_s2", 40, 96, 38, 37, 96, 1, 2, 0, 1, 4, None, (64, 1)),             # groups that share cache lines
]


# About one 128x128 tile per CU: the 8-wave form of that tile.
W8_SHAPES = [
    ("k512", 31, 512, 29, 28, 120, 1, 1, 0, 1, 1),           # ragged rows and columns
    ("k576", 15, 64, 57, 29, 136, 3, 1, 1, 1, 1),            # padded 3x3
]


@pytest.mark.parametrize("dtype", [I.F16, I.BF16])
@pytest.mark.parametrize("s", W8_SHAPES, ids=[s[0] for s in W8_SHAPES])
def test_eight_wave_tile(nnlib, oracle_lib, s, dtype):
    name, n, c, h, w, k, r, stride, pad, dil, groups = s
    case = U.Case(I.Layer(name, n, c, h, w, k, r, r, stride, pad, dil, groups), dtype=dtype,
                  x_kind="normal", cfg=102, layer_id=W8_SHAPES.index(s))
    U.assert_runs(case, "fwd", "igemm_c64_kernel", 128, 128, 4, 2)
    U.full_parity(case, passes=("fwd", "dgrad"))


@pytest.mark.parametrize("dtype", [I.F16, I.BF16])
@pytest.mark.parametrize("s", MIX_SHAPES, ids=[s[0] for s in MIX_SHAPES])
def test_mixed_tap_tiles(nnlib, oracle_lib, s, dtype):
    name, n, c, h, w, k, r, stride, pad, dil, groups, fwd, dgrad = s
    case = U.Case(I.Layer(name, n, c, h, w, k, r, r, stride, pad, dil, groups), dtype=dtype,
                  x_kind="normal", cfg=99, layer_id=MIX_SHAPES.index(s))
    for p, tile in (("fwd", fwd), ("dgrad", dgrad)):
        if tile:  # 128 rows x columns, 4 waves, 64-element slices, stages
            U.assert_runs(case, p, "igemm_c64_kernel", 128, tile[0], 2, 2, 8, tile[1])
    U.full_parity(case, passes=("fwd", "dgrad"))
