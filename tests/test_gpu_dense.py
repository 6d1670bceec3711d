"""The scheduled forward on the matrix cores (plans with many points per
segment) against the float64 oracle, at the edges of its tiles and of its rule,
and with infinite and NaN features.

Tolerance per element: |gpu - oracle| <= tol * sum|terms| + 1e-6, tol = 1e-5
(float32 inputs) or 2e-3 (float16 inputs).
"""

import numpy as np
import pytest
import torch

import _gpu
import oracle
from paper_2211_17111_amd import bevpool as bp
from workloads import draw_small, random_coor

pytestmark = pytest.mark.gpu

MIN_POINTS = 18  # points per segment from which the forward multiplies


def _column_coor(shape, run):
    """Every pixel column of a view meets cell after cell, `run` bins each."""
    B, N, D, H, W, X, Y, Z = (shape[k] for k in "BNDHWXYZ")
    b, n, d, h, w = np.indices((B, N, D, H, W))
    cell = (d // run + (w // 2) + 3 * n) % (X * Y * Z)
    return np.stack([cell % X, cell // X % Y, cell // (X * Y)], axis=-1).reshape(-1, 3).astype(np.int32)


def _forward(coor, data, shape, out_dtype):
    sched = bp.schedule(_gpu.run_prepare(coor, shape))
    dense = sched.plan.n_valid >= MIN_POINTS * (sched.plan.n_intervals + sched.n_slots)
    out = bp.forward_scheduled(_gpu.to_dev(data["depth"]), _gpu.to_dev(data["feat"]), sched,
                               out_dtype=_gpu.torch_dtype(out_dtype))
    return out.cpu().numpy(), dense, sched


# strips of 3 x 17, 5 x 7 and 41 x 2 pixels and more: pixels of no whole matrix
# tile; channels of one tile, of a part of one, of an odd number, of two chunks
@pytest.mark.parametrize("C", [40, 52, 80, 96, 128, 264, 520])
@pytest.mark.parametrize("dtype,out_dtype", [("f32", "f32"), ("f16", "f16"), ("f16", "f32")])
def test_dense_channels(C, dtype, out_dtype):
    if dtype == "f16" and C % 8:
        C += 4
    shape = dict(B=2, N=2, D=48, H=41, W=9, C=C, X=7, Y=3, Z=2)
    data = draw_small(np.random.default_rng(C), shape, dtype=dtype, out_dtype=out_dtype)
    coor = _column_coor(shape, 12)
    out, dense, _ = _forward(coor, data, shape, out_dtype)
    assert dense, "the case is meant for the matrix cores"
    ref, mag = oracle.forward_ref(data["depth"], data["feat"], coor, shape)
    _gpu.assert_within(out, ref, mag, dtype, f"C={C} {dtype} {out_dtype}")


# (3, 17) one image row of odd pixels; a strip whose segments outnumber the
# index table (many cells, short runs over many rows); one point in all
@pytest.mark.parametrize("H,W,D,run,X", [(3, 17, 70, 30, 3), (5, 7, 118, 59, 5), (40, 6, 112, 1, 40), (16, 44, 59, 4, 16)])
def test_dense_strips(H, W, D, run, X):
    shape = dict(B=1, N=3, D=D, H=H, W=W, C=80, X=X, Y=4, Z=1)
    data = draw_small(np.random.default_rng(H), shape)
    coor = _column_coor(shape, run)
    out, dense, _ = _forward(coor, data, shape, "f32")
    assert dense, "the case is meant for the matrix cores"
    ref, mag = oracle.forward_ref(data["depth"], data["feat"], coor, shape)
    _gpu.assert_within(out, ref, mag, "f32", f"{H}x{W} D={D}")


# A pixel meets a cell again and again (runs of pairs of one segment and pixel),
# up to more pairs in a segment than the byte index numbers
@pytest.mark.parametrize("X,Y,D", [(2, 2, 40), (1, 2, 118), (3, 3, 200)])
def test_dense_repeated_pixels(X, Y, D):
    shape = dict(B=1, N=2, D=D, H=9, W=11, C=80, X=X, Y=Y, Z=1)
    rng = np.random.default_rng(D)
    data = draw_small(rng, shape)
    coor = random_coor(rng, shape, spread=1)
    out, dense, _ = _forward(coor, data, shape, "f32")
    assert dense, "the case is meant for the matrix cores"
    ref, mag = oracle.forward_ref(data["depth"], data["feat"], coor, shape)
    _gpu.assert_within(out, ref, mag, "f32", f"X={X} Y={Y} D={D}")


@pytest.mark.parametrize("dtype", ["f32", "f16"])
def test_dense_infinite_and_nan_features(dtype):
    """An infinite or NaN feature reaches the cells its pixel's points fall in,
    and no other cell of its strip."""
    shape = dict(B=1, N=2, D=48, H=40, W=6, C=80, X=8, Y=3, Z=1)
    data = draw_small(np.random.default_rng(5), shape, dtype=dtype)
    coor = _column_coor(shape, 6)
    coor.reshape(2, 48, 40, 6, 3)[:, :, 13, :, 0] = -1         # row 13: no kept points ...
    coor.reshape(2, 48, 40, 6, 3)[0, 7, 13, 3] = (5, 2, 0)     # ... but one of column 3
    data["depth"] = np.abs(data["depth"]) + np.asarray(0.01, dtype=data["depth"].dtype)
    data["feat"][0, 0, 13, 3, 7] = np.inf
    data["feat"][0, 1, 13, 1, 11] = np.nan                     # its pixel has no points
    data["feat"][0, 1, 20, 2, 9] = -np.inf
    out, dense, _ = _forward(coor, data, shape, dtype)
    assert dense, "the case is meant for the matrix cores"
    with np.errstate(invalid="ignore"):
        ref, mag = oracle.forward_ref(data["depth"], data["feat"], coor, shape)
    fine = np.isfinite(ref)
    assert np.array_equal(np.isfinite(out), fine)
    assert np.array_equal(out[~fine].astype(np.float64), ref[~fine])
    assert (~fine).sum() > 1
    _gpu.assert_within(out[fine], ref[fine], mag[fine], dtype, "finite elements")


def _leave_in_lds(value):
    """Fills every compute unit's staged rows and weights with `value`."""
    shape = dict(B=1, N=6, D=40, H=40, W=100, C=64, X=4, Y=4, Z=1)
    sched = bp.schedule(_gpu.run_prepare(_column_coor(shape, 10), shape))
    assert sched.plan.n_valid >= MIN_POINTS * (sched.plan.n_intervals + sched.n_slots)
    bp.forward_scheduled(torch.full((1, 6, 40, 40, 100), value, device=_gpu.DEV),
                         torch.full((1, 6, 40, 100, 64), value, device=_gpu.DEV), sched)


@pytest.mark.parametrize("C,dtype,out_dtype", [(52, "f32", "f32"), (36, "f32", "f32"), (100, "f32", "f32"),
                                               (72, "f16", "f32"), (72, "f16", "f16"), (40, "f16", "f32")])
@pytest.mark.parametrize("H,W", [(23, 61), (7, 19)])
def test_dense_bits_do_not_depend_on_what_lds_held(H, W, C, dtype, out_dtype):
    """Channels that do not fill their matrix tiles: the tiles' other rows read
    past the staged features."""
    shape = dict(B=1, N=2, D=48, H=H, W=W, C=C, X=9, Y=3, Z=1)
    data = draw_small(np.random.default_rng(C), shape, dtype=dtype, out_dtype=out_dtype)
    coor = _column_coor(shape, 6)
    outs = []
    for value in (0.0, float("nan"), float("inf")):
        _leave_in_lds(value)
        out, dense, _ = _forward(coor, data, shape, out_dtype)
        assert dense, "the case is meant for the matrix cores"
        outs.append(out)
    ref, mag = oracle.forward_ref(data["depth"], data["feat"], coor, shape)
    _gpu.assert_within(outs[0], ref, mag, dtype, f"C={C} {dtype} {out_dtype}")
    for out in outs[1:]:
        assert (out != outs[0]).sum() == 0


def test_dense_zero_weight_of_an_infinite_feature():
    """A kept point of score 0 and an infinite feature make its cell NaN."""
    shape = dict(B=1, N=1, D=40, H=40, W=4, C=80, X=4, Y=1, Z=1)
    data = draw_small(np.random.default_rng(6), shape)
    coor = _column_coor(shape, 10)
    data["feat"][0, 0, 20, 1, 3] = np.inf
    data["depth"][0, 0, :, 20, 1] = 0.0
    out, dense, _ = _forward(coor, data, shape, "f32")
    assert dense, "the case is meant for the matrix cores"
    with np.errstate(invalid="ignore"):
        ref, mag = oracle.forward_ref(data["depth"], data["feat"], coor, shape)
    nan = np.isnan(ref)
    assert nan.any() and np.array_equal(np.isnan(out), nan)
    _gpu.assert_within(out[~nan], ref[~nan], mag[~nan], "f32", "finite elements")
