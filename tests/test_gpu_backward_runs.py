"""The backward from the plan alone where consecutive depth bins of a pixel share
their cell, against the float64 oracle: runs that end with a chunk of bins, cross
it or fill it, pixels of one bin, and infinite gradients.

Tolerance per element: |gpu - oracle| <= tol * sum|terms| + 1e-6, tol = 1e-5
(float32 inputs) or 2e-3 (float16 inputs).
"""

import numpy as np
import pytest

import _gpu
import oracle
from paper_2211_17111_amd import bevpool as bp
from workloads import draw_small

pytestmark = pytest.mark.gpu


def _run_coor(shape, run):
    """Each pixel's bins go from cell to cell every `run` bins; some are dropped."""
    B, N, D, H, W, X, Y = (shape[k] for k in "BNDHWXY")
    b, n, d, h, w = np.indices((B, N, D, H, W))
    cell = ((d + h) // run + w + n) % (X * Y)
    coor = np.stack([cell % X, cell // X, np.where((d + w) % 11 == 5, -1, 0)], axis=-1)
    return coor.reshape(-1, 3).astype(np.int32)


def _backward(data, coor, shape):
    gd, gf = bp.backward(_gpu.to_dev(data["grad_out"]), _gpu.to_dev(data["depth"]), _gpu.to_dev(data["feat"]),
                         _gpu.run_prepare(coor, shape))
    return gd.float().cpu().numpy(), gf.float().cpu().numpy()


# C picks lane groups of 1 to 64 lanes, so chunks of 1 to 64 bins
@pytest.mark.parametrize("C", [1, 4, 20, 80, 260, 600])
@pytest.mark.parametrize("D,run", [(1, 1), (15, 4), (16, 16), (17, 5), (70, 40), (130, 3)])
@pytest.mark.parametrize("dtype", ["f32", "f16"])
def test_runs(C, D, run, dtype):
    shape = dict(B=2, N=1, D=D, H=3, W=7, C=C, X=5, Y=3, Z=1)
    data = draw_small(np.random.default_rng(C + D), shape, dtype=dtype)
    coor = _run_coor(shape, run)
    gd, gf = _backward(data, coor, shape)
    rgd, rgf, mgd, mgf = oracle.backward_ref(data["grad_out"], data["depth"], data["feat"], coor, shape)
    _gpu.assert_within(gd, rgd, mgd, dtype, f"C={C} D={D} run={run} grad_depth")
    _gpu.assert_within(gf, rgf, mgf, dtype, f"C={C} D={D} run={run} grad_feat")


def test_runs_with_an_infinite_gradient():
    """Scores of both signs and zeros against an infinite gradient of their cell:
    each point adds for itself, as in the oracle."""
    shape = dict(B=1, N=1, D=40, H=2, W=3, C=80, X=5, Y=1, Z=1)
    data = draw_small(np.random.default_rng(1), shape)
    coor = _run_coor(shape, 8)
    data["depth"][0, 0, ::7] = 0.0
    data["depth"][0, 0, 3::9] *= -1.0
    data["grad_out"][0, 0, 0, 2, 5] = np.inf
    gd, gf = _backward(data, coor, shape)
    with np.errstate(invalid="ignore"):
        rgd, rgf, mgd, mgf = oracle.backward_ref(data["grad_out"], data["depth"], data["feat"], coor, shape)
    assert np.array_equal(np.isnan(gf), np.isnan(rgf)) and np.isnan(rgf).any()
    for got, ref, mag in ((gd, rgd, mgd), (gf, rgf, mgf)):
        fine = np.isfinite(ref)
        assert np.array_equal(np.isfinite(got), fine)
        _gpu.assert_within(got[fine], ref[fine], mag[fine], "f32", "finite elements")
