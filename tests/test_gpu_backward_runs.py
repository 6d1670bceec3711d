"""The pixel kernel of both backwards against the float64 oracle: from the plan
alone where consecutive depth bins of a pixel share their cell (runs that end with
a chunk of bins, cross it or fill it, pixels of one bin, infinite gradients), and
in its channel layouts, launch sizes and the largest gradients.

Tolerance per element: |gpu - oracle| <= tol * sum|terms| + 1e-6, tol = 1e-5
(float32 inputs) or 2e-3 (float16 inputs).
"""

import numpy as np
import pytest
import torch

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


# 5, 6 and 8 channels per lane in groups of 8, 16 and 32 lanes; few pixels (8 pairs
# a step), and pixels for many waves (4 a step) whose last wave is not full
@pytest.mark.parametrize("C", [40, 48, 64, 80, 96, 160, 192])
@pytest.mark.parametrize("dtype,out_dtype", [("f32", "f32"), ("f16", "f16"), ("f16", "f32")])
@pytest.mark.parametrize("B,H,W,D", [(1, 3, 7, 20), (3, 73, 75, 4)])
@pytest.mark.parametrize("path", ["plan", "scheduled"])
def test_channel_layouts(C, dtype, out_dtype, B, H, W, D, path):
    shape = dict(B=B, N=1, D=D, H=H, W=W, C=C, X=5, Y=3, Z=1)
    data = draw_small(np.random.default_rng(C + D), shape, dtype=dtype, out_dtype=out_dtype)
    coor = _run_coor(shape, 2)
    plan = _gpu.run_prepare(coor, shape)
    args = [_gpu.to_dev(data[k]) for k in ("grad_out", "depth", "feat")]
    gd, gf = bp.backward(*args, plan) if path == "plan" else bp.backward_scheduled(*args, bp.schedule(plan))
    rgd, rgf, mgd, mgf = oracle.backward_ref(data["grad_out"], data["depth"], data["feat"], coor, shape)
    _gpu.assert_within(gd.float().cpu().numpy(), rgd, mgd, dtype, f"C={C} {path} grad_depth")
    _gpu.assert_within(gf.float().cpu().numpy(), rgf, mgf, dtype, f"C={C} {path} grad_feat")


# rows of one or two 32-byte vectors, and those around them
@pytest.mark.parametrize("C", [4, 8, 12, 16, 24])
@pytest.mark.parametrize("dtype,out_dtype", [("f32", "f32"), ("f16", "f32")])
@pytest.mark.parametrize("B,H,W,D", [(1, 3, 7, 20), (1, 73, 225, 4)])
@pytest.mark.parametrize("path", ["plan", "scheduled"])
def test_narrow_rows(C, dtype, out_dtype, B, H, W, D, path):
    test_channel_layouts(C, dtype, out_dtype, B, H, W, D, path)


# rows of two parts, the second of one lane up to all of them; few pixels and many
@pytest.mark.parametrize("C", [520, 768, 1024])
@pytest.mark.parametrize("dtype,out_dtype", [("f32", "f32"), ("f16", "f16"), ("f16", "f32")])
@pytest.mark.parametrize("B,H,W,D", [(1, 3, 7, 20), (1, 41, 55, 3)])
@pytest.mark.parametrize("path", ["plan", "scheduled"])
def test_rows_of_two_parts(C, dtype, out_dtype, B, H, W, D, path):
    test_channel_layouts(C, dtype, out_dtype, B, H, W, D, path)


@pytest.mark.parametrize("path", ["plan", "scheduled"])
def test_gradient_of_a_gibibyte(path):
    """grad_out of 1 GiB: its rows lie beyond what the 32-bit offsets address."""
    shape = dict(B=1, N=1, D=6, H=2, W=3, C=256, X=1024, Y=1024, Z=1)
    rng = np.random.default_rng(3)
    coor = np.stack([rng.integers(0, 1024, 36), rng.integers(0, 1024, 36), np.zeros(36, dtype=np.int64)], axis=1)
    coor[5] = (1023, 1023, 0)
    coor[7] = (-1, 3, 0)
    depth = rng.random((1, 1, 6, 2, 3), dtype=np.float32)
    feat = rng.standard_normal((1, 1, 2, 3, 256), dtype=np.float32)
    grad = torch.randn((1, 1, 1024, 1024, 256), device=_gpu.DEV, generator=torch.Generator(_gpu.DEV).manual_seed(1))
    plan = _gpu.run_prepare(coor.astype(np.int32), shape)
    args = (grad, _gpu.to_dev(depth), _gpu.to_dev(feat))
    gd, gf = bp.backward(*args, plan) if path == "plan" else bp.backward_scheduled(*args, bp.schedule(plan))
    kept = np.flatnonzero(coor[:, 0] >= 0)
    cells = torch.from_numpy(coor[kept, 1] * 1024 + coor[kept, 0]).to(_gpu.DEV)
    up = grad.view(-1, 256)[cells].double().cpu().numpy()
    rows = feat.reshape(-1, 256).astype(np.float64)[kept % 6]
    rgd, mgd, rgf, mgf = np.zeros(36), np.zeros(36), np.zeros((6, 256)), np.zeros((6, 256))
    rgd[kept], mgd[kept] = (up * rows).sum(1), np.abs(up * rows).sum(1)
    np.add.at(rgf, kept % 6, depth.reshape(-1)[kept, None] * up)
    np.add.at(mgf, kept % 6, depth.reshape(-1)[kept, None] * np.abs(up))
    _gpu.assert_within(gd.cpu().numpy().reshape(-1), rgd, mgd, "f32", f"{path} grad_depth")
    _gpu.assert_within(gf.cpu().numpy().reshape(6, 256), rgf, mgf, "f32", f"{path} grad_feat")
