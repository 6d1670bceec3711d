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
import _sched
import oracle
from paper_2211_17111_amd import bevpool as bp
from workloads import draw_small, random_coor

pytestmark = pytest.mark.gpu


def _dense(sched, half):
    """Whether the library pools the schedule on the matrix cores."""
    return _sched.dense_forward(sched.plan.shape, sched.plan.n_valid, sched.plan.n_intervals, sched.n_slots, half)


def _roomy(shape):
    """The grid with empty cells along x, at least as many as a pixel has bins: the
    rule then expects a pair per bin, so few cells do not make the bins fine."""
    return dict(shape, X=max(shape["X"], shape["D"]))


def _column_coor(shape, run):
    """Every pixel column of a view meets cell after cell, `run` bins each."""
    B, N, D, H, W, X, Y, Z = (shape[k] for k in "BNDHWXYZ")
    b, n, d, h, w = np.indices((B, N, D, H, W))
    cell = (d // run + (w // 2) + 3 * n) % (X * Y * Z)
    return np.stack([cell % X, cell // X % Y, cell // (X * Y)], axis=-1).reshape(-1, 3).astype(np.int32)


def _forward(coor, data, shape, out_dtype):
    sched = bp.schedule(_gpu.run_prepare(coor, shape))
    dense = _dense(sched, data["feat"].dtype == np.float16)
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


# strips of 3 x 17 and 5 x 7 pixels, of 17 x 6 in several bands, of 16 x 6 in
# several columns; runs of a whole ray down to single bins
@pytest.mark.parametrize("H,W,D,run,X", [(3, 17, 70, 30, 3), (5, 7, 118, 59, 5), (40, 6, 112, 1, 40), (16, 44, 59, 4, 16)])
def test_dense_strips(H, W, D, run, X):
    shape = dict(B=1, N=3, D=D, H=H, W=W, C=80, X=X, Y=4, Z=1)
    data = draw_small(np.random.default_rng(H), shape)
    coor = _column_coor(shape, run)
    shape = _roomy(shape)
    out, dense, _ = _forward(coor, data, shape, "f32")
    assert dense, "the case is meant for the matrix cores"
    ref, mag = oracle.forward_ref(data["depth"], data["feat"], coor, shape)
    _gpu.assert_within(out, ref, mag, "f32", f"{H}x{W} D={D}")


# runs of bins around the number of depth scores taken at a time; 41 rows (segments
# that see most of a strip's pixels) or 2 (few of them: not on the matrix cores)
@pytest.mark.parametrize("H,dtype,C,run", [(41, dtype, C, run) for dtype, C in (("f32", 80), ("f16", 72))
                                           for run in (1, 2, 3, 5, 6, 7, 10, 11, 14, 40)]
                         + [(2, "f32", 80, run) for run in (6, 7, 10, 11, 40)])
@pytest.mark.parametrize("logits", [False, True])
def test_dense_points_per_pair(H, dtype, C, run, logits):
    shape = dict(B=1, N=2, D=5 * run, H=H, W=20 if H > 2 else 40, C=C, X=3 if H > 2 else 8, Y=2, Z=1)
    data = draw_small(np.random.default_rng(run), shape, dtype=dtype, softmax=not logits)
    coor = _column_coor(shape, run)
    if H == 2:
        coor.reshape(2, -1, 2, 40, 3)[:, 3 * run:] = -1    # three pairs to a pixel
    sched = bp.schedule(_gpu.run_prepare(coor, shape))
    assert _dense(sched, dtype == "f16") == (H > 2)
    forward, ref = ((bp.forward_scheduled_softmax, oracle.forward_softmax_ref) if logits
                    else (bp.forward_scheduled, oracle.forward_ref))
    out = forward(_gpu.to_dev(data["depth"]), _gpu.to_dev(data["feat"]), sched)
    want, mag = ref(data["depth"], data["feat"], coor, shape)
    _gpu.assert_within(out.cpu().numpy(), want, mag, dtype, f"run={run} H={H}")


# A pixel meets a cell again and again (runs of pairs of one segment and pixel),
# up to more pairs in a segment than the byte index numbers
@pytest.mark.parametrize("X,Y,D", [(2, 2, 40), (1, 2, 118), (3, 3, 200)])
def test_dense_repeated_pixels(X, Y, D):
    shape = dict(B=1, N=2, D=D, H=9, W=11, C=80, X=X, Y=Y, Z=1)
    rng = np.random.default_rng(D)
    data = draw_small(rng, shape)
    coor = random_coor(rng, shape, spread=1)
    shape = _roomy(shape)
    out, dense, _ = _forward(coor, data, shape, "f32")
    assert dense, "the case is meant for the matrix cores"
    ref, mag = oracle.forward_ref(data["depth"], data["feat"], coor, shape)
    _gpu.assert_within(out, ref, mag, "f32", f"X={X} Y={Y} D={D}")


def _alternate_coor(shape):
    """Every pixel's bins go to and fro among few cells: each bin a pair of its own,
    and segments of more pairs than a strip has pixels."""
    B, N, D, H, W, X, Y = (shape[k] for k in "BNDHWXY")
    b, n, d, h, w = np.indices((B, N, D, H, W))
    cell = (d * (h % 3 + 1) + w // 3 + n) % (X * Y)
    return np.stack([cell % X, cell // X, 0 * cell], axis=-1).reshape(-1, 3).astype(np.int32)


# lane groups of 1 to 64 lanes, of channels in one chunk or several; segments that
# fill an item, cross many groups' ranges, or end inside them
@pytest.mark.parametrize("C,dtype,out_dtype", [(40, "f32", "f32"), (52, "f32", "f32"), (80, "f16", "f32"),
                                               (128, "f16", "f16"), (256, "f32", "f32"), (260, "f32", "f32"),
                                               (264, "f16", "f16"), (520, "f16", "f32")])
@pytest.mark.parametrize("X,Y,D,H,W", [(2, 1, 64, 9, 11), (3, 1, 65, 40, 5), (5, 3, 75, 8, 33), (9, 7, 128, 3, 16)])
@pytest.mark.parametrize("logits", [False, True])
def test_dense_walked_items(X, Y, D, H, W, C, dtype, out_dtype, logits):
    shape = dict(B=1, N=2, D=D, H=H, W=W, C=C, X=X, Y=Y, Z=1)
    data = draw_small(np.random.default_rng(C + D), shape, dtype=dtype, out_dtype=out_dtype, softmax=not logits)
    coor = _alternate_coor(shape)
    shape = _roomy(shape)
    sched = bp.schedule(_gpu.run_prepare(coor, shape))
    assert _dense(sched, dtype == "f16")
    forward, ref = ((bp.forward_scheduled_softmax, oracle.forward_softmax_ref) if logits
                    else (bp.forward_scheduled, oracle.forward_ref))
    args = (_gpu.to_dev(data["depth"]), _gpu.to_dev(data["feat"]), sched)
    outs = [forward(*args, out_dtype=_gpu.torch_dtype(out_dtype)) for _ in range(2)]
    assert torch.equal(outs[0], outs[1])
    want, mag = ref(data["depth"], data["feat"], coor, shape)
    _gpu.assert_within(outs[0].cpu().numpy(), want, mag, dtype, f"{shape} {dtype} {out_dtype}")


def test_dense_walked_item_with_infinite_features():
    """Pairs of one pixel and cell, one of score 0, against an infinite feature:
    each adds for itself, so their cell is NaN."""
    shape = dict(B=1, N=1, D=48, H=40, W=4, C=80, X=3, Y=1, Z=1)
    data = draw_small(np.random.default_rng(8), shape)
    coor = _alternate_coor(shape)
    shape = _roomy(shape)
    data["depth"] = np.abs(data["depth"]) + np.float32(0.01)
    data["feat"][0, 0, 21, 1, 3] = np.inf
    data["depth"][0, 0, 9, 21, 1] = 0.0
    data["feat"][0, 0, 31, 2, 5] = -np.inf
    out, dense, _ = _forward(coor, data, shape, "f32")
    assert dense, "the case is meant for the matrix cores"
    with np.errstate(invalid="ignore"):
        ref, mag = oracle.forward_ref(data["depth"], data["feat"], coor, shape)
    assert np.isnan(ref).sum() == 1 and np.isinf(ref).sum() > 1
    fine = np.isfinite(ref)
    assert np.array_equal(out[~fine].astype(np.float64), ref[~fine], equal_nan=True)
    _gpu.assert_within(out[fine], ref[fine], mag[fine], "f32", "finite elements")


def _fastest(call, runs=5):
    """Shortest time of a call in ms."""
    call()
    times = []
    for _ in range(runs):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        call()
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b))
    return min(times)


def test_dense_repeated_pixels_stay_fast():
    """Random cells: the scheduled forward takes at most 3 times as long as the
    plan's (measured: 0.34; with each lane on its own through a segment of a
    thousand pairs: 60)."""
    shape = dict(B=1, N=6, D=118, H=40, W=100, C=80, X=3, Y=3, Z=1)
    data = draw_small(np.random.default_rng(3), dict(shape, D=1), softmax=False)
    plan = _gpu.run_prepare(random_coor(np.random.default_rng(3), shape, spread=1), shape)
    sched = bp.schedule(plan)
    assert _dense(sched, False)
    depth = torch.rand((1, 6, 118, 40, 100), device=_gpu.DEV)
    feat = _gpu.to_dev(data["feat"])
    assert _fastest(lambda: bp.forward_scheduled(depth, feat, sched)) < 3 * _fastest(lambda: bp.forward(depth, feat, plan))


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


# channels of whole tiles, of part of one, of two chunks; float16's tiles in pairs and alone
@pytest.mark.parametrize("C,dtype,out_dtype", [(80, "f32", "f32"), (52, "f32", "f32"), (264, "f32", "f32"),
                                               (48, "f16", "f32"), (72, "f16", "f16"), (128, "f16", "f32"),
                                               (264, "f16", "f16")])
@pytest.mark.parametrize("logits", [False, True])
def test_dense_infinite_features_in_every_layout(C, dtype, out_dtype, logits):
    shape = dict(B=1, N=2, D=48, H=23, W=13, C=C, X=8, Y=3, Z=1)
    data = draw_small(np.random.default_rng(C), shape, dtype=dtype, out_dtype=out_dtype, softmax=not logits)
    if not logits:
        data["depth"] = np.abs(data["depth"]) + np.asarray(0.01, dtype=data["depth"].dtype)
    coor = _column_coor(shape, 6)
    coor.reshape(2, 48, 23, 13, 3)[0, 8:, 5, 4] = -1
    for h, w, c, x in [(5, 4, 0, np.inf), (11, 0, C - 1, -np.inf), (22, 12, C // 2, np.nan), (0, 7, 17, np.inf)]:
        data["feat"][0, 0, h, w, c] = x
    shape = _roomy(shape)
    sched = bp.schedule(_gpu.run_prepare(coor, shape))
    assert _dense(sched, dtype == "f16")
    forward, ref = ((bp.forward_scheduled_softmax, oracle.forward_softmax_ref) if logits
                    else (bp.forward_scheduled, oracle.forward_ref))
    out = forward(_gpu.to_dev(data["depth"]), _gpu.to_dev(data["feat"]), sched, out_dtype=_gpu.torch_dtype(out_dtype))
    out = out.cpu().numpy()
    with np.errstate(invalid="ignore"):
        want, mag = ref(data["depth"], data["feat"], coor, shape)
    fine = np.isfinite(want)
    assert (~fine).sum() > 8 and fine.sum() > 8
    assert np.array_equal(out[~fine].astype(np.float64), want[~fine], equal_nan=True)
    _gpu.assert_within(out[fine], want[fine], mag[fine], dtype, "finite elements")


def test_dense_infinite_features_stay_fast():
    """A feature map of infinities takes at most 4 times as long as a finite one
    (640x1600: 1.6, and 1.5 with one infinity; with a chain of global loads per pair
    and channel: 38)."""
    shape = dict(B=1, N=6, D=118, H=40, W=100, C=80, X=40, Y=8, Z=1)
    sched = bp.schedule(_gpu.run_prepare(_column_coor(shape, 4), shape))
    assert _dense(sched, False)
    depth = torch.rand((1, 6, 118, 40, 100), device=_gpu.DEV)
    feat = torch.randn((1, 6, 40, 100, 80), device=_gpu.DEV)
    finite = _fastest(lambda: bp.forward_scheduled(depth, feat, sched))
    assert _fastest(lambda: bp.forward_scheduled(depth, feat / 0, sched)) < 4 * finite
    feat[0, :, 7::16, 5::16, 3] = float("inf")
    assert _fastest(lambda: bp.forward_scheduled(depth, feat, sched)) < 4 * finite


def _leave_in_lds(value):
    """Fills every compute unit's staged rows and weights with `value`."""
    shape = dict(B=1, N=6, D=40, H=40, W=100, C=64, X=4, Y=4, Z=1)
    sched = bp.schedule(_gpu.run_prepare(_column_coor(shape, 10), shape))
    assert _dense(sched, False)
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
    shape = _roomy(shape)
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


def _cells_coor(shape, rows, run):
    """Runs of `run` bins and bands of `rows` image rows, shifted from column to
    column, each a cell of its own: strips of many segments of few pixels."""
    B, N, D, H, W, X, Y = (shape[k] for k in "BNDHWXY")
    b, n, d, h, w = np.indices((B, N, D, H, W))
    bands, runs = -(-H // rows), -(-D // run)
    cell = ((n * W + w) * bands + (h + 2 * w) % H // rows) * runs + d // run
    assert cell.max() < X * Y
    return np.stack([cell % X, cell // X, 0 * cell], axis=-1).reshape(-1, 3).astype(np.int32)


def _tiles_and_rounds(sched, shape, dtype, logits):
    """Most tiles of 16 segments that an item takes at once, and most rounds of the
    index table."""
    n = sched.plan.n_valid
    got = _sched.decode(sched.buffer.cpu().numpy(), shape, n, sched.plan.n_intervals)
    segs = int(np.diff(got["item_seg0"]).max())
    table = _sched.dense_table(shape, n, dtype == "f16", logits, got["n"]["shares"])
    return -(-min(segs, table) // 16), -(-segs // table)


def _check_many_segments(shape, coor, dtype, out_dtype, logits, tiles, rounds):
    data = draw_small(np.random.default_rng(shape["C"]), shape, dtype=dtype, out_dtype=out_dtype, softmax=not logits)
    # infinite and NaN features at both ends of a strip and inside it
    for h, w, c, x in [(0, 0, 1, np.inf), (shape["H"] - 1, 1, shape["C"] - 1, np.nan), (17, 2, 9, -np.inf)]:
        data["feat"][0, 0, h, w, c] = x
    if not logits:
        data["depth"] = np.abs(data["depth"]) + np.asarray(0.01, dtype=data["depth"].dtype)
    sched = bp.schedule(_gpu.run_prepare(coor, shape))
    assert _dense(sched, dtype == "f16")
    got = _tiles_and_rounds(sched, shape, dtype, logits)
    assert got[0] >= tiles and got[1] >= rounds, got
    forward, ref = ((bp.forward_scheduled_softmax, oracle.forward_softmax_ref) if logits
                    else (bp.forward_scheduled, oracle.forward_ref))
    out = forward(_gpu.to_dev(data["depth"]), _gpu.to_dev(data["feat"]), sched, out_dtype=_gpu.torch_dtype(out_dtype))
    out = out.cpu().numpy()
    with np.errstate(invalid="ignore"):
        want, mag = ref(data["depth"], data["feat"], coor, shape)
    fine = np.isfinite(want)
    assert (~fine).sum() > 8
    assert np.array_equal(out[~fine].astype(np.float64), want[~fine], equal_nan=True)
    _gpu.assert_within(out[fine], want[fine], mag[fine], dtype, f"{shape} {dtype} {out_dtype}")


# three tiles and more, in one pass of channels and in several, of 2 to 5 channel tiles
@pytest.mark.parametrize("C", [40, 52, 80, 96, 128, 264, 520])
@pytest.mark.parametrize("dtype,out_dtype", [("f32", "f32"), ("f16", "f16"), ("f16", "f32")])
@pytest.mark.parametrize("logits", [False, True])
def test_dense_many_tiles(C, dtype, out_dtype, logits):
    if dtype == "f16" and C % 8:
        C += 4
    shape = dict(B=1, N=2, D=48, H=41, W=4, C=C, X=432, Y=2, Z=1)
    _check_many_segments(shape, _cells_coor(shape, 5, 8), dtype, out_dtype, logits, tiles=3, rounds=1)


# items of more segments than the index table holds: the table again and again, with
# the strips too many for the large one (a table of 48 to 112), and with few strips
@pytest.mark.parametrize("B,N,W,D,run,C,dtype,out_dtype", [(4, 8, 45, 16, 4, 36, "f32", "f32"), (4, 8, 45, 24, 6, 64, "f32", "f32"),
                                                           (4, 8, 45, 18, 5, 40, "f16", "f16"), (4, 8, 45, 18, 5, 40, "f16", "f32"),
                                                           (1, 2, 4, 48, 8, 40, "f32", "f32"), (1, 2, 4, 48, 8, 40, "f16", "f32")])
@pytest.mark.parametrize("logits", [False, True])
def test_dense_rounds_of_the_index_table(B, N, W, D, run, C, dtype, out_dtype, logits):
    shape = dict(B=B, N=N, D=D, H=40 if B > 1 else 41, W=W, C=C, X=160, Y=72 if B > 1 else 3, Z=1)
    rows = 8 if C == 36 else 5
    _check_many_segments(shape, _cells_coor(shape, rows, run), dtype, out_dtype, logits, tiles=3, rounds=2)


@pytest.mark.parametrize("dtype,unit", [("f32", 2.0 ** -149), ("f16", 2.0 ** -24)])
@pytest.mark.parametrize("tiny", ["feat", "depth"])
def test_dense_keeps_subnormal_operands(dtype, unit, tiny):
    """Whole multiples of the smallest subnormal: sums below 2^23 of it, exact in any
    order."""
    shape = dict(B=1, N=1, D=12, H=40, W=4, C=80, X=12, Y=4, Z=1)
    coor = _column_coor(shape, 3)
    rng = np.random.default_rng(9)
    np_type = np.float16 if dtype == "f16" else np.float32
    whole = dict(depth=rng.integers(1, 4, (1, 1, 12, 40, 4)), feat=rng.integers(-100, 100, (1, 1, 40, 4, 80)))
    data = {k: (v * (unit if k == tiny else 1.0)).astype(np_type) for k, v in whole.items()}
    out, dense, _ = _forward(coor, data, shape, "f32")
    assert dense, "the case is meant for the matrix cores"
    ref, _ = oracle.forward_ref(whole["depth"].astype(np.float64), whole["feat"].astype(np.float64), coor, shape)
    assert np.abs(ref).max() < 2 ** 23 and np.abs(ref).max() > 0
    assert np.array_equal(out.astype(np.float64) / unit, ref)
