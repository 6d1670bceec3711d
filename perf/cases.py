"""Performance cases of the BEV pooling path.

A case is one call that a detector makes through the package's public
functions: the pooling of a frame from a stored schedule, the same from depth
logits, a training step, the building of a plan and its schedule, or a whole
frame whose cameras moved.  The rig is the one of the repository's workloads:
N pinhole cameras 60 degrees apart (70 degrees of horizontal view, stride-16
feature maps), here with a small yaw and shift per sample, as calibration
gives, and with the order of the cameras and flips of their images drawn from
the seed, as augmentation gives.

``listed`` gives the cases by name, ``draw`` more of the same ranges.  A state
holds what a program keeps between calls (the plan, the schedule, the forward's
workspace) and the call's inputs on the GPU.
"""

from __future__ import annotations

import functools
import math
import random

import torch

from paper_2211_17111_amd import bevpool as bp

STRIDE = 16.0
HFOV = math.radians(70.0)
CAM_HEIGHT = 1.5
Z_LO, Z_HI = -5.0, 3.0
MAX_WORK = 4 * 6 * 118 * 40 * 110 * 80  # frustum points x channels of the largest listed case
DTYPES = {"f32": (torch.float32, torch.float32), "f16": (torch.float16, torch.float16),
          "f16_f32": (torch.float16, torch.float32)}


def _case(name, op, B, N, H, W, D, C, X, Z=1, dtype="f32", step=None, half=51.2):
    """X = Y cells over [-half, half) metres, Z height bins over [-5, 3), D
    depth bins from 1 m in steps of ``step`` metres (59 m in all if not given)."""
    case = dict(op=op, B=B, N=N, H=H, W=W, D=D, C=C, X=X, Z=Z, dtype=dtype,
                step=59.0 / D if step is None else step, half=half)
    return dict(case, name=name) if name else case


def listed():
    return [
        # One small camera into a 16 x 16 grid: a call whose cost is its launches.
        _case("tiny_forward", "forward", 1, 1, 4, 8, 8, 16, 16, step=1.0, half=8.0),
        # A frame of the 256 x 704 detector with 59 bins and 64 channels.
        _case("frame_256x704", "forward", 1, 6, 16, 44, 59, 64, 128),
        # A frame of the 640 x 1600 detector (the workload bench.py times).
        _case("frame_640x1600", "forward", 1, 6, 40, 100, 118, 80, 128),
        # The same frame when the depth net hands over logits.
        _case("logits_640x1600", "softmax", 1, 6, 40, 100, 118, 80, 128),
        # The same frame into 16 height bins: many cells with few points each.
        _case("frame_voxels", "forward", 1, 6, 40, 100, 118, 80, 128, Z=16),
        # Four half-precision frames at 640 x 1760 into 0.4 m cells.
        _case("frames_f16", "forward", 4, 6, 40, 110, 118, 80, 256, dtype="f16"),
        # A training step of eight samples at 256 x 704: pooling and both gradients.
        _case("train_256x704", "step", 8, 6, 16, 44, 118, 80, 128),
        # The largest: a half-precision training step, four samples at 640 x 1760.
        _case("train_f16", "step", 4, 6, 40, 110, 118, 80, 256, dtype="f16"),
        # A step from the plan alone, as a program that builds no schedule runs it.
        _case("plan_step_640x1600", "plan_step", 1, 6, 40, 100, 118, 80, 128),
        # The plan and its schedule for a new rig, from the voxel indices.
        _case("build_640x1600", "build", 1, 6, 40, 100, 118, 80, 128),
        # A frame whose cameras moved: voxel indices, plan, schedule and pooling.
        _case("moving_256x704", "moving", 1, 6, 16, 44, 118, 80, 128),
        # Sizes that are multiples of nothing: five cameras, odd maps, bins and grid.
        _case("ragged_step", "step", 2, 5, 23, 61, 77, 52, 111),
    ]


def draw(rng: random.Random):
    def spread(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choice(["forward", "forward", "forward", "softmax", "step", "step", "step", "plan_step", "build",
                     "moving"])
    dtype = rng.choice(["f32", "f32", "f16", "f16_f32"])
    while True:
        B, N = spread(1, 8), rng.randint(1, 6)
        H, W, D = spread(4, 44), spread(8, 110), spread(8, 118)
        C = rng.choice([16, 32, 48, 52, 64, 72, 80, 80, 96, 128, rng.randint(17, 127)])
        X = rng.choice([128, 128, 256, spread(16, 256)])
        Z = rng.choice([1, 1, 1, 1, 2, 16])
        half = 51.2 if X >= 48 else 8.0
        step = 59.0 / D if half > 8.0 else 9.0 / D
        # (no dearer than the largest listed case: its points x channels, and
        # an output of no more than its cells)
        if B * N * D * H * W * C <= MAX_WORK and B * X * X * Z <= 4 * 256 * 256:
            return _case(None, op, B, N, H, W, D, C, X, Z, dtype, step, half)


# ------------------------------------------------------------------- the rig

def _shape(c):
    return dict(B=c["B"], N=c["N"], D=c["D"], H=c["H"], W=c["W"], C=c["C"], X=c["X"], Y=c["X"], Z=c["Z"])


def _frustum(c):
    return dict(stride=STRIDE, depth_start=1.0, depth_step=c["step"], lo=(-c["half"], -c["half"], Z_LO),
                res=(2.0 * c["half"] / c["X"], 2.0 * c["half"] / c["X"], (Z_HI - Z_LO) / c["Z"]))


def _cameras(c, seed):
    """float64 (B, N, 16): fx, fy, cx, cy, camera-to-ego rotation, translation.
    A sample's rig has a small yaw (up to 5 degrees) and shift (up to 0.5 m);
    the seed orders its cameras and flips their images, as augmentation does,
    so that every seed has another plan, of the same number of points."""
    jitter, rng = random.Random(c["N"]), random.Random(seed)
    focal = (c["W"] * STRIDE / 2.0) / math.tan(HFOV / 2.0)
    cams = torch.empty((c["B"], c["N"], bp.CAMERA_WORDS), dtype=torch.float64)
    for b in range(c["B"]):
        yaw = math.radians(jitter.uniform(-5.0, 5.0))
        dx, dy = jitter.uniform(-0.5, 0.5), jitter.uniform(-0.5, 0.5)
        for i, n in enumerate(rng.sample(range(c["N"]), c["N"])):
            s, k = math.sin(yaw + math.radians(60.0 * n)), math.cos(yaw + math.radians(60.0 * n))
            flips = (seed + b if i == 0 else rng.randrange(4)) % 4
            fx, fy = -focal if flips & 1 else focal, -focal if flips & 2 else focal
            cams[b, i] = torch.tensor([fx, fy, c["W"] * STRIDE / 2.0, c["H"] * STRIDE / 2.0,
                                       s, 0.0, k, -k, 0.0, s, 0.0, -1.0, 0.0, dx, dy, CAM_HEIGHT],
                                      dtype=torch.float64)
    return cams


def _voxels(c, cams):
    """int64 (B * N * D * H * W, 3) voxel indices, each operation rounded once
    in float64, in the order that bevpool_geometry documents."""
    f = _frustum(c)
    dev = cams.device
    u = ((torch.arange(c["W"], dtype=torch.float64, device=dev) + 0.5) * STRIDE).view(1, 1, 1, 1, -1)
    v = ((torch.arange(c["H"], dtype=torch.float64, device=dev) + 0.5) * STRIDE).view(1, 1, 1, -1, 1)
    d = (f["depth_start"] + torch.arange(c["D"], dtype=torch.float64, device=dev) * f["depth_step"])
    d = d.view(1, 1, -1, 1, 1)
    w = [cams[:, :, i].reshape(cams.shape[0], cams.shape[1], 1, 1, 1) for i in range(16)]
    xc, yc = ((u - w[2]) * d) / w[0], ((v - w[3]) * d) / w[1]
    idx = []
    for i in range(3):
        e = ((w[4 + 3 * i] * xc + w[5 + 3 * i] * yc) + w[6 + 3 * i] * d) + w[13 + i]
        e = torch.floor((e - f["lo"][i]) / f["res"][i]).clamp(-2.0 ** 30, 2.0 ** 30)
        idx.append(e.expand(cams.shape[0], c["N"], c["D"], c["H"], c["W"]).reshape(-1).to(torch.int64))
    return torch.stack(idx, dim=1)


def _kept(c, voxels):
    """Frustum index and cell of every kept point, in frustum order."""
    x, y, z = voxels[:, 0], voxels[:, 1], voxels[:, 2]
    keep = (x >= 0) & (x < c["X"]) & (y >= 0) & (y < c["X"]) & (z >= 0) & (z < c["Z"])
    p = torch.nonzero(keep).squeeze(1)
    b = p // (c["N"] * c["D"] * c["H"] * c["W"])
    return p, ((b * c["Z"] + z[p]) * c["X"] + y[p]) * c["X"] + x[p]


# -------------------------------------------------------------------- inputs

def _inputs(c, seed):
    """Image features and output gradients ~ N(0, 1), depth logits ~ 3 N(0, 1)
    and the scores their softmax over the bins gives."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    tin, tout = DTYPES[c["dtype"]]
    B, N, D, H, W, C = (c[k] for k in "BNDHWC")

    def normal(*size):
        return torch.randn(size, generator=gen, device="cuda", dtype=torch.float32)

    feat = normal(B, N, H, W, C).to(tin)
    logits = (3.0 * normal(B, N, D, H, W)).to(tin)
    depth = torch.softmax(logits.float(), dim=2).to(tin)
    grad = normal(B, c["Z"], c["X"], c["X"], C).to(tout)
    return feat, logits, depth, grad


def prepare(case, seed):
    feat, logits, depth, grad = _inputs(case, seed)
    cams = _cameras(case, seed).cuda()
    state = dict(op=case["op"], shape=_shape(case), frustum=_frustum(case), out_dtype=DTYPES[case["dtype"]][1])
    if case["op"] == "moving":
        return dict(state, cams=cams, feat=feat, depth=depth)
    coor = bp.geometry(cams, state["frustum"], state["shape"])
    if case["op"] == "build":
        return dict(state, coor=coor)
    plan = bp.prepare(coor, state["shape"])
    if case["op"] == "plan_step":
        return dict(state, plan=plan, depth=depth.requires_grad_(), feat=feat.requires_grad_(), grad=grad)
    sched = bp.schedule(plan)
    if case["op"] == "step":
        return dict(state, plan=sched, depth=depth.requires_grad_(), feat=feat.requires_grad_(), grad=grad)
    return dict(state, sched=sched, workspace=bp.forward_scheduled_workspace(sched), feat=feat,
                scores=logits if case["op"] == "softmax" else depth)


def _plan_arrays(plan):
    return [plan.ranks_depth, plan.ranks_feat, plan.ranks_bev, plan.interval_starts, plan.interval_lengths]


def run(state):
    op = state["op"]
    if op == "forward":
        return bp.forward_scheduled(state["scores"], state["feat"], state["sched"], state["out_dtype"],
                                    workspace=state["workspace"])
    if op == "softmax":
        return bp.forward_scheduled_softmax(state["scores"], state["feat"], state["sched"],
                                            out_dtype=state["out_dtype"], workspace=state["workspace"])
    if op in ("step", "plan_step"):
        depth, feat = state["depth"], state["feat"]
        out = bp.bev_pool(depth, feat, state["plan"], state["out_dtype"])
        return [out.detach(), *torch.autograd.grad(out, (depth, feat), state["grad"])]
    if op == "build":
        plan = bp.prepare(state["coor"], state["shape"])
        sched = bp.schedule(plan)
        return _plan_arrays(plan) + [torch.tensor(sched.counts[:8], dtype=torch.int32)]
    coor = bp.geometry(state["cams"], state["frustum"], state["shape"])
    plan = bp.prepare(coor, state["shape"])
    sched = bp.schedule(plan)
    return [coor, *_plan_arrays(plan), bp.forward_scheduled(state["depth"], state["feat"], sched, state["out_dtype"])]


# ------------------------------------------------------------ work, tolerance

@functools.lru_cache(maxsize=None)
def _counts(key):
    """Kept points and occupied cells of one sample of the rig."""
    c = dict(key, B=1)
    _, cell = _kept(c, _voxels(c, _cameras(c, 0)))
    return int(cell.numel()), int(torch.unique(cell).numel())


def work(case):
    """Bytes: of every input and output array what the call has to touch once
    (scores of kept points, features, the plan's two ranks and interval table,
    whole outputs; a gradient of the output for its occupied cells only; three
    voxel words per point).  Flops: one multiply-add per kept point and channel
    of each product."""
    c = case
    key = tuple((k, v) for k, v in sorted(c.items()) if k not in ("name", "op", "dtype", "B"))
    kept, occ = (c["B"] * v for v in _counts(key))
    tin, tout = DTYPES[c["dtype"]]
    si, so = tin.itemsize, tout.itemsize
    rows = c["B"] * c["N"] * c["H"] * c["W"]
    points, cells = rows * c["D"], c["B"] * c["Z"] * c["X"] * c["X"]
    plan = 8 * kept + 12 * occ
    out = so * cells * c["C"]
    forward = si * kept + si * rows * c["C"] + plan + out
    backward = so * occ * c["C"] + si * rows * c["C"] + si * kept + plan + si * points + si * rows * c["C"]
    fused = si * points + si * rows * c["C"] + plan + out
    built = 12 * kept + 8 * occ
    mac = 2 * kept * c["C"]
    total = {"forward": (forward, mac), "softmax": (fused, mac + 4 * points),
             "step": (forward + backward, 3 * mac), "plan_step": (forward + backward, 3 * mac),
             "build": (12 * points + built, 0),
             "moving": (12 * points + built + si * kept + si * rows * c["C"] + out, 40 * points + mac)}[c["op"]]
    return {"bytes": total[0], "flops": total[1]}


def tolerance(case):
    """Measured against ``exact``: float32 results are 5e-8 to 1.6e-7 off, and
    half-precision ones 2.1e-4, one rounding.  (Plans are whole numbers.)"""
    if case["op"] == "build":
        return "exact"
    if case["dtype"] == "f32":
        return {"rel": 1e-6, "max": 2e-5}
    return {"rel": 8e-4, "max": 4e-3}


# --------------------------------------------------------------------- exact

def _exact_plan(c, cell, p):
    order = torch.sort(cell, stable=True).indices
    rd, rb = p[order], cell[order]
    hw = c["H"] * c["W"]
    _, lengths = torch.unique_consecutive(rb, return_counts=True)
    starts = torch.cumsum(lengths, 0) - lengths
    rf = (rd // (c["D"] * hw)) * hw + rd % hw
    return [t.to(torch.int32) for t in (rd, rf, rb, starts, lengths)]


def exact(case, seed):
    """The same results in float64, the frustum feature formed view by view."""
    c = case
    feat, logits, depth, grad = _inputs(c, seed)
    voxels = _voxels(c, _cameras(c, seed).cuda())
    p, cell = _kept(c, voxels)
    plan = _exact_plan(c, cell, p) if c["op"] in ("build", "moving") else []
    if c["op"] == "build":
        return plan + [None]
    scores = torch.softmax(logits.double(), dim=2) if c["op"] == "softmax" else depth.double()
    C, hw = c["C"], c["H"] * c["W"]
    view_points = c["D"] * hw
    out = torch.zeros((c["B"] * c["Z"] * c["X"] * c["X"], C), dtype=torch.float64, device="cuda")
    gd, gf = torch.zeros_like(depth, dtype=torch.float64), torch.zeros_like(feat, dtype=torch.float64)
    rows, g, s = feat.reshape(-1, C), grad.reshape(-1, C), scores.reshape(-1)
    cuts = torch.searchsorted(p, torch.arange(c["B"] * c["N"] + 1, device="cuda") * view_points).tolist()
    for v, (lo, hi) in enumerate(zip(cuts[:-1], cuts[1:])):
        q, k = p[lo:hi], cell[lo:hi]
        f = v * hw + q % hw
        row = rows[f].double()
        out.index_add_(0, k, s[q].unsqueeze(1) * row)
        if "step" in c["op"]:
            up = g[k].double()
            gd.view(-1)[q] = (up * row).sum(1)
            gf.view(-1, C).index_add_(0, f, s[q].unsqueeze(1) * up)
    out = out.view(c["B"], c["Z"], c["X"], c["X"], C)
    if "step" in c["op"]:
        return [out, gd, gf]
    if c["op"] == "moving":
        return [voxels.to(torch.int32), *plan, out]
    return out
