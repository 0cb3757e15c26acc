"""Performance cases of the BEV pooling: the calls that a camera-to-BEV model makes.

Every case is a camera rig (cameras on a ring, as on a car), a frustum, a BEV
grid and per-frame inputs, and one of three uses:

  pool    a plan kept from the calibration, and frames pooled with it
          (``Plan.forward`` / ``SlabPlan.forward``), where asked handed on as
          channel planes (``to_nchw``): inference
  train   pooling as a differentiable layer (``bev_pool``): the map and the
          gradients of the depth probabilities and of the features
  replan  a plan built for this frame's calibration and one frame pooled
          with it: calibration that changes per sample (augmentation, online
          calibration)

``pitch`` and ``roll`` (degrees) tilt every camera: 0 is the ideal rig, about
1 what mounted cameras have, about 5 what rotation augmentation adds. The
association of points and cells in ``exact`` is evaluated in numpy float64 in
the order that include/bevpool.h states; the sums are plain torch in float64.
"""
import math
import types

import numpy as np
import torch

import paper_2205_13542_amd as bev

_TORCH = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}

# Six cameras, 32x88 features (256x704 images at stride 8), 118 depth bins of
# 0.5 m, 80 channels, 360x360 cells of 0.3 m: the typical frame.
_FRAME = {"use": "pool", "cams": 6, "h": 32, "w": 88, "bins": 118, "grid": 360, "nz": 1, "channels": 80,
          "batch": 1, "dtype": "f32", "reduce": "sum", "depth": "peaked", "pitch": 0.0, "roll": 0.0,
          "nchw": False}
# The same rig at twice the resolution everywhere: 512x1408 images, 236 bins
# of 0.25 m, 128 channels, 720x720 cells of 0.15 m.
_HIGH = dict(_FRAME, h=64, w=176, bins=236, grid=720, channels=128, depth="sparse")


def listed():
    return [
        # one small camera on a coarse grid: what a call costs at least
        dict(_FRAME, name="tiny", cams=1, h=4, w=8, bins=8, grid=16, channels=8, depth="normal"),
        # the typical frame in fp32, one at a time: online inference
        dict(_FRAME, name="frame"),
        # mounted cameras, half-precision network, map as planes for the convolutional BEV encoder
        dict(_FRAME, name="mounted_bf16_nchw", dtype="bf16", pitch=1.0, roll=0.5, nchw=True),
        # strongly tilted cameras (rotation augmentation), half precision
        dict(_FRAME, name="tilted_f16", dtype="f16", pitch=5.0, roll=2.0),
        # sizes that divide nothing: five cameras, odd maps, odd channels, mean aggregation
        dict(_FRAME, name="odd_mean", cams=5, h=29, w=51, bins=59, grid=187, channels=67, pitch=0.7,
             roll=0.3, reduce="mean"),
        # eight frames per call: offline inference
        dict(_FRAME, name="batch8", batch=8),
        # the high-resolution frame (16 M points)
        dict(_HIGH, name="highres"),
        # four stacked z slabs, their channels concatenated
        dict(_FRAME, name="slabs4", nz=4),
        # a training step of the layer on the ideal rig
        dict(_FRAME, name="train", use="train"),
        # mounted cameras, mixed precision, two frames per GPU
        dict(_FRAME, name="train_mounted_bf16", use="train", dtype="bf16", batch=2, pitch=1.0, roll=0.5),
        # a training step at high resolution
        dict(_HIGH, name="train_highres", use="train"),
        # new calibration with every frame
        dict(_FRAME, name="replan", use="replan", pitch=1.0, roll=0.5),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    limit = 0.25 * _cost(_HIGH)
    while True:
        c = dict(_FRAME, use=rng.choice(["pool", "pool", "pool", "train", "train", "replan"]),
                 cams=rng.randint(1, 8), h=_log(rng, 6, 64), w=_log(rng, 12, 176), bins=_log(rng, 12, 236),
                 grid=_log(rng, 40, 720), batch=_log(rng, 1, 8),
                 channels=rng.choice([16, 32, 64, 80, 96, 128, rng.randint(5, 160), 8 * rng.randint(1, 20)]),
                 dtype=rng.choice(["f32", "bf16", "f16"]), depth=rng.choice(["peaked", "normal", "sparse"]),
                 pitch=rng.choice([0.0, round(rng.uniform(0.1, 2.0), 2), round(rng.uniform(0.1, 6.0), 2)]))
        c["roll"] = round(0.45 * c["pitch"], 3)
        if c["use"] == "pool":
            c["reduce"] = rng.choice(["sum", "sum", "sum", "mean", "max"])
            c["nz"] = rng.choice([1, 1, 1, 2, 4])
            c["nchw"] = rng.random() < 0.25
        # two and more points per cell of the map's outline, and no map of 2 GiB
        if c["cams"] * c["w"] * c["bins"] < 4 * c["grid"] or c["grid"] ** 2 * c["nz"] * c["channels"] >= 1 << 28:
            continue
        if _cost(c) <= limit:
            return c


def _cost(c):
    return c["batch"] * c["channels"] * (c["cams"] * c["h"] * c["w"] * c["bins"] + 4 * c["nz"] * c["grid"] ** 2)


# ------------------------------------------------------------------ rig

def _rig(c, jitter=None):
    """Cameras on a ring of 1 m at 1.5 m height facing outward, pitched and
    rolled; depth 1..60 m; a BEV map of 108 m x 108 m; z in [-10, 10) m, cut
    into nz slabs. jitter: degrees of yaw added to each camera."""
    n, nz = c["cams"], c["nz"]
    a, b = math.radians(c["pitch"]), math.radians(c["roll"])
    pitch = np.array([[1.0, 0.0, 0.0], [0.0, math.cos(a), -math.sin(a)], [0.0, math.sin(a), math.cos(a)]])
    roll = np.array([[math.cos(b), -math.sin(b), 0.0], [math.sin(b), math.cos(b), 0.0], [0.0, 0.0, 1.0]])
    E = np.zeros((n, 12))
    for k in range(n):
        psi = math.radians(360.0 / n * k + (0.0 if jitter is None else float(jitter[k])))
        s, co = math.sin(psi), math.cos(psi)
        R = np.array([[s, 0.0, co], [-co, 0.0, s], [0.0, -1.0, 0.0]]) @ pitch @ roll
        E[k] = np.concatenate([R, np.array([[co], [s], [1.5]])], axis=1).reshape(12)
    f = 70.0 / 88.0 * c["w"]
    return types.SimpleNamespace(
        n_cams=n, feat_h=c["h"], feat_w=c["w"], n_depth=c["bins"], depth_min=1.0, depth_step=59.0 / c["bins"],
        pixel_offset=0.5, nx=c["grid"], ny=c["grid"], x_min=-54.0, y_min=-54.0, cell_x=108.0 / c["grid"],
        cell_y=108.0 / c["grid"], z_min=-10.0, z_cell=20.0 / nz,
        intrinsics=np.tile(np.array([[f, f, c["w"] / 2.0, c["h"] / 2.0]]), (n, 1)), extrinsics=E)


def _case_rig(c, seed):
    if c["use"] != "replan":
        return _rig(c)
    return _rig(c, np.random.default_rng(seed).uniform(-2.0, 2.0, c["cams"]))


def _cells(rig, nz):
    """int64 [N][D][H][W]: the cell of every point, -1 for a dropped one."""
    out = []
    u = np.arange(rig.feat_w) + rig.pixel_offset
    v = (np.arange(rig.feat_h) + rig.pixel_offset)[:, None]
    d = (rig.depth_min + np.arange(rig.n_depth) * rig.depth_step)[:, None, None]
    for n in range(rig.n_cams):
        fx, fy, cx, cy = rig.intrinsics[n]
        E = rig.extrinsics[n]
        x, y, z = d * ((u - cx) / fx), d * ((v - cy) / fy), d
        X = ((E[0] * x + E[1] * y) + E[2] * z) + E[3]
        Y = ((E[4] * x + E[5] * y) + E[6] * z) + E[7]
        Z = ((E[8] * x + E[9] * y) + E[10] * z) + E[11]
        qx = np.floor((X - rig.x_min) / rig.cell_x)
        qy = np.floor((Y - rig.y_min) / rig.cell_y)
        qz = np.floor((Z - rig.z_min) / rig.z_cell)
        keep = (qx >= 0) & (qx < rig.nx) & (qy >= 0) & (qy < rig.ny) & (qz >= 0) & (qz < nz)
        out.append(np.where(keep, (qy * rig.nx + qx) * nz + qz, -1.0).astype(np.int64))
    return np.stack(out)


# ------------------------------------------------------------------ inputs

def _inputs(c, seed):
    """Depth probabilities (a softmax over the bins) and features, and for
    training the gradient that arrives from the layers above."""
    dev = torch.device("cuda")
    g = torch.Generator(device=dev).manual_seed(int(seed))
    shape = (c["batch"], c["cams"], c["bins"], c["h"], c["w"])
    z = torch.randn(shape, generator=g, device=dev)
    if c["depth"] != "normal":
        top = torch.randint(0, c["bins"], (shape[0], shape[1], 1, shape[3], shape[4]), generator=g, device=dev)
        off = torch.arange(c["bins"], device=dev).view(1, 1, -1, 1, 1) - top
    if c["depth"] == "peaked":      # a peak of sigma 3 bins, with noise
        z = 0.5 * z - off.square() / 18.0
    P = torch.softmax(z, dim=2)
    if c["depth"] == "sparse":      # nine pixels in ten sure of their bin
        sure = torch.rand(top.shape, generator=g, device=dev) < 0.9
        P = torch.where(sure, (off == 0).float(), P)
    P = P.to(_TORCH[c["dtype"]])
    F = torch.randn((c["batch"], c["cams"], c["h"], c["w"], c["channels"]), generator=g, device=dev)
    F = F.to(_TORCH[c["dtype"]])
    G = None
    if c["use"] == "train":
        G = torch.randn((c["batch"], c["grid"], c["grid"], c["channels"]), generator=g, device=dev)
    return P, F, G


def prepare(case, seed):
    c = dict(case)
    rig = _case_rig(c, seed)
    P, F, G = _inputs(c, seed)
    s = {"case": c, "P": P, "F": F, "G": G, "rig": rig, "plan": None}
    if c["use"] == "train":
        P.requires_grad_(True)
        F.requires_grad_(True)
    if c["use"] != "replan":
        s["plan"] = bev.SlabPlan.from_rig(rig, c["nz"]) if c["nz"] > 1 else bev.Plan.from_rig(rig)
    return s


def run(s):
    c = s["case"]
    if c["use"] == "train":
        out = bev.bev_pool(s["P"], s["F"], s["plan"])
        dP, dF = torch.autograd.grad(out, (s["P"], s["F"]), s["G"])
        return {"map": out.detach(), "depth_grad": dP, "feature_grad": dF}
    if c["use"] == "replan":
        # the build waits for the stream, so the last plan is no longer in use after it
        plan = bev.Plan.from_rig(s["rig"])
        if s["plan"] is not None:
            s["plan"].close()
        s["plan"] = plan
        return plan.forward(s["P"], s["F"])
    out = s["plan"].forward(s["P"], s["F"], reduce=c["reduce"])
    return bev.to_nchw(out) if c["nchw"] else out


# ------------------------------------------------------------------ work and results

def work(case):
    """Inputs read once, outputs written once (a gradient of the map only in
    the rows that points have); one product and one sum for each kept point
    and channel, and twice that for the two gradients."""
    c = dict(case)
    cells = _cells(_case_rig(c, 1), c["nz"])
    kept = int((cells >= 0).sum())
    rows = int(np.unique(cells[cells >= 0]).size)
    es = 4 if c["dtype"] == "f32" else 2
    points, pixels = cells.size, c["cams"] * c["h"] * c["w"]
    inputs = (points + pixels * c["channels"]) * es
    bev_map = c["nz"] * c["grid"] ** 2 * c["channels"] * 4
    b, f = inputs + bev_map, 2 * kept * c["channels"]
    if c["nchw"]:
        b += 2 * bev_map
    if c["use"] == "train":
        b += 2 * inputs + rows * c["channels"] * 4
        f *= 3
    if c["use"] == "replan":
        b += 2 * points * 4     # the cells of the points, and the points by cell
    return {"bytes": c["batch"] * b, "flops": max(1, c["batch"] * f)}


def tolerance(case):
    if case["use"] == "train" and case["dtype"] != "f32":
        return {"rel": 7e-3, "max": 2e-2}     # gradients rounded to 16 bits: 1.7e-3 from exact
    return {"rel": 1e-6, "max": 4e-5}         # fp32 sums: at most 1.6e-7 from exact (norm)


def exact(case, seed):
    c = dict(case)
    P, F, G = (None if t is None else t.double() for t in _inputs(c, seed))
    cells = _cells(_case_rig(c, seed), c["nz"])
    B, N, D, H, W = P.shape
    C, n_cells = c["channels"], c["nz"] * c["grid"] ** 2
    maxr = c["reduce"] == "max"
    out = torch.full((B, n_cells, C), -math.inf if maxr else 0.0, dtype=torch.float64, device=P.device)
    dP = torch.zeros_like(P) if G is not None else None
    dF = torch.zeros_like(F) if G is not None else None
    count = torch.zeros(n_cells, dtype=torch.float64, device=P.device)
    for n in range(N):
        cell = torch.from_numpy(cells[n].reshape(-1)).to(P.device)
        point = (cell >= 0).nonzero().reshape(-1)
        for at in torch.split(point, 1 << 20):
            to, pix = cell[at], at % (H * W)
            count.index_add_(0, to, torch.ones_like(to, dtype=torch.float64))
            for b in range(B):
                p, f = P[b, n].reshape(-1)[at], F[b, n].reshape(-1, C)[pix]
                v = p[:, None] * f
                if maxr:
                    out[b].index_reduce_(0, to, v, "amax")
                else:
                    out[b].index_add_(0, to, v)
                if G is not None:
                    g = G[b].reshape(-1, C)[to]
                    dP[b, n].view(-1)[at] = (f * g).sum(1)
                    dF[b, n].view(-1, C).index_add_(0, pix, p[:, None] * g)
    if c["reduce"] == "mean":
        out /= count.clamp(min=1.0)[:, None]
    if maxr:
        out[:, count == 0] = 0.0
    out = out.view(B, c["grid"], c["grid"], c["nz"] * C)
    if c["nchw"]:
        out = out.permute(0, 3, 1, 2).contiguous()
    if G is not None:
        return {"map": out, "depth_grad": dP, "feature_grad": dF}
    return out
