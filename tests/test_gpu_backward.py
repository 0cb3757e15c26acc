"""Backward pass on the GPU against the oracle's gradients (same inputs, same
association). Bounds, per element: |dP - ref| <= 1e-4 sqrt(C) (a dot product
of C terms of order one) and |dF - ref| <= 1e-4 sqrt(k), k the pixel's kept
depth bins; dropped points and pixels without kept points exactly 0."""
import dataclasses

import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.fixture(scope="module")
def pkg():
    import paper_2205_13542_amd as bp
    bp._binding.load()
    return bp


def _say(msg):
    print(msg, flush=True)


def _dev(torch, a, dtype):
    t = torch.from_numpy(np.ascontiguousarray(a)).cuda()
    return t.to({"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[dtype]).contiguous()


def _host_values(torch, a, dtype):
    """The values the GPU sees: a rounded to dtype, widened back to fp32."""
    return _dev(torch, a, dtype).float().cpu().numpy()


def _check(torch, pkg, oracle_lib, w, G, dtype="f32", want_depth=True, want_feat=True):
    rig = w.rig
    P = _dev(torch, w.P, dtype)
    F = _dev(torch, w.F, dtype)
    Gd = torch.from_numpy(G).cuda().contiguous()
    plan = pkg.Plan.from_rig(rig)
    gd, gf = plan.backward(Gd, P, F, want_depth=want_depth, want_feat=want_feat)
    torch.cuda.synchronize()
    cop = oracle_lib.cell_map(rig)
    refP, refF = oracle_lib.backward(rig, cop, _host_values(torch, w.P, dtype),
                                     _host_values(torch, w.F, dtype), G)
    C = w.channels
    kept = cop >= 0
    if want_depth:
        got = gd.cpu().numpy().reshape(w.batch, -1)
        ref = refP.reshape(w.batch, -1)
        err = np.abs(got.astype(np.float64) - ref)
        assert (err <= 1e-4 * np.sqrt(C)).all(), f"dP max err {err.max():.3g}"
        assert (got[:, ~kept] == 0).all()
    else:
        assert gd is None
    if want_feat:
        got = gf.cpu().numpy().reshape(w.batch, rig.n_pixels, C)
        ref = refF.reshape(w.batch, rig.n_pixels, C)
        k = kept.reshape(rig.n_cams, rig.n_depth, -1).sum(axis=1).reshape(-1)
        bound = 1e-4 * np.sqrt(np.maximum(k, 1))[None, :, None]
        err = np.abs(got.astype(np.float64) - ref)
        assert (err <= bound).all(), f"dF max err/bound {(err / bound).max():.3g}"
        assert (got[:, k == 0] == 0).all()
    else:
        assert gf is None
    plan.close()
    return gd, gf


def _grad(w, seed):
    rng = np.random.default_rng(seed)
    return rng.standard_normal((w.batch, w.rig.ny, w.rig.nx, w.channels)).astype(np.float32)


@pytest.mark.parametrize("name,seed", [("tiny", 0), ("tiny_identity", 1), ("nuscenes", 2),
                                       ("nuscenes_tilted", 3), ("nuscenes_tilt1", 5)])
def test_backward_matches_oracle(torch_cuda, pkg, oracle_lib, name, seed):
    """Level rig: every combo clean (one gradient row per combo); tilted rig:
    mostly rows with cells of their own."""
    _say(f"[backward] {name} seed={seed}")
    w = wl.make(name, seed=seed)
    _check(torch_cuda, pkg, oracle_lib, w, _grad(w, seed + 10))


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_backward_reduced_precision_inputs(torch_cuda, pkg, oracle_lib, dtype):
    _say(f"[backward] nuscenes {dtype}")
    w = wl.make("nuscenes", seed=4)
    _check(torch_cuda, pkg, oracle_lib, w, _grad(w, 14), dtype=dtype)


@pytest.mark.parametrize("channels", [1, 5, 17, 64, 81, 160, 260])
def test_backward_channel_counts(torch_cuda, pkg, oracle_lib, channels):
    """The per-row kernel (1, 5, 17, 81) and the matrix cores (64, 160, 260), and
    channel slices (81, 160, 260: dP adds the slices' dot products)."""
    _say(f"[backward] nuscenes_tilted C={channels}")
    w = wl.make("nuscenes_tilted", seed=5, channels=channels)
    _check(torch_cuda, pkg, oracle_lib, w, _grad(w, channels))


def test_backward_batch_and_single_outputs(torch_cuda, pkg, oracle_lib):
    _say("[backward] batch 2, one output at a time")
    w = wl.make("nuscenes", seed=6, batch=2)
    G = _grad(w, 16)
    gd, gf = _check(torch_cuda, pkg, oracle_lib, w, G)
    gd1, _ = _check(torch_cuda, pkg, oracle_lib, w, G, want_feat=False)
    _, gf1 = _check(torch_cuda, pkg, oracle_lib, w, G, want_depth=False)
    assert torch_cuda.equal(gd, gd1) and torch_cuda.equal(gf, gf1)


def test_backward_deterministic(torch_cuda, pkg):
    torch = torch_cuda
    w = wl.make("nuscenes_tilted", seed=7)
    plan = pkg.Plan.from_rig(w.rig)
    P, F = _dev(torch, w.P, "f32"), _dev(torch, w.F, "f32")
    G = torch.from_numpy(_grad(w, 17)).cuda()
    a = plan.backward(G, P, F)
    b = plan.backward(G, P, F)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    plan.close()


def test_backward_adjoint_on_gpu(torch_cuda, pkg):
    """<G, forward(P, F)> = <P, dP> = <F, dF> with the GPU's own forward and
    backward, in double on the host."""
    torch = torch_cuda
    w = wl.make("nuscenes", seed=8)
    plan = pkg.Plan.from_rig(w.rig)
    P, F = _dev(torch, w.P, "f32"), _dev(torch, w.F, "f32")
    G = torch.from_numpy(_grad(w, 18)).cuda()
    out = plan.forward(P, F)
    gd, gf = plan.backward(G, P, F)
    torch.cuda.synchronize()
    d = lambda x: x.double().cpu()
    lhs = float((d(G) * d(out)).sum())
    via_p = float((d(P) * d(gd)).sum())
    via_f = float((d(F) * d(gf)).sum())
    scale = float((d(G).abs() * d(out).abs()).sum())
    assert abs(lhs - via_p) <= 1e-5 * scale and abs(lhs - via_f) <= 1e-5 * scale
    plan.close()


def test_autograd_function_matches_oracle(torch_cuda, pkg, oracle_lib):
    """bev_pool under autograd: a scalar loss sum(out * G) gives the oracle's
    gradients for G (and the same tensors as calling backward directly)."""
    torch = torch_cuda
    w = wl.make("nuscenes_tilted", seed=19)
    plan = pkg.Plan.from_rig(w.rig)
    P = torch.from_numpy(w.P).cuda().requires_grad_(True)
    F = torch.from_numpy(w.F).cuda().requires_grad_(True)
    G = torch.from_numpy(_grad(w, 29)).cuda()
    out = pkg.bev_pool(P, F, plan)
    (out * G).sum().backward()
    torch.cuda.synchronize()
    gd, gf = plan.backward(G, P.detach(), F.detach())
    assert torch.equal(P.grad, gd) and torch.equal(F.grad, gf)
    cop = oracle_lib.cell_map(w.rig)
    refP, refF = oracle_lib.backward(w.rig, cop, w.P, w.F, _grad(w, 29))
    assert (np.abs(P.grad.cpu().numpy().astype(np.float64) - refP) <= 1e-4 * np.sqrt(w.channels)).all()
    k = (cop >= 0).reshape(w.rig.n_cams, w.rig.n_depth, -1).sum(axis=1).reshape(-1)
    bound = 1e-4 * np.sqrt(np.maximum(k, 1))[None, :, None]
    got = F.grad.cpu().numpy().reshape(w.batch, w.rig.n_pixels, w.channels)
    assert (np.abs(got - refF.reshape(got.shape)) <= bound).all()
    plan.close()


# ------------------------------------------------------------ the two kernels
#
# A call with a channel count that is a multiple of 4 and aligned rows runs on
# the matrix-core kernel, on every rig whose depth bins do not take many slots
# each (test_backward_by_slots); all other calls run on the per-row kernel.

from test_gpu_parity import RIGS  # noqa: E402


def _rig_workload(rig, channels, seed, batch=1, dtype="f32"):
    P, F = wl.frames(rig, channels, batch, "peaked", seed=seed, dtype=dtype)
    return wl.Workload("c", rig, channels, batch, dtype, P, F)


@pytest.mark.parametrize("channels", [4, 16, 48, 64, 80, 84, 160, 200, 5, 17, 81])
def test_backward_level_channel_counts(torch_cuda, pkg, oracle_lib, channels):
    """Matrix-core launches of 1..8 channel tiles, ragged last tiles (4, 84:
    one slice of 6 tiles; 200: slices of 112 and 88), two slices adding into dP
    (160, 200); 5, 17 and 81 channels take the per-row kernel."""
    _say(f"[backward level] nuscenes C={channels}")
    w = _rig_workload(wl.ring_rig(), channels, seed=channels)
    _check(torch_cuda, pkg, oracle_lib, w, _grad(w, channels + 1))


@pytest.mark.parametrize("name", ["odd", "odd_tilted", "anisotropic", "coarse", "coarse_tilted",
                                  "one_cell", "empty", "tiny_identity", "tall"])
@pytest.mark.parametrize("channels", [8, 20, 7, 63])
def test_backward_edge_rigs(torch_cuda, pkg, oracle_lib, name, channels):
    """Both kernels (8 and 20 channels: matrix cores; 7 and 63: per-row, slices
    of one and four values a lane) on odd sizes (27 columns: the last list has
    three; 13 rows: a partial row block; 37 bins: partial depth steps), an empty
    grid, one cell, cells fed by many combos, and 16,400 rows (no clean combo)."""
    _say(f"[backward edge] {name} C={channels}")
    w = _rig_workload(RIGS[name](), channels, seed=channels + 3)
    _check(torch_cuda, pkg, oracle_lib, w, _grad(w, channels + 7))


def _one_tilted_camera_rig():
    """The ring rig with camera 0 pitched 5 degrees: its depth bins have several
    slots and its combos are not clean, the other cameras' are."""
    base = wl.ring_rig()
    tilted = wl.tilt_rig(base, 5.0, 2.0)
    E = base.extrinsics.copy()
    E[0] = tilted.extrinsics[0]
    return dataclasses.replace(base, extrinsics=E)


@pytest.mark.parametrize("channels", [80, 67])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_backward_mixed_blocks(torch_cuda, pkg, oracle_lib, dtype, channels):
    """Lists of one and of several slots to a bin in one call of the matrix-core
    kernel (80 channels); clean and other combos in one of the per-row kernel."""
    _say(f"[backward mixed] one tilted camera {dtype} C={channels}")
    w = _rig_workload(_one_tilted_camera_rig(), channels, seed=21, batch=2, dtype=dtype)
    _check(torch_cuda, pkg, oracle_lib, w, _grad(w, 22), dtype=dtype)


def test_backward_highres(torch_cuda, pkg, oracle_lib):
    """6 x 236 bins x 64 x 176, C = 128: 8 channel tiles, four columns."""
    _say("[backward highres] C=128")
    w = wl.make("highres", seed=3)
    _check(torch_cuda, pkg, oracle_lib, w, _grad(w, 23))


@pytest.mark.parametrize("tilt,dtype", [(0.0, "f32"), (5.0, "bf16")])
def test_backward_unaligned_features(torch_cuda, pkg, oracle_lib, tilt, dtype):
    """F one element past a 16-byte boundary: the per-row kernel takes the call;
    the result matches the oracle within the bounds."""
    torch = torch_cuda
    _say(f"[backward] unaligned F, tilt={tilt} {dtype}")
    rig = wl.tilt_rig(wl.ring_rig(), tilt, 0.4 * tilt) if tilt else wl.ring_rig()
    w = _rig_workload(rig, 80, seed=24, dtype=dtype)
    plan = pkg.Plan.from_rig(w.rig)
    P, F = _dev(torch, w.P, dtype), _dev(torch, w.F, dtype)
    buf = torch.empty(w.F.size + 1, dtype=F.dtype, device="cuda")
    buf[1:] = F.reshape(-1)
    F_un = buf[1:].view(w.F.shape)
    G = torch.from_numpy(_grad(w, 25)).cuda()
    gd, gf = plan.backward(G, P, F_un)
    torch.cuda.synchronize()
    cop = oracle_lib.cell_map(w.rig)
    refP, refF = oracle_lib.backward(w.rig, cop, _host_values(torch, w.P, dtype), _host_values(torch, w.F, dtype),
                                     _grad(w, 25))
    assert (np.abs(gd.cpu().numpy().astype(np.float64) - refP) <= 1e-4 * np.sqrt(80)).all()
    k = (cop >= 0).reshape(w.rig.n_cams, w.rig.n_depth, -1).sum(axis=1).reshape(-1)
    bound = 1e-4 * np.sqrt(np.maximum(k, 1))[None, :, None]
    got = gf.cpu().numpy().reshape(1, w.rig.n_pixels, 80)
    assert (np.abs(got - refF.reshape(got.shape)) <= bound).all()
    plan.close()


def test_backward_level_deterministic(torch_cuda, pkg):
    torch = torch_cuda
    w = wl.make("nuscenes", seed=26)
    plan = pkg.Plan.from_rig(w.rig)
    P, F = _dev(torch, w.P, "f32"), _dev(torch, w.F, "f32")
    G = torch.from_numpy(_grad(w, 27)).cuda()
    a = plan.backward(G, P, F)
    b = plan.backward(G, P, F)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    plan.close()


def _edge_workload(H, W, D, C, tilt, dtype, seed, batch=2):
    """Two cameras with an H x W map and D bins on a 40 x 40 grid."""
    base = wl.ring_rig()
    intr = base.intrinsics[:2].copy()
    intr[:] = [0.8 * max(W, 4), 0.8 * max(W, 4), W / 2.0, H / 2.0]
    rig = dataclasses.replace(base, n_cams=2, feat_h=H, feat_w=W, n_depth=D, depth_step=59.0 / D, nx=40, ny=40,
                              cell_x=2.7, cell_y=2.7, intrinsics=intr, extrinsics=base.extrinsics[:2].copy())
    if tilt:
        rig = wl.tilt_rig(rig, tilt, 0.4 * tilt)
    return _rig_workload(rig, C, seed=seed, batch=batch, dtype=dtype)


@pytest.mark.parametrize("H,W,D,C,tilt,dtype", [
    (16, 4, 16, 16, 0.0, "f32"),      # one whole tile and step
    (1, 1, 1, 4, 0.0, "f32"),         # the smallest
    (17, 5, 15, 20, 3.0, "f32"),      # one past a tile, one short of a step
    (15, 3, 17, 84, 8.0, "bf16"),     # one short of a tile, many slots per bin
    (33, 8, 70, 112, 8.0, "f16"),     # 7 channel tiles run as 8
    (48, 6, 33, 128, 20.0, "f32"),    # the widest slice, W even and not a multiple of 4
    (31, 12, 40, 132, 5.0, "f32"),    # two slices, the second adds to dP
    (20, 7, 300, 96, 1.0, "bf16"),    # 6 tiles, odd W, lists of several steps per wave
    (16, 4, 1100, 8, 6.0, "f32"),     # more bins than are placed at a time
    # the per-row kernel (8 rows x 4 columns, chunks of 32 bins, slices of at most 80 channels):
    (8, 4, 32, 15, 0.0, "bf16"),      # one whole block and chunk, one value a lane
    (7, 3, 31, 31, 8.0, "f16"),       # one short of each, two values
    (9, 5, 33, 45, 3.0, "bf16"),      # one past each, three values
    (17, 6, 130, 63, 8.0, "f16"),     # a chunk and two bins to a wave, four values
    (12, 7, 40, 79, 1.0, "bf16"),     # five values, the last of one lane short
    (20, 9, 70, 162, 5.0, "f16"),     # three slices of 54, the later ones add to dP
])
def test_backward_tile_edges(torch_cuda, pkg, oracle_lib, H, W, D, C, tilt, dtype):
    """Both kernels at the edges of their tiles, steps, chunks and slices."""
    _say(f"[backward edges] H={H} W={W} D={D} C={C} tilt={tilt} {dtype}")
    w = _edge_workload(H, W, D, C, tilt, dtype, seed=40)
    _check(torch_cuda, pkg, oracle_lib, w, _grad(w, 41), dtype=dtype)


@pytest.mark.parametrize("H,W,D,C,tilt,dtype,batch", [
    (16, 4, 1100, 20, 6.0, "f16", 19),    # 2 tiles: from 40 thousand bins of a tilted rig
    (33, 8, 700, 80, 0.0, "f32", 11),     # 5 tiles: from 90 thousand of a level one
    (33, 8, 1100, 132, 1.0, "f32", 12),   # slices of 5 and 4 tiles, from 150 thousand
    (31, 12, 1100, 96, 5.0, "bf16", 12),  # 6 tiles
    (33, 7, 1100, 68, 1.0, "f32", 12),    # odd W: columns move one by one
])
def test_backward_four_columns(torch_cuda, pkg, oracle_lib, H, W, D, C, tilt, dtype, batch):
    """Enough bins over all frames that a workgroup takes four columns."""
    _say(f"[backward four columns] H={H} W={W} D={D} C={C} tilt={tilt} {dtype} batch={batch}")
    w = _edge_workload(H, W, D, C, tilt, dtype, seed=42, batch=batch)
    _check(torch_cuda, pkg, oracle_lib, w, _grad(w, 43), dtype=dtype)


def _imported_check(torch, pkg, oracle_lib, w, cells, G, dtype):
    """_check's bounds for a plan from a stored cell map."""
    rig, C = w.rig, w.channels
    plan = pkg.Plan.from_cells(cells, rig)
    gd, gf = plan.backward(torch.from_numpy(G).cuda(), _dev(torch, w.P, dtype), _dev(torch, w.F, dtype))
    torch.cuda.synchronize()
    refP, refF = oracle_lib.backward(rig, cells, _host_values(torch, w.P, dtype), _host_values(torch, w.F, dtype), G)
    got = gd.cpu().numpy().reshape(w.batch, -1).astype(np.float64)
    assert (np.abs(got - refP.reshape(got.shape)) <= 1e-4 * np.sqrt(C)).all()
    assert (got[:, cells < 0] == 0).all()
    k = (cells >= 0).reshape(rig.n_cams, rig.n_depth, -1).sum(axis=1).reshape(-1)
    got = gf.cpu().numpy().reshape(w.batch, rig.n_pixels, C).astype(np.float64)
    assert (np.abs(got - refF.reshape(got.shape)) <= 1e-4 * np.sqrt(np.maximum(k, 1))[None, :, None]).all()
    plan.close()


@pytest.mark.parametrize("H,W,D,C,rows,dtype,batch", [
    (33, 8, 40, 80, 1, "f32", 2),      # 16 slots to a bin: the per-row kernel
    (17, 10, 33, 148, 1, "bf16", 3),   # two slices of it, the second adds to dP
    (13, 9, 20, 16, 1, "f16", 2),      # 16 channels; 13 rows in 13 cells
    (33, 8, 40, 88, 1, "f32", 2),      # 88 channels: the matrix cores at any number of slots
    (33, 8, 40, 64, 2, "f32", 2),      # 8 slots to a bin: few workgroups stay on the matrix cores
    (33, 8, 40, 64, 2, "f32", 22),     # 264 lists do not
    (33, 7, 1100, 8, 40, "f32", 4),    # one slot to a bin, odd W, few channels: the per-row kernel
])
def test_backward_by_slots(torch_cuda, pkg, oracle_lib, H, W, D, C, rows, dtype, batch):
    """Both sides of the rule that takes calls of many slots to a bin (cells that
    change every `rows` rows) to the per-row kernel, and odd level maps of few
    channels."""
    _say(f"[backward by slots] H={H} W={W} D={D} C={C} rows={rows} {dtype} batch={batch}")
    w = _edge_workload(H, W, D, C, 0.0, dtype, seed=46, batch=batch)
    rng = np.random.default_rng(47)
    cells = rng.integers(-1, 1600, (2, D, -(-H // rows), W)).repeat(rows, axis=2)[:, :, :H]
    _imported_check(torch_cuda, pkg, oracle_lib, w, np.ascontiguousarray(cells, dtype=np.int32).reshape(-1),
                    _grad(w, 48), dtype)


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("offset", [1, 2])
def test_backward_unaligned_probabilities(torch_cuda, pkg, dtype, offset):
    """P one and two elements past a 16-byte boundary: columns move one by one
    or in pairs, and the gradients are the same bits as with an aligned P."""
    torch = torch_cuda
    _say(f"[backward] P {offset} elements past alignment, {dtype}")
    w = _edge_workload(17, 8, 40, 36, 3.0, dtype, seed=44)
    plan = pkg.Plan.from_rig(w.rig)
    P, F = _dev(torch, w.P, dtype), _dev(torch, w.F, dtype)
    buf = torch.empty(P.numel() + offset, dtype=P.dtype, device="cuda")
    buf[offset:] = P.reshape(-1)
    G = torch.from_numpy(_grad(w, 45)).cuda()
    a = plan.backward(G, P, F)
    b = plan.backward(G, buf[offset:].view(P.shape), F)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    plan.close()


@pytest.mark.parametrize("C,tilt,dtype", [
    (20, 0.0, "f32"), (80, 1.0, "bf16"), (132, 8.0, "f32"),               # matrix cores
    (5, 0.0, "f32"), (67, 0.0, "bf16"), (63, 8.0, "f16"), (90, 1.0, "f32"),   # per-row kernel
])
def test_backward_non_finite_gradients(torch_cuda, pkg, oracle_lib, C, tilt, dtype):
    """Infinities and NaN in the gradients of a few cells reach the pixels with
    a point in such a cell and no others (sums of other pixels stay finite)."""
    _say(f"[backward non-finite] C={C} tilt={tilt} {dtype}")
    torch = torch_cuda
    w = _edge_workload(33, 8, 40, C, tilt, dtype, seed=50)
    rig = w.rig
    cop = oracle_lib.cell_map(rig)
    G = _grad(w, 51)
    cells = np.random.default_rng(52).choice(np.unique(cop[cop >= 0]), 4, replace=False)
    rows = G.reshape(w.batch, -1, C)
    rows[:, cells[0], 0] = np.inf
    rows[0, cells[1], C - 1] = -np.inf
    rows[1, cells[2], :] = np.nan
    rows[0, cells[3], C // 2] = np.inf
    plan = pkg.Plan.from_rig(rig)
    gd, gf = plan.backward(torch.from_numpy(G).cuda(), _dev(torch, w.P, dtype), _dev(torch, w.F, dtype))
    torch.cuda.synchronize()
    with np.errstate(all="ignore"):
        refP, refF = oracle_lib.backward(rig, cop, _host_values(torch, w.P, dtype), _host_values(torch, w.F, dtype), G)
    k = (cop >= 0).reshape(rig.n_cams, rig.n_depth, -1).sum(axis=1).reshape(-1)
    for got, ref, bound in ((gd, refP, 1e-4 * np.sqrt(C)),
                            (gf, refF, 1e-4 * np.sqrt(np.maximum(k, 1))[None, :, None])):
        got = got.cpu().numpy().astype(np.float64).reshape((w.batch, -1) if got is gd else (w.batch, rig.n_pixels, C))
        ref = ref.reshape(got.shape)
        fin = np.isfinite(ref)
        assert not fin.all()
        assert (np.isfinite(got) == fin).all()
        assert (np.where(fin, np.abs(got - np.where(fin, ref, 0.0)), 0.0) <= bound).all()
    plan.close()


def _call_us(torch, fn, calls=20):
    """Median over five of the GPU's time for a call among others."""
    fn()
    times = []
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(calls):
            fn()
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b) * 1e3 / calls)
    return sorted(times)[2]


@pytest.mark.parametrize("C", [80, 128, 67])
def test_backward_infinite_gradient(torch_cuda, pkg, C):
    """A gradient that is infinite everywhere (a loss scale too large) reaches
    every kept point and every pixel with one, and costs one walk over the points
    of each pixel: measured 3.5 times a finite one's time, asserted at most 12 (a
    walk for each value took 33)."""
    torch = torch_cuda
    w = _rig_workload(wl.ring_rig(), C, seed=60)
    plan = pkg.Plan.from_rig(w.rig)
    P, F = _dev(torch, w.P, "f32"), _dev(torch, w.F, "f32")
    G = torch.from_numpy(_grad(w, 61)).cuda()
    inf = torch.full_like(G, float("inf"))
    gd, gf = plan.backward(inf, P, F)
    kept = (torch.from_numpy(plan.export()[0]) >= 0).cuda().reshape(w.rig.n_cams, w.rig.n_depth, -1)
    assert torch.equal(~gd.reshape(kept.shape).isfinite(), kept)
    pixels = kept.any(1).reshape(-1)
    assert torch.equal(~gf.reshape(-1, C).isfinite(), pixels[:, None].expand(-1, C))
    assert (gf.reshape(-1, C)[~pixels] == 0).all()
    finite, infinite = (_call_us(torch, lambda: plan.backward(g, P, F)) for g in (G, inf))
    _say(f"[backward infinite] C={C}: finite {finite:.1f} us, infinite {infinite:.1f} us")
    assert infinite <= 12.0 * finite
    plan.close()


@pytest.mark.parametrize("width,backward", [((1 << 25) + 4, True), ((1 << 26) + 4, False)])
def test_plan_without_backward_lists(torch_cuda, pkg, width, backward):
    """One row, one bin and so many columns that the backward lists (four columns
    each) would not fit a grid of two workgroups, or one, for each: the plan has
    none, the forward and, where the per-row kernel's grid fits, the backward work.
    One point in 64 is kept; each pixel has one point, so gradients are exact."""
    torch = torch_cuda
    _say(f"[lists] {width} columns")
    base = wl.ring_rig()
    rig = dataclasses.replace(base, n_cams=1, feat_h=1, feat_w=width, n_depth=1, nx=1024, ny=1024,
                              intrinsics=base.intrinsics[:1].copy(), extrinsics=base.extrinsics[:1].copy())
    C = 4 if backward else 1
    rng = np.random.default_rng(70)
    at = np.sort(rng.choice(width // 64, width // 128, replace=False).astype(np.int64) * 64 + 63)
    cells = np.full(width, -1, np.int32)
    cells[at] = rng.integers(0, 1 << 20, at.size)
    plan = pkg.Plan.from_cells(cells, rig)
    assert plan.info.n_kept == at.size
    at, to = torch.from_numpy(at).cuda(), torch.from_numpy(cells[at].astype(np.int64)).cuda()
    g = torch.Generator(device="cuda").manual_seed(71)
    P = torch.rand((1, 1, 1, 1, width), generator=g, device="cuda")
    F = torch.randn((1, 1, 1, width, C), generator=g, device="cuda")
    out = plan.forward(P, F).reshape(-1, C)
    p, f = P.reshape(-1)[at].double(), F.reshape(-1, C)[at].double()
    ref = torch.zeros((1 << 20, C), dtype=torch.float64, device="cuda").index_add_(0, to, p[:, None] * f)
    assert float((out - ref).abs().max()) <= 1e-4
    if backward:
        G = torch.randn((1, 1024, 1024, C), generator=g, device="cuda")
        gd, gf = plan.backward(G, P, F)
        rows = G.reshape(-1, C)[to]
        assert torch.equal(gf.reshape(-1, C)[at], P.reshape(-1)[at][:, None] * rows)
        ref = (f * rows.double()).sum(1)
        assert float((gd.reshape(-1)[at] - ref).abs().max()) <= 1e-4 * C ** 0.5
        assert int((gd != 0).sum()) <= at.numel() and int((gf != 0).sum()) <= at.numel() * C
    plan.close()
