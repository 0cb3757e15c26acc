"""The block of temporaries that plan builds of one device hand on to each
other: builds of other sizes after one another while a plan lives, builds on two
threads and streams at once, and its return with the device's last plan. What a
plan holds and computes must be the same bits as when it is built alone."""
import gc
import threading

import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu

NAMES = ["tiny", "nuscenes_tilt1", "nuscenes_tilted", "nuscenes"]


def _say(msg):
    print(msg, flush=True)


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.fixture(scope="module")
def pkg(torch_cuda):
    import paper_2205_13542_amd as bp
    bp._binding.load()
    return bp


def _inputs(torch, name):
    w = wl.make(name, seed=1)
    g = torch.Generator(device="cuda").manual_seed(2)
    G = torch.randn((w.batch, w.rig.ny, w.rig.nx, w.channels), generator=g, device="cuda")
    return w.rig, torch.from_numpy(w.P).cuda(), torch.from_numpy(w.F).cuda(), G


def _results(torch, plan, P, F, G, stream):
    """Everything that a plan decides: its association, its sizes, a map and its
    gradients."""
    arrays = plan.export()
    i = plan.info
    sizes = tuple(getattr(i, f) for f, _ in i._fields_)
    with torch.cuda.stream(stream):
        tensors = (plan.forward(P, F), *plan.backward(G, P, F))
    stream.synchronize()
    return arrays, sizes, tensors


def _same(torch, a, b):
    return (all(np.array_equal(x, y) for x, y in zip(a[0], b[0])) and a[1] == b[1]
            and all(torch.equal(x, y) for x, y in zip(a[2], b[2])))


@pytest.fixture(scope="module")
def alone(torch_cuda, pkg):
    """Per name: inputs, and the results of a plan that no other plan precedes."""
    out = {}
    for name in NAMES:
        gc.collect()
        rig, P, F, G = _inputs(torch_cuda, name)
        plan = pkg.Plan.from_rig(rig)
        out[name] = (rig, P, F, G), _results(torch_cuda, plan, P, F, G, torch_cuda.cuda.current_stream())
        plan.close()
    return out


@pytest.mark.parametrize("order", [
    ["tiny", "nuscenes", "tiny", "nuscenes_tilted"],          # a larger build after a smaller one, and back
    ["nuscenes_tilted", "tiny", "nuscenes_tilt1", "tiny"],
])
def test_builds_after_one_another(torch_cuda, pkg, alone, order):
    torch = torch_cuda
    _say(f"[plan memory] {order}")
    plans = []                                                # all live to the end: the block is handed on
    for name in order:
        (rig, P, F, G), ref = alone[name]
        plans.append((name, pkg.Plan.from_rig(rig)))
        assert _same(torch, _results(torch, plans[-1][1], P, F, G, torch.cuda.current_stream()), ref), name
    for name, plan in plans:                                  # and no later build touched an earlier plan
        (_, P, F, G), ref = alone[name]
        assert _same(torch, _results(torch, plan, P, F, G, torch.cuda.current_stream()), ref), name
        plan.close()


def test_builds_on_two_threads(torch_cuda, pkg, alone):
    """Two host threads, each with a stream of its own, build plans of different
    sizes at the same time: neither gets the other's block."""
    torch = torch_cuda
    _say("[plan memory] two threads")
    torch.cuda.synchronize()
    keep = pkg.Plan.from_rig(alone["tiny"][0][0])             # the block stays from build to build
    wrong, start = [], threading.Barrier(2)

    def work(names):
        stream = torch.cuda.Stream()
        start.wait(timeout=60)
        for name in names:
            (rig, P, F, G), ref = alone[name]
            plan = pkg.Plan.from_rig(rig, stream=stream)
            if not _same(torch, _results(torch, plan, P, F, G, stream), ref):
                wrong.append(name)
            plan.close()

    threads = [threading.Thread(target=work, args=(n,)) for n in
               (["nuscenes", "tiny", "nuscenes_tilted"] * 4, ["nuscenes_tilt1", "nuscenes_tilted", "tiny"] * 4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(timeout=100)
    assert not any(t.is_alive() for t in threads) and not wrong
    keep.close()


def test_memory_returns_with_the_last_plan(torch_cuda, pkg, alone):
    """While a plan lives the device keeps a block, of which include/bevpool.h
    states the most; the last plan's close gives it back."""
    torch = torch_cuda
    _say("[plan memory] release")
    gc.collect()
    torch.cuda.synchronize()
    (rig, _, _, _), _ = alone["nuscenes"]
    first = pkg.Plan.from_rig(rig)
    first.close()                                             # (what the runtime itself allocates at first use)
    before = torch.cuda.mem_get_info()[0]
    small = pkg.Plan.from_rig(alone["tiny"][0][0])
    large = pkg.Plan.from_rig(rig)
    large.close()
    held = before - torch.cuda.mem_get_info()[0]
    # 32 MB of temporaries for two million points, and tiny's plan: block and
    # plan together stay below the 64 MB of freed memory that the runtime keeps
    # to hand out again, so that closing a plan before building the next unmaps
    # nothing
    assert (16 << 20) < held <= (40 << 20)
    small.close()
    assert torch.cuda.mem_get_info()[0] >= before - (4 << 20)
