"""Grouped launches of the batched form: groups of one and of several instances, instances of one shape
on different schedules, groups split over two streams (calls long enough for the second) and not; work
before and after the call on the caller's own stream; replays of a captured call.  Every instance equals
its own plan bit for bit."""
import pytest

import pfc_inputs as P
from gpu_common import rounded, say, to_dev

pytestmark = pytest.mark.gpu

SHAPES = [(1024, 1024), (512, 512), (512, 512), (64, 64), (64, 64), (64, 64), (1024, 32), (32, 1024), (256, 256), (128, 512)]


@pytest.fixture(scope="module")
def pfc():
    import paper_2603_26818_amd as m

    m.load_library()
    return m


def _setup(pfc, dtype):
    insts = [dict(shape=s, dtype=dtype, r=-0.3 + 0.01 * i, dt=0.25) for i, s in enumerate(SHAPES)]
    psi0 = [to_dev(rounded(P.pfc_initial_field(71 + i, d["shape"], d["r"]), dtype), dtype) for i, d in enumerate(insts)]
    b = pfc.Batch(insts).bind([x.clone() for x in psi0])
    tuning = [list(v) for v in b.get_tuning()]
    tuning[2] = [1, 1, 1]  # 512 x 512: two groups of one shape
    tuning[4] = [0, 1, 0]  # 64 x 64: one of three on another y schedule
    b.set_tuning(tuning)
    plans = [pfc.Plan(d["shape"], dtype=dtype, r=d["r"], dt=0.25) for d in insts]
    for p, t in zip(plans, tuning):
        p.set_tuning(t)
    return b, plans, psi0


def _plan_runs(plans, psi0, steps):
    out = []
    for p, x in zip(plans, psi0):
        x = x.clone()
        s = p.state_init(x)
        for n in steps:
            p.step(x, s, n)
        out.append((x, s))
    return out


def _equal(b, ref, what):
    import torch

    for k, (x, s) in enumerate(ref):
        assert torch.equal(b.psi[k], x) and torch.equal(b.state[k], s), f"{what}: instance {k} {SHAPES[k]} differs"


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_groups_on_the_callers_stream(pfc, dtype):
    import torch

    b, plans, psi0 = _setup(pfc, dtype)
    ref = _plan_runs(plans, psi0, (1, 6))
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    got = []
    with torch.cuda.stream(s):
        for x in b.psi:
            x.zero_()
        for x, y in zip(b.psi, psi0):  # the fields are written just before, and read just after
            x.copy_(y)
        b.state_init()
        b.step(1)
        b.step(6)
        got = [(x.clone(), y.clone()) for x, y in zip(b.psi, b.state)]
        for x in b.psi:
            x.zero_()
    s.synchronize()
    say(f"[batch groups] {dtype}: {len(SHAPES)} instances, {b.grid} workgroups")
    for k, ((x, y), (rx, ry)) in enumerate(zip(got, ref)):
        assert torch.equal(x, rx) and torch.equal(y, ry), f"instance {k} {SHAPES[k]} differs"


def test_captured_call(pfc):
    import torch

    b, plans, psi0 = _setup(pfc, "f32")
    b.state_init()
    b.step(6)  # the batch's stream and events exist before the capture
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        b.step(6)
    for rep in range(3):
        for x, y in zip(b.psi, psi0):
            x.copy_(y)
        b.state_init()
        g.replay()
        torch.cuda.synchronize()
        _equal(b, _plan_runs(plans, psi0, (6,)), f"replay {rep}")
