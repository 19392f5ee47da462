"""Batches of many shapes, whose small groups share their launches by class of y lengths: every shape the
batched form takes, several instances of some, groups on launches of their own among them (large ones, tuned
ones).  Every instance equals its own plan bit for bit, and the number of launches does not grow with the
number of shapes.  A step captured as the first call of a batch."""
import ctypes
import itertools

import pytest

import pfc_inputs as P
from gpu_common import rounded, say, to_dev

pytestmark = pytest.mark.gpu

LENGTHS = [32, 64, 128, 256, 512, 1024]
ALL = list(itertools.product(LENGTHS, LENGTHS))
CASES = {
    "all shapes": (ALL, {}),
    # several instances, out of order; 5 of 256 x 512 fill the chip by themselves; two tuned instances
    "mixed": ([(32, 32), (1024, 64), (256, 512), (64, 1024), (256, 512), (32, 32), (512, 32), (256, 512), (32, 256), (1024, 64),
               (512, 512), (256, 512), (128, 32), (32, 32), (256, 512), (1024, 1024), (64, 64), (128, 32)], {6: [0, 1, 0], 13: [1, 0, 1]}),
    "all tuned": (ALL, {i: [1, 1, 1] for i in range(len(ALL))}),
    "tunings mixed": (ALL + ALL[::5], {i: [i % 2, i // 2 % 2, i // 4 % 2] for i in range(len(ALL) + 8)}),
    "one class": ([(64, 128), (128, 64), (256, 32)], {}),
    "one length": ([(512, 32), (512, 64), (512, 64)], {}),
}


def _setup(shapes, tuned, dtype):
    import paper_2603_26818_amd as pfc

    insts = [dict(shape=s, dtype=dtype, r=-0.3 + 0.002 * i, dt=0.25) for i, s in enumerate(shapes)]
    psi0 = [to_dev(rounded(P.pfc_initial_field(400 + i, d["shape"], d["r"]), dtype), dtype) for i, d in enumerate(insts)]
    b = pfc.Batch(insts).bind([x.clone() for x in psi0])
    tuning = [tuned.get(i, list(v)) for i, v in enumerate(b.get_tuning())]
    b.set_tuning(tuning)
    return pfc, b, psi0, insts, tuning


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("case", CASES)
def test_units_equal_own_plans(case, dtype):
    import torch

    shapes, tuned = CASES[case]
    say(f"[batch units] {case}: {len(shapes)} instances, {dtype}")
    pfc, b, psi0, insts, tuning = _setup(shapes, tuned, dtype)
    b.state_init()
    b.step(1)
    b.step(4)
    for k, (d, x, t) in enumerate(zip(insts, psi0, tuning)):
        p = pfc.Plan(d["shape"], dtype=dtype, r=d["r"], dt=0.25)
        p.set_tuning(t)
        s = p.state_init(x)
        p.step(x, s, 1)
        p.step(x, s, 4)
        assert torch.equal(b.psi[k], x) and torch.equal(b.state[k], s), f"instance {k} {shapes[k]} differs"


# three passes of at most a class each for y up to 256, 512 and 1024 or, on tuned schedules, of a launch per
# length, and of a few groups that fill the chip by themselves; one launch per shape and pass would be 108
@pytest.mark.parametrize("tuning,most", [([0, 0, 0], 18), ([1, 1, 1], 24)], ids=str)
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_launches_of_many_shapes(dtype, tuning, most):
    import torch

    pfc, b, _, _, _ = _setup(ALL, {i: tuning for i in range(len(ALL))}, dtype)
    b.state_init()
    b.step(1)
    torch.cuda.synchronize()
    lib = pfc.load_library()  # (also finds the HIP runtime's entry points)
    s = torch.cuda.Stream()
    graph, n = ctypes.c_void_p(), ctypes.c_size_t(0)
    with torch.cuda.stream(s):
        assert lib.hipStreamBeginCapture(ctypes.c_void_p(s.cuda_stream), ctypes.c_int(2)) == 0
        b.step(1)
        assert lib.hipStreamEndCapture(ctypes.c_void_p(s.cuda_stream), ctypes.byref(graph)) == 0
    assert lib.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    assert lib.hipGraphDestroy(graph) == 0
    say(f"[batch units] {len(ALL)} shapes, one step: {n.value} launches")
    assert n.value <= most


def test_first_step_under_capture():
    import torch

    shapes = [(1024, 1024), (512, 512), (512, 512), (64, 64), (32, 256)]  # 6 steps take the second stream
    _, b, psi0, _, _ = _setup(shapes, {}, "f32")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        b.step(6)
    got = []
    for rep in range(3):
        for x, y in zip(b.psi, psi0):
            x.copy_(y)
        b.state_init()
        g.replay() if rep < 2 else b.step(6)  # the eager call last
        torch.cuda.synchronize()
        got.append([x.clone() for x in b.psi + b.state])
    for rep in range(2):
        assert all(torch.equal(x, y) for x, y in zip(got[rep], got[2])), f"replay {rep} differs from the eager call"
