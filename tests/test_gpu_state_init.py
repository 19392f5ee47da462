"""The state set-up's own FP32 schedules (mixed radices decimated in time, their stage tables; 128- and
256-point rows, 2D pencils): every such length on every axis, full and narrow tiles, against the oracle;
and the batched set-up equals the single plan's bit for bit."""
import pytest

import oracle
import pfc_inputs as P
from gpu_common import TOL_FFT, parity_err, rounded, say, to_dev, to_np

pytestmark = pytest.mark.gpu

SHAPES = [(6, 10, 12), (14, 12, 28), (12, 6, 30), (20, 60, 40), (30, 150, 60), (60, 30, 120), (150, 20, 300), (150, 30, 24),
          (700, 14, 20), (1400, 10, 12), (750, 6, 1400), (12, 700, 750), (10, 750, 1500 // 125), (20, 1400, 24), (30, 300),
          (150, 60), (700, 120), (64, 256), (256, 512), (2048, 64), (64, 64, 256), (150, 150, 150 * 2)]


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_state_init(shape, dtype):
    import paper_2603_26818_amd as pfc

    say(f"[state init] shape={shape} dtype={dtype}")
    psi0 = rounded(P.normal(91, shape), dtype)
    plan = pfc.Plan(shape, dtype=dtype, r=-0.3)
    half = plan.state_export(plan.state_init(to_dev(psi0, dtype)))
    assert parity_err(to_np(half), oracle.rfftn(psi0)) < TOL_FFT[dtype]


def test_batched_state_init():
    import torch

    import paper_2603_26818_amd as pfc

    shapes = [(128, 256), (256, 512), (512, 128), (1024, 1024)]
    psi = [to_dev(rounded(P.pfc_initial_field(92 + i, s, -0.3), "f32"), "f32") for i, s in enumerate(shapes)]
    b = pfc.Batch([dict(shape=s, dtype="f32", r=-0.3, dt=0.25) for s in shapes]).bind(psi)
    b.state_init()
    for k, s in enumerate(shapes):
        want = pfc.Plan(s, dtype="f32", r=-0.3, dt=0.25).state_init(psi[k])
        assert torch.equal(b.state[k], want), s
