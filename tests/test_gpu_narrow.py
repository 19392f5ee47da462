"""Narrow tiles of the strided passes and the 2D schedules, which launches with few column tiles take:
grids whose rows are shorter than a narrow tile, end in a partial one, or leave an odd number of them;
every length that has its own 2D schedule; 3D pair tiles of two columns.  Transforms both ways, steps
(the folded column's single round) and one adjoint step, against the oracle."""
import pytest

import oracle
import pfc_inputs as P
from gpu_common import TOL_FFT, TOL_STEP, parity_err, rounded, say, to_dev, to_np

pytestmark = pytest.mark.gpu

SHAPES = [(8, 4), (128, 4), (512, 30), (1024, 20), (2048, 8), (750, 28), (1400, 12), (64, 256), (256, 512), (512, 1024),
          (16, 4, 8), (128, 4, 60), (1024, 6, 20), (512, 2048, 4), (1400, 10, 12), (4, 512, 30), (64, 64, 64)]


@pytest.fixture(scope="module")
def pfc():
    import paper_2603_26818_amd as m

    m.load_library()
    return m


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_few_tiles(pfc, shape, dtype):
    say(f"[narrow] shape={shape} dtype={dtype}")
    p = oracle.Params(shape, r=-0.3, dt=0.5)
    psi0 = rounded(P.pfc_initial_field(51, shape, -0.3), dtype)
    plan = pfc.Plan(shape, dtype=dtype, r=-0.3, dt=0.5)
    half = plan.fft_r2c(to_dev(psi0, dtype))
    ref = oracle.rfftn(psi0)
    assert parity_err(to_np(half), ref) < TOL_FFT[dtype]
    assert parity_err(to_np(plan.fft_c2r(half)), psi0) < 2 * TOL_FFT[dtype]
    psi = to_dev(psi0, dtype)
    state = plan.state_init(psi)
    plan.step(psi, state, 3)
    mid, smid = oracle.step(p, psi0, oracle.state_init(p, psi0), 3)
    assert parity_err(to_np(psi), mid) < TOL_STEP[dtype]
    assert parity_err(to_np(plan.state_export(state)), smid) < TOL_STEP[dtype]
    # one adjoint step from given fields: three transforms, multipliers of a few units
    nxt, _ = oracle.step(p, mid, smid, 1)
    lam = rounded(P.normal(52, shape), dtype)
    a, b = rounded(mid, dtype), rounded(nxt, dtype)
    got, dr = plan.step_backward(to_dev(a, dtype), to_dev(b, dtype), to_dev(lam, dtype))
    want, dr_ref = oracle.step_backward(p, a, b, lam)
    tol = 10 * TOL_FFT[dtype]
    assert parity_err(to_np(got), want) < tol
    # dL/dr is a sum of products: its terms bound its rounding
    scale = 0.5 * float(abs(want).sum()) * float(abs(b).max())
    assert abs(float(dr[0]) - dr_ref) < tol * max(scale, abs(dr_ref))
