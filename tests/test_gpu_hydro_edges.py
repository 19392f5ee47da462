"""The merged passes of the hydrodynamic step where their dispatch has edges: the smallest grids, rows
with and without padding (three or four work spectra), plane pairs, the longest last axis (the folded
pencils' exchange fills the LDS), y lengths that read their pencil twice, the longest rows, mixed radices
and narrow tiles; two steps, so that the kept spectrum of psi^3 is used, against the oracle."""
import numpy as np
import pytest

import oracle
import pfc_inputs as P
from gpu_common import TOL_STEP, parity_err, rounded, say, to_dev, to_np

pytestmark = pytest.mark.gpu

CASES = [((4, 4), 0), ((2048, 12), 0), ((60, 1024), 0), ((4, 4, 4), 0), ((2048, 4, 8), 0), ((4, 1024, 8), 0), ((4, 2048, 4), 0),
         ((6, 1400, 4), 0), ((4, 4, 2048), 0), ((4, 8, 1400), 0), ((14, 6, 60), 0), ((750, 4, 12), 0), ((1400, 4, 40), 0),
         ((256, 16, 32), 0x30), ((8, 256, 512), 0), ((64, 64, 128), 0)]


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("shape,flags", CASES, ids=str)
def test_hydro_edges(shape, flags, dtype):
    import paper_2603_26818_amd as pfc

    if dtype == "f32" and max(shape) == 4:
        # every mode of a 4-point grid is strongly damped: rounding the oracle's own psi to FP32 already
        # costs 4.7e-5 (2D) and 1.2e-4 (3D) of the mean-removed measure, against a gate of 1e-4
        pytest.skip("fluctuations below FP32's resolution of the field")
    say(f"[hydro edges] shape={shape} flags={flags:#x} dtype={dtype}")
    d = len(shape)
    psi0 = rounded(P.pfc_initial_field(61, shape, -0.3), dtype)
    v0 = np.stack([rounded(P.uniform(610 + j, shape, -0.05, 0.05), dtype) for j in range(d)])
    p, h = oracle.Params(shape, r=-0.3, dt=0.25), oracle.Hydro(0.8, 1.5, 1.1)
    ref = oracle.hydro_step(p, h, psi0, oracle.rfftn(psi0), v0, np.stack([oracle.rfftn(x) for x in v0]), 2)
    plan = pfc.Plan(shape, dtype=dtype, r=-0.3, dt=0.25, flags=flags)
    psi, v = to_dev(psi0, dtype), to_dev(v0, dtype)
    S, V = plan.hydro_state_init(psi, v)
    plan.hydro_step(psi, S, v, V, 2, 0.8, 1.5, 1.1)
    tol = TOL_STEP[dtype]
    assert parity_err(to_np(psi), ref[0]) < tol
    assert parity_err(to_np(plan.state_export(S)), ref[1]) < tol
    for j in range(d):
        assert parity_err(to_np(v[j]), ref[2][j]) < tol
        assert parity_err(to_np(plan.state_export(V[j].contiguous())), ref[3][j]) < tol
