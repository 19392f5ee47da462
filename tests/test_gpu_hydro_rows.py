"""Rows whose threads do not divide a wavefront (x = 1500: 750 packed points over 25 threads, two rows and
50 threads per workgroup) in the x passes of the hydrodynamic step: even and odd numbers of workgroups, 2D
and 3D.  The shortest rows, whose last-axis tiles are half a row and its mirror's, at row counts with and
without a last incomplete group.  Two steps, against the oracle."""
import numpy as np
import pytest

import oracle
import pfc_inputs as P
from gpu_common import TOL_STEP, parity_err, rounded, say, to_dev, to_np

pytestmark = pytest.mark.gpu


def _run(shape, dtype):
    """(psi, its spectrum, v, their spectra) after two steps, of the library and of the oracle."""
    import paper_2603_26818_amd as pfc

    say(f"[hydro rows] shape={shape} dtype={dtype}")
    d = len(shape)
    psi0 = rounded(P.pfc_initial_field(62, shape, -0.3), dtype)
    v0 = np.stack([rounded(P.uniform(620 + j, shape, -0.05, 0.05), dtype) for j in range(d)])
    p, h = oracle.Params(shape, r=-0.3, dt=0.25), oracle.Hydro(0.8, 1.5, 1.1)
    ref = oracle.hydro_step(p, h, psi0, oracle.rfftn(psi0), v0, np.stack([oracle.rfftn(x) for x in v0]), 2)
    plan = pfc.Plan(shape, dtype=dtype, r=-0.3, dt=0.25)
    psi, v = to_dev(psi0, dtype), to_dev(v0, dtype)
    S, V = plan.hydro_state_init(psi, v)
    plan.hydro_step(psi, S, v, V, 2, 0.8, 1.5, 1.1)
    got = [to_np(psi), to_np(plan.state_export(S))]
    want = [ref[0], ref[1]]
    for j in range(d):
        got += [to_np(v[j]), to_np(plan.state_export(V[j].contiguous()))]
        want += [ref[2][j], ref[3][j]]
    return got, want


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("shape", [(4, 1500), (6, 1500), (64, 1500), (4, 6, 1500), (6, 10, 1500), (16, 4, 1500)], ids=str)
def test_rows_of_750(shape, dtype):
    for a, b in zip(*_run(shape, dtype)):
        assert parity_err(a, b) < TOL_STEP[dtype]


SHORT = [(700, 20, 4), (750, 14, 8), (1400, 6, 8), (1400, 12, 4), (1024, 20, 8), (2048, 6, 4), (256, 60, 8), (128, 150, 4),
         (512, 30, 8), (60, 128, 4), (64, 256, 8)]


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("shape", SHORT, ids=str)
def test_short_rows(shape, dtype):
    for a, b in zip(*_run(shape, dtype)):
        assert parity_err(a, b) < TOL_STEP[dtype]
