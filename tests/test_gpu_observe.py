"""Energy, mass mode and state export on row lengths where the passes over modes have edges: rows
shorter than one group of loads, rows that are no multiple of a group, padded rows, plane pairs."""
import pytest

import oracle
import pfc_inputs as P
from gpu_common import TOL_FFT, parity_err, rounded, say, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pfc():
    import paper_2603_26818_amd as m

    m.load_library()
    return m


# n_x / 2 = 2, 6, 15, 30, 375 (padded 3D rows), 64 rows of more than one group of threads, plane pairs
SHAPES = [(4, 4), (6, 12), (4, 6, 30), (14, 12, 60), (4, 6, 750), (4, 2048), (256, 64, 2048)]


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_energy_mass_export(pfc, shape, dtype):
    say(f"[observe] shape={shape} dtype={dtype}")
    psi0 = rounded(P.pfc_initial_field(31, shape, -0.3), dtype)
    plan = pfc.Plan(shape, dtype=dtype, r=-0.3)
    psi = to_dev(psi0, dtype)
    state = plan.state_init(psi)
    half = to_np(plan.state_export(state))
    energy = to_np(plan.energy(psi, state))
    assert parity_err(half, oracle.rfftn(psi0)) < TOL_FFT[dtype]
    # the mass mode: an FP64 sum rounded once (n terms of one sign: n eps is far below 1e-12)
    total = float(psi0.sum())
    assert abs(half.flat[0].real - total) <= abs(total) * (1e-12 if dtype == "f64" else 2.0 ** -23)
    # the energy of the exported spectrum: FP64 sums of at most 2^25 terms in another order
    # (sqrt(n) eps = 1e-12); in FP32 the export has rounded the planes kx = 0 and n_x / 2 once
    # (2^-24 each, squared in the energy)
    p = oracle.Params(shape, r=-0.3)
    F = oracle.energy(p, psi0, half)[0]
    assert abs(energy[0] - F) <= (1e-11 if dtype == "f64" else 1e-6) * abs(F), (energy[0], F)
    assert abs(energy[1] - half.flat[0].real / psi0.size) <= 1e-15
