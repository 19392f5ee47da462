"""The smallest FP32 grids of the hydrodynamic step, in the measures that rounding of the field does not
swamp, against the oracle."""
import numpy as np
import pytest

import oracle
import pfc_inputs as P
from gpu_common import parity_errs, rounded, say, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(4, 4), (4, 4, 4)], ids=str)
def test_smallest_f32(shape):
    import paper_2603_26818_amd as pfc

    say(f"[hydro smallest] shape={shape}")
    d = len(shape)
    psi0 = rounded(P.pfc_initial_field(62, shape, -0.3), "f32")
    v0 = np.stack([rounded(P.uniform(620 + j, shape, -0.05, 0.05), "f32") for j in range(d)])
    p, h = oracle.Params(shape, r=-0.3, dt=0.25), oracle.Hydro(0.8, 1.5, 1.1)
    ref = oracle.hydro_step(p, h, psi0, oracle.rfftn(psi0), v0, np.stack([oracle.rfftn(x) for x in v0]), 2)
    plan = pfc.Plan(shape, dtype="f32", r=-0.3, dt=0.25)
    psi, v = to_dev(psi0, "f32"), to_dev(v0, "f32")
    S, V = plan.hydro_state_init(psi, v)
    plan.hydro_step(psi, S, v, V, 2, 0.8, 1.5, 1.1)
    pairs = [(psi, ref[0]), (plan.state_export(S), ref[1])]
    for j in range(d):
        pairs += [(v[j], ref[2][j]), (plan.state_export(V[j].contiguous()), ref[3][j])]
    # Two steps are eight transforms and four updates of at most 64 values: some 50 roundings of 6e-8 on
    # the way to each output, which the update multiplies by at most a few (its modes are damped).
    # The mean-removed measure is left out: rounding psi itself costs up to 1.2e-4 of it here.
    for a, b in pairs:
        plain, _, maxabs = parity_errs(to_np(a), b)
        assert plain < 1e-5 and maxabs < 1e-5, (plain, maxabs)
