"""FP32 energies right after the state set-up keep their values: the set-up's transforms have schedules of
their own (Dit, InitXPlan, InitAxisPlan), so that the energy of a field, an FP64 sum over their FP32 spectrum,
does not move when the step's schedules change.  The values below are those of the library before mixed
radices took prime-factor DFTs and 2D grids their own schedules; with the ordinary schedules they are off by
1e-9 to 6e-8."""
import numpy as np
import pytest

import pfc_inputs as P
from gpu_common import say, to_dev

pytestmark = pytest.mark.gpu

ENERGY = {
    (6, 10, 12): 172.79154000904086, (14, 12, 28): 1176.9715180006986, (30, 30, 60): 13677.170953423974,
    (60, 60, 60): 54677.74376205374, (150, 60, 300): 683629.3109491552, (30, 150, 60): 68466.32993405442,
    (12, 6, 30): 568.3476362616274, (30, 300): 1459.9113834407665, (150, 60): 1439.2944837918562,
    (60, 120): 1151.5988296786845, (700, 120): 13713.713671580428, (700, 14, 20): 50285.769714821334,
    (1400, 10, 12): 43843.84540712926, (750, 6, 1400): 1673214.445681896, (12, 700, 750): 1613873.4186055704,
    (20, 1400, 24): 171028.67911653075, (64, 64, 256): 265216.7894572501, (128, 128): 2619.708228428379,
    (64, 256): 2618.156985195621, (256, 512): 21411.434254398817, (512, 512): 42821.547629650566,
    (2048, 64): 21563.777457007094,
}


@pytest.mark.parametrize("shape", ENERGY, ids=str)
def test_energy_after_set_up(shape):
    import paper_2603_26818_amd as pfc

    psi = to_dev(P.pfc_initial_field(131, shape, -0.3).astype(np.float32), "f32")
    plan = pfc.Plan(shape, dtype="f32", r=-0.3)
    got = float(plan.energy(psi, plan.state_init(psi))[0])
    say(f"[state energy] {shape}: {got!r}")
    # the same FP32 spectrum: only the order of the FP64 sums may differ (at most 2^22 terms of one sign
    # but for a few: some 1e-13)
    assert abs(got - ENERGY[shape]) <= 1e-12 * abs(ENERGY[shape])
