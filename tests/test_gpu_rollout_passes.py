"""pfc_step_trajectory and pfc_rollout_backward against the single steps they stand for: the same fields and
adjoints bit for bit, the same dL/dr up to the order of its FP64 sums; with and without the fused x passes
(1024-point rows, tuned x schedules), 2D and 3D, mixed radices, plane pairs, one step and several."""
import pytest

import pfc_inputs as P
from gpu_common import rounded, say, to_dev

pytestmark = pytest.mark.gpu

CASES = [((64, 128), 0, 5), ((512, 512), 0, 3), ((8, 2048), 0, 3), ((60, 300), 0, 4), ((32, 16, 64), 0, 4), ((12, 10, 60), 0, 3),
         ((256, 16, 32), 0x30, 2), ((64, 64), 0, 1), ((128, 256), "tuned", 4)]


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("shape,flags,nsteps", CASES, ids=str)
def test_trajectory_and_its_adjoint(shape, flags, nsteps, dtype):
    import torch

    import paper_2603_26818_amd as pfc

    say(f"[rollout passes] shape={shape} flags={flags} nsteps={nsteps} dtype={dtype}")
    plan = pfc.Plan(shape, dtype=dtype, r=-0.3, dt=0.5, flags=0 if flags == "tuned" else flags)
    if flags == "tuned":
        plan.set_tuning([1] + [0] * (len(plan.get_tuning()) - 1))
    psi0 = to_dev(rounded(P.pfc_initial_field(81, shape, -0.3), dtype), dtype)
    zero = torch.zeros_like(plan.empty_state())  # padding of the rows, which no kernel writes
    state = plan.state_init(psi0, zero.clone())
    keep = psi0.clone()
    traj = plan.step_trajectory(psi0, state, nsteps)
    x, s = psi0.clone(), plan.state_init(psi0, zero.clone())
    fields = [psi0]
    for n in range(nsteps):
        plan.step(x, s, 1)
        fields.append(x.clone())
        assert torch.equal(traj[n], x), f"field after step {n + 1} differs"
    assert torch.equal(state, s) and torch.equal(psi0, keep)
    lam = to_dev(rounded(P.normal(82, shape), dtype), dtype)
    a, da = lam.clone(), torch.full((1,), 2.0, dtype=torch.float64, device=lam.device)
    plan.rollout_backward(psi0, traj, a, da)
    b, db, size = lam.clone(), torch.zeros(1, dtype=torch.float64, device=lam.device), 0.0
    for n in range(nsteps - 1, -1, -1):
        one = torch.zeros(1, dtype=torch.float64, device=lam.device)
        plan.step_backward(fields[n], fields[n + 1], b, lambda_n=b, dLdr=one)
        db += one
        size += float(b.double().norm() * fields[n + 1].double().norm())
    assert torch.equal(a, b), "adjoint differs from the single steps"
    # FP64 sums in another order: at most n eps of the sum of magnitudes (n <= 2^18 terms: 6e-11)
    assert abs(float(da[0]) - 2.0 - float(db[0])) <= 1e-10 * (size + 2.0)
