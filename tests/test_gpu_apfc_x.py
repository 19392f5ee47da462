"""The fused x pass of the amplitude step (inverse rows, nonlinearity, forward rows in one kernel) and the
narrow tiles of its last axis: every row length the fused pass takes, from one field group per wavefront
to the most fields a workgroup holds, ragged row counts, and neighbours that keep the separate passes
(more fields, longer or mixed-radix rows, FP64 rows past the LDS).  Three steps in one call against the
oracle, and bit for bit against three calls of one step."""
import numpy as np
import pytest

import oracle
import pfc_inputs as P
from gpu_common import TOL_STEP, parity_err, say

pytestmark = pytest.mark.gpu

CASES = [("triangular", (6, 16)), ("square", (30, 32)), ("triangular2", (10, 64)), ("bcc", (4, 6, 128)), ("fcc2", (8, 4, 256)),
         ("triangular", (14, 512)), ("square", (8, 1024)), ("triangular", (1024, 64)), ("triangular2", (512, 256)),
         ("triangular", (8, 2048)), ("bcc", (4, 4, 60)), ("triangular30", (8, 16)), ("bcc", (64, 64, 16))]


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("lattice,shape", CASES, ids=str)
def test_fused_x(lattice, shape, dtype):
    import torch

    import paper_2603_26818_amd as pfc

    k = P.lattice_vectors(lattice)
    many = len(k) > 8
    say(f"[apfc x] {lattice} ({len(k)}) shape={shape} dtype={dtype}")
    kw = dict(dB=-0.15, Bx=1.0, t=0.3, v=1.0, dt=0.1 if many else 0.5)
    eta0 = P.amplitude_fields(96, len(k), shape, *((0.01, 0.005) if many else (0.1, 0.05)))
    ct = torch.complex64 if dtype == "f32" else torch.complex128
    dev = torch.from_numpy(np.ascontiguousarray(eta0)).to("cuda:0").to(ct)
    eta0 = dev.cpu().numpy().astype(np.complex128)
    obj = pfc.Apfc(shape, k, dtype=dtype, **kw)
    a, b = dev.clone(), dev.clone()
    A, B = obj.state_init(a), obj.state_init(b)
    obj.step(a, A, 3)
    for _ in range(3):
        obj.step(b, B, 1)
    torch.cuda.synchronize()
    assert torch.equal(a, b) and torch.equal(A, B), "one call of three steps differs from three calls"
    o = oracle.Apfc(shape, k, **kw)
    ref, sref = oracle.apfc_step(o, eta0, oracle.apfc_state_init(o, eta0), 3)
    assert parity_err(a.cpu().numpy().astype(np.complex128), ref) < TOL_STEP[dtype]
    assert parity_err(A.cpu().numpy().astype(np.complex128), sref) < TOL_STEP[dtype]
