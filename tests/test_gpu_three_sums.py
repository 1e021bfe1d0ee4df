"""GPU: the 3D adjoint's sum of three fields against the FP64 oracle, at the
column lengths where its column pass takes them side by side (up to 128
points) and one at a time (256)."""
import numpy as np
import pytest

import synth
from oracle import kspace as K

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1603_02329_amd as pat  # noqa: E402


@pytest.mark.parametrize("n", [(16, 16, 16), (64, 16, 32), (32, 16, 128), (16, 16, 256)])
@pytest.mark.parametrize("lossy", [True, False])
def test_adjoint_sum_of_three(n, lossy):
    inst = synth.small_instance(600 + n[2], n=n, nt=7, ns=6, pml=3, lossy=lossy)
    plan = pat.Plan(inst.desc, inst.c0, inst.rho0, inst.alpha0_db, inst.sensors, device="cuda")
    h = np.random.default_rng(n[0]).standard_normal((7, 6)).astype(np.float32)
    img = plan.adjoint(torch.from_numpy(h).cuda()).cpu().numpy().astype(np.float64)
    ref = K.adjoint(K.make_plan(inst.desc, inst.c0, inst.rho0, inst.alpha0_db, inst.sensors), h)
    assert np.linalg.norm(img - ref) <= 1e-5 * np.linalg.norm(ref)
