"""The rules of the resident solves on the host, and the solves that change
sides by them: a single time step over all dies, alone and as a segment."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_rules_on_the_host(tmp_path):
    exe = str(tmp_path / "solve_rule_check")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-fsanitize=address,undefined",
                        os.path.join(ROOT, "tests", "solve_rule_check.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "all checks passed" in r.stdout, r.stdout[-2000:]


@pytest.mark.gpu
@pytest.mark.parametrize("lossy", [True, False])
@pytest.mark.parametrize("n", [(512, 256), (64, 64)])
def test_single_steps_bitwise(n, lossy):
    """Segments of one step (launches over all dies, resident on one) between
    longer ones, and the shortest solves."""
    torch = pytest.importorskip("torch")
    import paper_1603_02329_amd as pat
    i = synth.small_instance(77, n=n, nt=11, ns=9, pml=6, lossy=lossy)
    plan = pat.Plan(i.desc, i.c0, i.rho0, i.alpha0_db, i.sensors, device="cuda")
    p0 = torch.from_numpy(i.p0).cuda()
    ref = plan.forward(p0).clone()
    d = torch.zeros_like(ref)
    state = torch.empty(plan.state_bytes, dtype=torch.uint8, device="cuda")
    for a, b in ((0, 2), (2, 3), (3, 7), (7, 8), (8, 9), (9, 11)):
        plan.forward_range(p0 if a == 0 else None, d, a, b, state)
    assert torch.equal(d, ref)
    s = synth.small_instance(78, n=n, nt=2, ns=9, pml=6, lossy=lossy)
    short = pat.Plan(s.desc, s.c0, s.rho0, s.alpha0_db, s.sensors, device="cuda")
    h = torch.from_numpy(np.random.default_rng(1).standard_normal((2, 9)).astype(np.float32)).cuda()
    got = short.forward(p0).clone(), short.adjoint(h).clone()
    pat.timing_begin(0, 0, 7)
    try:
        want = short.forward(p0).clone(), short.adjoint(h).clone()
    finally:
        torch.cuda.synchronize()
        pat.timing_end()
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
