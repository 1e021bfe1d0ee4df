"""How the proximal map is cut into launches: the rule by itself on the host,
and thin images on either side of it against the two launches an iteration
(which run where the result overwrites the lower bound), bitwise."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_rule_on_the_host(tmp_path):
    exe = str(tmp_path / "prox_plan_check")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-fsanitize=address,undefined",
                        os.path.join(ROOT, "tests", "prox_plan_check.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "all checks passed" in r.stdout, r.stdout[-2000:]


@pytest.mark.gpu
@pytest.mark.parametrize("n_iter", [1, 13, 35])
@pytest.mark.parametrize("shape", [(200000, 1), (60000, 8), (1, 60000), (3, 20000)])
def test_thin_images_bitwise(shape, n_iter):
    torch = pytest.importorskip("torch")
    import paper_1603_02329_amd as pat
    rng = np.random.default_rng(n_iter)
    z = torch.from_numpy(rng.standard_normal(shape).astype(np.float32)).cuda()
    lower = torch.from_numpy((0.3 * rng.standard_normal(shape)).astype(np.float32)).cuda()
    both = lower.clone()
    pat.tv_prox(z, 0.3, n_iter, lower=both, out=both)
    assert torch.equal(pat.tv_prox(z, 0.3, n_iter, lower=lower), both)
    small = torch.from_numpy(rng.standard_normal((40, 50)).astype(np.float32)).cuda()
    got = pat.tv_prox_batched([z, small], [0.3, 0.2], n_iter, lowers=[lower, None])
    assert torch.equal(got[0], both) and torch.equal(got[1], pat.tv_prox(small, 0.2, n_iter))


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(1, 1), (1, 3), (4, 1), (7, 9)])
def test_step_beyond_float_bitwise(shape):
    """lambda > 0 whose step 1 / (8 lambda) is infinite in float32: a point
    without neighbours keeps max(z, lower)."""
    torch = pytest.importorskip("torch")
    import paper_1603_02329_amd as pat
    z = torch.linspace(0.25, 2.0, shape[0] * shape[1]).reshape(shape).cuda()
    zero = torch.zeros_like(z)
    pat.tv_prox(z, 1e-40, 3, lower=zero, out=zero)
    if z.numel() == 1:
        assert torch.equal(zero, z)
    got = pat.tv_prox(z, 1e-40, 3)
    assert torch.equal(got.view(torch.int32), zero.view(torch.int32))
    assert torch.equal(pat.tv_prox_batched([z], [1e-40], 3)[0].view(torch.int32), zero.view(torch.int32))


@pytest.mark.gpu
def test_result_in_the_workspace_bitwise():
    """The result may lie where the workspace's dual iterate does: nothing
    reads that once the result is written."""
    torch = pytest.importorskip("torch")
    import paper_1603_02329_amd as pat
    shape = (120, 200)
    z = torch.from_numpy(np.random.default_rng(3).standard_normal(shape).astype(np.float32)).cuda()
    for n_iter in (5, 20, 40):
        ref = pat.tv_prox(z, 0.3, n_iter)
        work = torch.empty(5 * z.numel(), device="cuda")
        out = work[:z.numel()].view(shape)
        pat.tv_prox(z, 0.3, n_iter, out=out, work=work.view(torch.uint8))
        assert torch.equal(out, ref)
        pat.tv_prox_batched([z], [0.3], n_iter, outs=[out], works=[work.view(torch.uint8)])
        assert torch.equal(out, ref)
