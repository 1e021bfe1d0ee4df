"""GPU: a resident solve whose workgroups give up waiting for each other (here
after one poll, set from the host; every workgroup still ends normally) shows:
its results are NaN throughout, the plan says so once, the solver raises, and
instances of a batch's queue that were never begun are reported like the rest."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1603_02329_amd as pat  # noqa: E402
from paper_1603_02329_amd import solver  # noqa: E402

DEV = "cuda"


def _case(seed, **kw):
    i = synth.small_instance(seed, **kw)
    plan = pat.Plan(i.desc, i.c0, i.rho0, i.alpha0_db, i.sensors, device=DEV)
    rng = np.random.default_rng(seed)
    h = torch.from_numpy(rng.standard_normal((i.desc.nt, i.ns)).astype(np.float32)).to(DEV)
    return plan, torch.from_numpy(i.p0).to(DEV), h


def _raises_once(plan):
    with pytest.raises(pat.PatError) as e:
        plan.sync()
    assert e.value.code == pat.PAT_EHIP
    plan.sync()


@pytest.mark.parametrize("lossy", [True, False])
@pytest.mark.parametrize("n", [(64, 64), (256, 256), (512, 512)])
def test_given_up_solve_is_nan_and_reported(n, lossy):
    plan, p0, h = _case(11, n=n, nt=9, ns=7, pml=6, lossy=lossy)
    ref_d, ref_i = plan.forward(p0).clone(), plan.adjoint(h).clone()
    plan.sync()
    plan.wait_limit(1)
    assert torch.isnan(plan.forward(p0)).all()
    _raises_once(plan)
    assert torch.isnan(plan.adjoint(h)).all()
    with pytest.raises(pat.PatError):
        pat.solves_check([plan])
    pat.solves_check([plan])
    plan.wait_limit(0)
    assert torch.equal(plan.forward(p0), ref_d) and torch.equal(plan.adjoint(h), ref_i)
    plan.sync()


@pytest.mark.parametrize("n", [(64, 64), (256, 128), (512, 256)])
def test_all_or_nothing_at_any_limit(n):
    """Whichever wait runs out (joining, claiming, a barrier): a result is
    either whole or NaN throughout, and the latter is reported."""
    plan, p0, h = _case(14, n=n, nt=25, ns=9, pml=6, lossy=True)
    ref = plan.forward(p0).clone(), plan.adjoint(h).clone()
    for polls in (2, 4, 8, 12, 16, 24, 32, 64, 128):
        plan.wait_limit(polls)
        for call, arg, want in ((plan.forward, p0, ref[0]), (plan.adjoint, h, ref[1])):
            out = call(arg)
            whole = torch.equal(out, want)
            assert whole or torch.isnan(out).all(), polls
            if whole:
                plan.sync()
            else:
                _raises_once(plan)


def test_given_up_segment_spoils_the_later_ones():
    plan, p0, _ = _case(12, n=(128, 64), nt=12, ns=9, pml=6, lossy=True)
    ref = plan.forward(p0).clone()
    d = torch.zeros_like(ref)
    state = torch.empty(plan.state_bytes, dtype=torch.uint8, device=DEV)
    plan.forward_range(p0, d, 0, 4, state)
    plan.wait_limit(1)
    plan.forward_range(None, d, 4, 7, state)
    plan.wait_limit(0)
    plan.forward_range(None, d, 7, 12, state)
    assert torch.equal(d[:4], ref[:4]) and torch.isnan(d[4:]).all()
    _raises_once(plan)


def test_both_flags_are_told_one_after_the_other():
    i = synth.small_instance(13, n=(64, 64), nt=6, ns=5, pml=4, lossy=True)
    plan = pat.Plan(i.desc, i.c0, i.rho0, i.alpha0_db, i.sensors, device=DEV, check_finite=True)
    p0 = torch.full((64, 64), float("inf"), device=DEV)
    plan.forward(p0)
    plan.wait_limit(1)
    plan.forward(p0)
    codes = []
    for _ in range(3):
        try:
            plan.sync()
            codes.append(pat.PAT_OK)
        except pat.PatError as e:
            codes.append(e.code)
    assert codes == [pat.PAT_EHIP, pat.PAT_ENONFINITE, pat.PAT_OK]


def test_batch_reports_every_instance_of_its_queue():
    """Two grids over all dies are one domain's queue: the second is never
    begun.  Two more on one die each have their own."""
    cases = [_case(20 + k, n=n, nt=nt, ns=6, pml=6, lossy=True)
             for k, (n, nt) in enumerate([((512, 256), 41), ((512, 256), 40), ((64, 64), 30), ((64, 64), 30)])]
    plans, p0, h = zip(*cases)
    ref = [(p.forward(x).clone(), p.adjoint(y).clone()) for p, x, y in cases]
    for p in plans[:2]:
        p.wait_limit(1)
    b = pat.Batch(list(plans))
    for p in plans:
        p.sync()
    for k, (call, args) in enumerate(((b.forward, p0), (b.adjoint, h))):
        out = call(list(args))
        assert torch.isnan(out[0]).all() and torch.isnan(out[1]).all()
        assert torch.equal(out[2], ref[2][k]) and torch.equal(out[3], ref[3][k])
        for p in plans[:2]:
            _raises_once(p)
        for p in plans[2:]:
            p.sync()
    b.forward(list(p0))
    with pytest.raises(pat.PatError) as e:
        pat.solves_check(list(plans))
    assert e.value.code == pat.PAT_EHIP
    pat.solves_check(list(plans))
    b.close()


@pytest.mark.parametrize("run", ["fista", "batched", "power"])
def test_solver_raises(run):
    plan, p0, h = _case(30, n=(64, 64), nt=9, ns=7, pml=6, lossy=True)
    level = solver.Level(plan, h, 1e-3, 0.05)
    plan.wait_limit(1)
    with pytest.raises(pat.PatError):
        if run == "fista":
            solver.fista(level, p0, 2)
        elif run == "batched":
            solver.fista_batched([level], [p0], 2)
        else:
            solver.power_iteration(plan, p0, 2)


@pytest.mark.parametrize("run", ["fista", "coarse", "batched"])
def test_solver_raises_when_only_the_adjoint_gave_up(run):
    """The prox makes zeros of a NaN image; the objective after it does not."""
    plan, p0, h = _case(31, n=(64, 64), nt=9, ns=7, pml=6, lossy=True)

    class OneBadAdjoint(solver.Level):
        def adjoint(self, r):
            self.plan.wait_limit(1)
            g = super().adjoint(r)
            self.plan.wait_limit(0)
            return g

    level = OneBadAdjoint(plan, h, 1e-3, 0.05)
    with pytest.raises(pat.PatError) as e:
        if run == "fista":
            solver.fista(level, p0, 1)
        elif run == "coarse":
            solver.coarse_fista(level, p0, torch.zeros_like(p0), torch.zeros_like(p0), 1e-2, 1, 1e-2)
        else:
            level.adjoint(h)
            solver.fista_batched([level], [p0], 1)
    assert e.value.code == pat.PAT_EHIP
    assert torch.isfinite(plan.forward(p0)).all()


def test_results_stay_nan_until_asked():
    plan, p0, h = _case(32, n=(512, 256), nt=6, ns=7, pml=6, lossy=False)
    ref = plan.forward(p0).clone()
    plan.wait_limit(1)
    plan.adjoint(h)
    plan.wait_limit(0)
    assert torch.isnan(plan.forward(p0)).all() and torch.isnan(plan.adjoint(h)).all()
    _raises_once(plan)
    assert torch.equal(plan.forward(p0), ref)
