"""GPU: resident solves (a 2D time loop in one launch) against the per-pass
launches, bitwise: every shape class at the edges of its range, segments,
batches, two streams at once, and replays of a captured solve.  The per-pass
launches run while pass timing is on (here for a row length no grid has)."""
import contextlib

import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1603_02329_amd as pat  # noqa: E402

DEV = "cuda"


@contextlib.contextmanager
def per_pass_launches():
    pat.timing_begin(0, 0, 7)
    try:
        yield
    finally:
        torch.cuda.synchronize()
        pat.timing_end()


def _solve(plan, p0, h):
    return plan.forward(p0).clone(), plan.adjoint(h).clone()


def _case(seed, **kw):
    i = synth.small_instance(seed, **kw)
    plan = pat.Plan(i.desc, i.c0, i.rho0, i.alpha0_db, i.sensors, device=DEV, check_finite=True)
    rng = np.random.default_rng(seed)
    h = torch.from_numpy(rng.standard_normal((i.desc.nt, i.ns)).astype(np.float32)).to(DEV)
    return plan, torch.from_numpy(i.p0).to(DEV), h


@pytest.mark.parametrize("lossy", [True, False])
@pytest.mark.parametrize("nx", [32, 64, 128, 256, 512])
def test_resident_matches_launches_bitwise(nx, lossy):
    """Every grid of the range; the shortest loops; rows with no sensor and
    rows with more sensors than a wavefront has lanes."""
    for k, ny in enumerate((32, 64, 128, 256, 512)):
        nt, ns = ((2, 1), (3, 900), (6, 31), (5, 7), (4, 257))[(k + nx // 32) % 5]
        plan, p0, h = _case(40 * nx + ny, n=(nx, ny), nt=nt, ns=ns, pml=5, lossy=lossy)
        d, im = _solve(plan, p0, h)
        plan.sync()
        with per_pass_launches():
            rd, rim = _solve(plan, p0, h)
        assert torch.equal(d, rd), (nx, ny)
        assert torch.equal(im, rim), (nx, ny)


def test_resident_segments_bitwise():
    for n in ((128, 64), (512, 512)):
        plan, p0, _ = _case(7, n=n, nt=12, ns=20, pml=6, lossy=True)
        ref = plan.forward(p0).clone()
        d = torch.zeros_like(ref)
        state = torch.empty(plan.state_bytes, dtype=torch.uint8, device=DEV)
        for a, b in ((0, 1), (1, 5), (5, 12)):
            plan.forward_range(p0 if a == 0 else None, d, a, b, state)
        assert torch.equal(d, ref), n


@pytest.mark.parametrize("which", ["dies", "all dies and one"])
def test_resident_batch_bitwise(which):
    """Several shapes and physics, more instances of one shape than dies; a
    grid over every die beside grids on one."""
    if which == "dies":
        specs = [dict(n=(64, 64), nt=9 + k, ns=5, pml=4, lossy=True) for k in range(11)]
        specs += [dict(n=(64, 128), nt=14, ns=40, pml=4, lossy=False), dict(n=(32, 64), nt=1, ns=3, pml=4, lossy=True),
                  dict(n=(32, 32), nt=20, ns=3, pml=4, lossy=True)]
    else:
        specs = [dict(n=(512, 512), nt=21, ns=30, pml=8, lossy=True), dict(n=(256, 256), nt=11, ns=30, pml=8, lossy=True),
                 dict(n=(128, 32), nt=40, ns=30, pml=8, lossy=False)]
    cases = [_case(100 + k, **s) for k, s in enumerate(specs)]
    plans, p0, h = zip(*cases)
    b = pat.Batch(plans)
    for _ in range(2):
        d, im = b.forward(list(p0)), b.adjoint(list(h))
        torch.cuda.synchronize()
        with per_pass_launches():
            ref = [_solve(p, x, y) for p, x, y in cases]
        for k, (rd, rim) in enumerate(ref):
            assert torch.equal(d[k], rd) and torch.equal(im[k], rim), k
    b.close()


def test_resident_two_streams_bitwise():
    cases = [_case(300 + k, n=n, nt=40, ns=9, pml=6, lossy=True)
             for k, n in enumerate([(512, 512), (128, 128), (512, 256), (256, 256)])]
    with per_pass_launches():
        ref = [_solve(*c) for c in cases]
    main, side = torch.cuda.current_stream(), torch.cuda.Stream()
    side.wait_stream(main)
    out = []
    for k, c in enumerate(cases):
        with torch.cuda.stream(side if k % 2 else main):
            out.append(_solve(*c))
    torch.cuda.synchronize()
    for k, ((d, im), (rd, rim)) in enumerate(zip(out, ref)):
        assert torch.equal(d, rd) and torch.equal(im, rim), k


@pytest.mark.parametrize("n", [(64, 64), (512, 256)])
def test_resident_capture_replays_bitwise(n):
    plan, p0, h = _case(500, n=n, nt=15, ns=9, pml=6, lossy=True)
    d, im = torch.empty(15, 9, device=DEV), torch.empty(n[1], n[0], device=DEV)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        plan.forward(p0, d)
        plan.adjoint(h, im)
        side.synchronize()
        with torch.cuda.graph(g, stream=side):
            plan.forward(p0, d)
            plan.adjoint(h, im)
    torch.cuda.synchronize()
    rng = np.random.default_rng(1)
    for rep in range(3):
        p0.copy_(torch.from_numpy(rng.standard_normal((n[1], n[0])).astype(np.float32)))
        h.copy_(torch.from_numpy(rng.standard_normal((15, 9)).astype(np.float32)))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        got = d.clone(), im.clone()
        ref = _solve(plan, p0, h)
        torch.cuda.synchronize()
        assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1]), rep
