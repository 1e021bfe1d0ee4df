"""GPU: which path a batch takes.  Explicit settings (chunk, parts, lanes, no
fusion, no stagger, a forced tile) run the launches they describe; only the
default settings may run as resident solves.  Tests of either path elsewhere
rest on this."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1603_02329_amd as pat  # noqa: E402

DEV = "cuda"


def _plans(specs):
    insts = [synth.small_instance(1200 + i, **s) for i, s in enumerate(specs)]
    plans = [pat.Plan(i.desc, i.c0, i.rho0, i.alpha0_db, i.sensors, device=DEV) for i in insts]
    p0 = [torch.from_numpy(i.p0).to(DEV) for i in insts]
    rng = np.random.default_rng(2)
    h = [torch.from_numpy(rng.standard_normal((i.desc.nt, i.ns)).astype(np.float32)).to(DEV) for i in insts]
    return plans, p0, h


TUNABLE = [dict(n=(128, 128), nt=13, ns=6, pml=6, lossy=True), dict(n=(128, 128), nt=13, ns=5, pml=5, lossy=True),
           dict(n=(64, 256), nt=11, ns=4, pml=4, lossy=False)]
MIXED = [dict(n=(128, 128), nt=7, ns=5, pml=6, lossy=True), dict(n=(256, 256), nt=11, ns=6, pml=8, lossy=True),
         dict(n=(128, 128), nt=9, ns=4, pml=6, lossy=False), dict(n=(64, 64), nt=8, ns=4, pml=4, lossy=True)]


@pytest.mark.parametrize("specs", [TUNABLE, MIXED])
@pytest.mark.parametrize("opts", [dict(chunk=1), dict(chunk=4), dict(chunk=64), dict(parts=1), dict(lanes=1),
                                  dict(fuse=False), dict(stagger=False)])
def test_explicit_settings_run_launches(specs, opts):
    plans, p0, h = _plans(specs)
    ref = [(p.forward(x).clone(), p.adjoint(y).clone()) for p, x, y in zip(plans, p0, h)]
    b = pat.Batch(plans, **opts)
    assert not b.resident
    for _ in range(2):
        d, im = b.forward(p0), b.adjoint(h)
        for k, (rd, ri) in enumerate(ref):
            assert torch.equal(d[k], rd) and torch.equal(im[k], ri), k
    b.close()


@pytest.mark.parametrize("specs", [
    TUNABLE, MIXED,
    [dict(n=(64, 64), nt=9 + k, ns=5, pml=4, lossy=True) for k in range(11)] + [dict(n=(64, 128), nt=14, ns=40, pml=4, lossy=False)],
    [dict(n=(512, 512), nt=21, ns=30, pml=8, lossy=True), dict(n=(256, 256), nt=11, ns=30, pml=8, lossy=True),
     dict(n=(128, 32), nt=40, ns=30, pml=8, lossy=False)]])
def test_default_settings_of_small_batches_are_resident(specs):
    plans, _, _ = _plans(specs)
    b = pat.Batch(plans)
    assert b.resident
    b.close()


def test_tile_and_tuning_of_a_resident_batch(tmp_path):
    plans, p0, h = _plans(TUNABLE)
    ref = [(p.forward(x).clone(), p.adjoint(y).clone()) for p, x, y in zip(plans, p0, h)]
    cache = tmp_path / "tiles.json"
    b = pat.Batch(plans)
    assert b.resident and b.autotune(reps=1, cache=str(cache)) == [] and b.tuning_report() == []
    assert b.resident and not cache.exists()
    e = dict(n=[128, 128, 1], nt=13, lossy=1, dir=0, tile=4)
    with pytest.raises(pat.PatError):
        b.set_tile(dict(e, **{"pass": 0}), 2)  # refused: nothing changes
    assert b.resident
    b.set_tile(dict(e, **{"pass": 0}))
    assert not b.resident
    d, im = b.forward(p0), b.adjoint(h)
    for k, (rd, ri) in enumerate(ref):
        assert torch.equal(d[k], rd) and torch.equal(im[k], ri), k
    b.close()
    one = pat.Batch(plans[:1], chunk=4)  # launches: timed, reported and stored as ever
    rep = one.autotune(reps=1, cache=str(cache))
    assert rep and cache.exists()
    one.close()
