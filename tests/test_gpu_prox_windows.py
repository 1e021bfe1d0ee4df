"""GPU: the proximal map's launches of several iterations (2D) against its
two launches per iteration, bitwise.  The latter run where the result
overwrites the lower bound."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1603_02329_amd as pat  # noqa: E402


def _image(shape, seed, special=False):
    rng = np.random.default_rng(seed)
    z = rng.standard_normal(shape).astype(np.float32)
    if special:
        z.flat[[0, z.size // 2, z.size - 1]] = [np.inf, np.nan, -np.inf]
    lower = (0.3 * rng.standard_normal(shape)).astype(np.float32)
    return torch.from_numpy(z).cuda(), torch.from_numpy(lower).cuda()


def _same(a, b):
    return torch.equal(a.view(torch.int32), b.view(torch.int32))


# kept part of a window: 62 x 46 after one iteration ... 32 x 16 after 16,
# one less where the result is formed; more than 32 iterations: both kinds
@pytest.mark.parametrize("n_iter", [1, 2, 12, 13, 20, 25, 32, 33, 40])
def test_windows_match_launches_bitwise(n_iter):
    shapes = [(1, 1), (1, 90), (90, 1), (16, 32), (17, 31), (23, 39), (24, 40), (25, 41), (27, 43), (28, 44), (45, 61), (46, 62), (100, 333)]
    for k, shape in enumerate(shapes):
        z, lower = _image(shape, 10 * n_iter + k, special=k % 4 == 3)
        both = lower.clone()
        pat.tv_prox(z, 0.3, n_iter, lower=both, out=both)
        assert _same(pat.tv_prox(z, 0.3, n_iter, lower=lower), both), shape
        zero = torch.zeros_like(z)
        pat.tv_prox(z, 0.02, n_iter, lower=zero, out=zero)
        assert _same(pat.tv_prox(z, 0.02, n_iter), zero), shape


def test_windows_batched_bitwise():
    shapes = [(24, 40), (64, 64), (1, 70), (131, 45)] * 7  # more than one launch holds
    images = [_image(s, k) for k, s in enumerate(shapes)]
    zs, lowers = [z for z, _ in images], [lo if k % 3 else None for k, (_, lo) in enumerate(images)]
    lams = [0.05 * (1 + k % 5) for k in range(len(zs))]
    for n_iter in (7, 20, 35):
        out = pat.tv_prox_batched(zs, lams, n_iter, lowers=lowers)
        for k, z in enumerate(zs):
            assert _same(out[k], pat.tv_prox(z, lams[k], n_iter, lower=lowers[k])), (n_iter, k)
