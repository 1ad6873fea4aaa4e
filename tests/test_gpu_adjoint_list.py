"""eri_backward on explicit lists: classes of few quartets (one launch, a
workgroup per quartet, side and some primitive pairs) and of many (derived
classes) in one call, at the edges of the split: deep contractions (batches of
source pairs and blocks of target pairs with remainders), a single quartet, a
class on either side of the line.  Against the oracle's analytic gradient."""
import os

import numpy as np
import pytest

import oracle as O
from paper_2303_13632_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
THREADS = min(16, os.cpu_count() or 1)
RTOL = 1e-10     # the bar of the other gradient tests, relative to the largest entry


def _check(sh, q, seed, density=False):
    from paper_2303_13632_amd import eri
    plan = eri.Plan(sh, q, bits=0)
    rng = np.random.default_rng(seed)
    if density:
        D = W.random_density(plan.nbf, seed=seed)
        D = D + 0.05 * rng.normal(size=D.shape)      # not symmetric: the pair's order counts
        kw, ref = {"density": torch.tensor(D, device="cuda")}, {"density": D}
    else:
        dl = rng.uniform(-1.0, 1.0, size=plan.out_values)
        kw, ref = {"dl": torch.tensor(dl, device="cuda")}, {"dl": plan.to_user(dl)}
    gc, ge, en = plan.backward(**kw)
    alone = plan.backward(energy_only=True, **kw)[2]
    torch.cuda.synchronize()
    E, gx, gex = O.gradient(sh, q, n_threads=THREADS, **ref)
    assert np.abs(gc.cpu().numpy() - gx).max() <= RTOL * np.abs(gx).max()
    assert np.abs(ge.cpu().numpy() - gex).max() <= RTOL * np.abs(gex).max()
    assert abs(en.item() - E) <= RTOL * abs(E)
    assert en.item() == alone.item()


@pytest.mark.parametrize("ls,ks", [
    ((0, 0, 0, 0), (16, 16, 16, 16)),
    ((1, 0, 0, 1), (7, 3, 1, 5)),
    ((0, 2, 2, 1), (3, 3, 5, 1)),
    ((2, 2, 1, 1), (2, 3, 3, 3)),
    ((1, 2, 2, 2), (3, 1, 2, 2)),
    ((2, 2, 2, 2), (3, 3, 1, 2)),
    ((2, 2, 2, 2), (1, 1, 1, 1)),
])
def test_one_quartet(ls, ks):
    rng = np.random.default_rng(sum(ls) + 100 * sum(ks))
    sh = W._pack(ls, ks, rng.uniform(0.0, 3.0, (4, 3)), [np.exp(rng.uniform(np.log(0.1), np.log(100.0), k)) for k in ks],
                 [rng.uniform(0.1, 1.0, k) for k in ks])
    _check(sh, np.array([[0, 1, 2, 3]], np.int32), 7)


@pytest.mark.parametrize("density", [False, True])
def test_every_class(density):
    """Each of the 81 classes of s, p and d shells twice, shells repeated within quartets."""
    sh = W.random_shells(9, lmax=2, seed=77, box=3.0)
    by = [np.flatnonzero(sh["L"] == l) for l in range(3)]
    assert min(len(b) for b in by) >= 2
    rng = np.random.default_rng(78)
    q = [[rng.choice(by[l]) for l in c] for c in np.ndindex(3, 3, 3, 3) for _ in range(2)]
    _check(sh, np.array(q, np.int32), 79, density)


@pytest.mark.parametrize("n", [2048, 2049])
def test_either_side_of_the_line(n):
    """n quartets of one class (listed up to 2048) and a few of others."""
    a = W.random_class_quartets(1, 0, 0, 0, n, 81, k_choices=(1, 2))
    b = W.random_class_quartets(2, 1, 1, 0, 5, 82)
    c = W.random_class_quartets(0, 0, 2, 2, 3, 83)
    _check(*W.merge([a, b, c]), 84)
