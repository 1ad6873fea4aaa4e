"""eri_backward of explicit lists on each of its routes: classes in one launch,
classes through derived classes (many or deep quartets, in passes and slices),
L from the class's own kernel beside either, several of these in one list; and
screened plans given dL/dERI.  Against the oracle's analytic gradient."""
import os

import numpy as np
import pytest

import oracle as O
from paper_2303_13632_amd import eri, workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
THREADS = min(16, os.cpu_count() or 1)
RTOL = 1e-10     # the bar of the other gradient tests, relative to the largest entry


def _check(sh, q, seed, density=False, **kw):
    plan = eri.Plan(sh, q, bits=0, **kw)
    rng = np.random.default_rng(seed)
    if density:
        D = 0.1 * rng.normal(size=(plan.nbf, plan.nbf))      # not symmetric: the pair's order counts
        kw, ref = {"density": torch.tensor(D, device="cuda")}, {"density": D}
    else:
        dl = rng.uniform(-1.0, 1.0, size=plan.out_values)
        kw, ref = {"dl": torch.tensor(dl, device="cuda")}, {"dl": plan.to_user(dl)}
    before = plan.backward(energy_only=True, **kw)[2]
    gc, ge, en = plan.backward(**kw)
    alone = plan.backward(energy_only=True, **kw)[2]
    torch.cuda.synchronize()
    E, gx, gex = O.gradient(sh, q, n_threads=THREADS, **ref)
    assert np.abs(gc.cpu().numpy() - gx).max() <= RTOL * np.abs(gx).max()
    assert np.abs(ge.cpu().numpy() - gex).max() <= RTOL * np.abs(gex).max()
    # (cancelling terms: against the size of the sum's terms as the gradient's scale gives it)
    assert abs(en.item() - E) <= RTOL * max(abs(E), np.abs(gx).max())
    assert before.item() == en.item() == alone.item()


def _part(L, n, seed, **kw):
    return W.random_class_quartets(*L, n, seed, box=3.0, **kw)


def _shared(L, n, pool, seed, k_choices=(1, 2)):
    """n quartets of class L over a pool of shells per angular momentum: pairs in
    either order of their shells, pairs of one shell with itself, repeats."""
    rng = np.random.default_rng(seed)
    ls = sorted(set(L))
    kind = np.repeat(ls, pool)
    ks = rng.choice(k_choices, size=len(kind))
    sh = W._pack(kind, ks, rng.uniform(0.0, 3.0, (len(kind), 3)),
                 [np.exp(rng.uniform(np.log(0.1), np.log(100.0), k)) for k in ks], [rng.uniform(0.1, 1.0, k) for k in ks])
    by = {l: np.flatnonzero(kind == l) for l in ls}
    return sh, np.stack([rng.choice(by[l], size=n) for l in L], axis=1).astype(np.int32)


@pytest.mark.parametrize("density", [False, True])
@pytest.mark.parametrize("L,pool", [((1, 1, 1, 1), 12), ((2, 1, 2, 1), 8), ((1, 2, 2, 1), 8), ((2, 2, 2, 2), 6),
                                    ((0, 2, 1, 0), 10), ((2, 2, 0, 0), 8), ((0, 0, 2, 2), 8)])
def test_more_quartets_than_the_line(L, pool, density):
    """Derived classes from slot kernels of every kind, mixed orientations."""
    _check(*_shared(L, 2200, pool, 1 + sum(L), k_choices=(1,) if sum(L) > 6 else (1, 2)), 31, density)


@pytest.mark.parametrize("density", [False, True])
def test_passes_and_slices(density):
    """chunk_quartets below the class: several passes, their L and gradients added up."""
    _check(*_shared((1, 1, 2, 1), 2500, 9, 5), 32, density, chunk_quartets=700)


@pytest.mark.parametrize("L,n,k", [((1, 1, 1, 0), 1000, 4), ((0, 0, 2, 2), 700, 4), ((2, 1, 2, 1), 250, 4)])
def test_deep_contractions(L, n, k):
    """Few quartets, but too deep for the launch over primitive quartets."""
    _check(*_part(L, n, 6, k_fixed=k), 33)


@pytest.mark.parametrize("density", [False, True])
def test_energy_from_the_class_kernels(density):
    """The gradient from the one launch, L from the classes' own kernels: lane and slot forms."""
    _check(*W.merge([_part((2, 2, 2, 2), 24, 7), _part((2, 0, 2, 0), 130, 8), _part((0, 0, 0, 0), 600, 9)]), 34, density)


@pytest.mark.parametrize("density", [False, True])
def test_all_routes_in_one_list(density):
    _check(*W.merge([_part((1, 0, 0, 0), 2100, 10, k_choices=(1, 2)), _part((1, 1, 1, 0), 1000, 11, k_fixed=4),
                     _part((1, 1, 1, 1), 700, 12), _part((0, 2, 1, 0), 5, 13), _part((0, 0, 0, 0), 3, 14, k_fixed=16)]),
           35, density)


@pytest.mark.parametrize("density", [False, True])
def test_blocks_of_target_pairs(density):
    """Enough target primitive pairs that a workgroup of the one launch takes more
    than one block of eight of them, with remainders, over many source batches."""
    parts = [_part(L, 45, 16 + i, k_choices=(7, 9, 10, 11, 12))
             for i, L in enumerate([(0, 0, 0, 0), (1, 0, 0, 0), (0, 1, 1, 0), (2, 0, 0, 0), (0, 0, 1, 1)])]
    sh, q = W.merge(parts)
    pairs = (sh["K"][q[:, 0]] * sh["K"][q[:, 1]] + sh["K"][q[:, 2]] * sh["K"][q[:, 3]]).sum()
    assert pairs // 4096 > 8
    _check(sh, q, 36, density)


def test_screened_plan_with_dl():
    """dL/dERI of a screened plan: its quartets' degeneracies count."""
    sh = W.molecule_basis(n_heavy=1, n_h=3, lattice=(2, 2, 1), seed=17)
    plan = eri.Plan(sh, None, bits=0, schwarz=1e-6)
    dl = np.random.default_rng(18).uniform(-1.0, 1.0, plan.out_values)
    gc, ge, en = plan.backward(dl=torch.tensor(dl, device="cuda"))
    q = np.concatenate([plan.class_quartet_list(c) for c in range(256) if plan.class_quartets[c]])
    a, b, c, d = q.T
    w = (1.0 + (a != b)) * (1.0 + (c != d)) * (1.0 + ~((a == c) & (b == d)))
    E, gx, gex = O.gradient(sh, q, weights=w, dl=dl, n_threads=THREADS)
    assert np.abs(gc.cpu().numpy() - gx).max() <= RTOL * np.abs(gx).max()
    assert np.abs(ge.cpu().numpy() - gex).max() <= RTOL * np.abs(gex).max()
    assert abs(en.item() - E) <= RTOL * max(abs(E), np.abs(gx).max())
