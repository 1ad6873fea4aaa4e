"""The density form of eri_backward on screened plans (Hermite potentials of
primitive pairs) against the oracle's analytic gradient over the plan's own
quartets: missing shell types (pair classes without pairs), screening that
cuts the pair ranges, a density that is not symmetric in the stored pair
order, and the energy's bits with and without a gradient."""
import os

import numpy as np
import pytest

import oracle as O
from paper_2303_13632_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
THREADS = min(16, os.cpu_count() or 1)
RTOL = 1e-10     # the bar of the other gradient tests, relative to the largest entry


def _weights(q):
    a, b, c, d = q.T
    same = ((a == c) & (b == d)) | ((a == d) & (b == c))
    return (1.0 + (a != b)) * (1.0 + (c != d)) * (1.0 + ~same)


def _shells(ls, ks, seed, box):
    """Shells of the given angular momenta; exponents up to 500."""
    rng = np.random.default_rng(seed)
    n = len(ls)
    return W._pack(ls, ks, rng.uniform(0.0, box, (n, 3)), [np.exp(rng.uniform(np.log(0.1), np.log(500.0), k)) for k in ks],
                   [rng.uniform(0.1, 1.0, k) for k in ks])


# (angular momenta, primitives per shell, box, Schwarz threshold)
SETS = {
    "one-shell": ([0], [1], 1.0, 0.0),
    "s-only": ([0] * 9, [1, 2, 3, 4, 5, 6, 1, 16, 2], 6.0, 1e-8),
    "d-only": ([2] * 3, [2, 1, 3], 3.0, 0.0),
    "p-and-d": ([1, 2, 1, 2], [3, 2, 1, 1], 4.0, 1e-6),
    "spd-cut": ([0, 1, 2, 0, 1, 0, 1], [4, 2, 1, 1, 3, 6, 1], 9.0, 1e-3),
    "all-cut": ([0, 0], [1, 1], 1.0, 1e6),
}


@pytest.mark.parametrize("name", sorted(SETS))
def test_against_oracle(name):
    from paper_2303_13632_amd import eri
    ls, ks, box, tau = SETS[name]
    sh = _shells(ls, ks, 300 + len(ls), box)
    plan = eri.Plan(sh, None, bits=0, schwarz=tau)
    D = W.random_density(plan.nbf, seed=len(ls))
    t = torch.tensor(D, device="cuda")
    gc, ge, en = plan.backward(density=t)
    alone = plan.backward(density=t, energy_only=True)[2]
    torch.cuda.synchronize()
    assert en.item() == alone.item()
    lists = [plan.class_quartet_list(c) for c in range(256) if plan.class_quartets[c]]
    if not lists:
        assert not gc.any() and not ge.any() and en.item() == 0.0
        return
    q = np.concatenate(lists)
    print(name, len(q), "quartets", flush=True)
    E, gx, gex = O.gradient(sh, q, weights=_weights(q), density=D, n_threads=THREADS)
    assert np.abs(gc.cpu().numpy() - gx).max() <= RTOL * np.abs(gx).max()
    assert np.abs(ge.cpu().numpy() - gex).max() <= RTOL * np.abs(gex).max()
    assert abs(en.item() - E) <= RTOL * abs(E)
    # added to what the caller's arrays hold; other geometry, same plan
    gc2, ge2, en2 = gc.clone(), ge.clone(), en.clone()
    plan.backward(density=t, grad_centers=gc2, grad_exps=ge2, energy=en2)
    assert (gc2 - 2 * gc).abs().max() <= 1e-12 * gc.abs().max() and abs(en2.item() - 2 * en.item()) <= 1e-14 * abs(E)
    x = np.array(sh["xyz"]) + 0.01
    plan.set_geometry(xyz=x)
    moved = plan.backward(density=t, energy_only=True)[2].item()     # all shells by the same vector
    assert abs(moved - en.item()) <= 1e-10 * abs(E)


def test_many_targets():
    """More than 64 primitive pairs per shell-pair group and jobs of several
    chunks: the sum of the centre gradients vanishes (translation), and the
    scaling identity sum R dE/dR - 2 sum alpha dE/dalpha = -E holds (coordinates by
    lambda, exponents by 1/lambda^2, normalised primitives)."""
    from paper_2303_13632_amd import eri
    sh = W.molecule_basis(n_heavy=4, n_h=8, lattice=(3, 2, 2), seed=W.SEED_BASE + 48)
    plan = eri.Plan(sh, None, bits=0, schwarz=0.0)
    D = torch.tensor(W.random_density(plan.nbf, seed=48), device="cuda")
    gc, ge, en = plan.backward(density=D)
    gc, ge, E = gc.cpu().numpy(), ge.cpu().numpy(), en.item()
    assert np.abs(gc.sum(0)).max() <= 1e-10 * np.abs(gc).max()
    lhs = float((gc * np.asarray(sh["xyz"])).sum() - 2.0 * (ge * sh["exps"]).sum())
    size = np.abs(gc * np.asarray(sh["xyz"])).sum() + 2.0 * np.abs(ge * sh["exps"]).sum()
    assert abs(lhs + E) <= 1e-10 * size


@pytest.mark.parametrize("value", [np.inf, np.nan])
@pytest.mark.parametrize("ls", [(0, 0, 0), (1, 0, 2), (2, 2, 2)])
def test_density_of_pairs_without_a_common_quartet(ls, value):
    """Of a strong shell a and weak shells e and c the plan keeps (aa|aa),
    (ae|aa) and (ac|aa): what the density holds for the pair ae does not reach
    the gradient of c."""
    from paper_2303_13632_amd import eri
    sh = _shells(ls, [3, 2, 2], 91, 1.0)
    sh["exps"][:] = [0.8, 1.3, 2.1, 0.9, 1.7, 1.1, 1.4]
    sh["coefs"][:] = [1.0, 0.5, 0.7, 1e-5, 1e-5, 1e-5, 1e-5]
    plan = eri.Plan(sh, None, bits=0, schwarz=1e-7)
    q = np.concatenate([plan.class_quartet_list(c) for c in range(256) if plan.class_quartets[c]])
    have = {tuple(sorted((tuple(sorted(x[:2])), tuple(sorted(x[2:]))))) for x in q.tolist()}
    aa, ae, ac = (0, 0), (0, 1), (0, 2)
    assert have == {(aa, aa), (aa, ae), (aa, ac)}
    n = [W.ncart(l) for l in ls]
    D = W.random_density(plan.nbf, seed=92)
    ref = plan.backward(density=torch.tensor(D, device="cuda"))[:2]
    D[:n[0], n[0]:n[0] + n[1]] = value
    D[n[0]:n[0] + n[1], :n[0]] = value
    got = plan.backward(density=torch.tensor(D, device="cuda"))[:2]
    for g, r in zip((got[0][2], got[1][5:]), (ref[0][2], ref[1][5:])):
        assert (g - r).abs().max().item() <= 1e-12 * r.abs().max().item()
    assert not torch.isfinite(got[0][1]).any()
