"""Device memory of eri_backward's workspaces, and shell sets without shells."""
import ctypes
import os

import numpy as np
import pytest

import oracle as O
from paper_2303_13632_amd import eri, workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
THREADS = min(16, os.cpu_count() or 1)


def _device_bytes(plan):
    info = eri.PlanInfo()
    assert eri.load().eri_plan_info_get(plan._h, ctypes.byref(info)) == eri.ERI_OK
    return info.device_bytes


def test_slices_of_a_list_over_many_shells():
    """Short classes of a plan over 65536 shells: the gradient's slices, which
    span all of them, stay within 32 MB (64 of them would take 190 MB)."""
    sh, q = W.merge([W.random_class_quartets(*L, 2048, 40 + i, k_choices=(1, 2), box=3.0)
                     for i, L in enumerate([(0, 0, 0, 0), (1, 0, 0, 0), (0, 1, 0, 0), (0, 0, 1, 0), (0, 0, 0, 1),
                                            (1, 0, 1, 0), (1, 1, 0, 0), (0, 0, 1, 1)])])
    plan = eri.Plan(sh, q, bits=0)
    before = _device_bytes(plan)
    dl = np.random.default_rng(41).uniform(-1.0, 1.0, plan.out_values)
    gc, ge, en = plan.backward(dl=torch.tensor(dl, device="cuda"))
    # item and work lists of 16384 quartets come on top
    assert _device_bytes(plan) - before <= (32 << 20) + 16384 * 1024
    E, gx, gex = O.gradient(sh, q, dl=plan.to_user(dl), n_threads=THREADS)
    assert np.abs(gc.cpu().numpy() - gx).max() <= 1e-10 * np.abs(gx).max()
    assert np.abs(ge.cpu().numpy() - gex).max() <= 1e-10 * np.abs(gex).max()
    assert abs(en.item() - E) <= 1e-10 * abs(E)


@pytest.mark.parametrize("batched", [False, True])
def test_no_shells(batched):
    """A plan over no shells has L = 0, with and without a gradient."""
    plan = eri.Plan(W._pack([], [], np.zeros((0, 3)), [], []), None if batched else np.zeros((0, 4), np.int32), bits=0)
    room = torch.full((4,), 2.0, dtype=torch.float64, device="cuda")
    ptr = ctypes.c_void_p(room.data_ptr())
    for grad in (None, ptr):
        energy = ctypes.c_void_p(room.data_ptr() + 8)
        assert eri.load().eri_backward(plan._h, None, None, ptr, 0, grad, grad, energy) == eri.ERI_OK
    torch.cuda.synchronize()
    assert (room == 2.0).all()


def test_no_density_rows_without_a_density():
    """The D_ab D_cd rows of a pass are held from the first call with a density on,
    and for the classes that use them: not for [pp|pp] here, whose 200 quartets have
    more values than the 2600 of the class that does."""
    sh = W.random_shells(12, lmax=2, seed=50, k_choices=(1, 2))
    by = [np.flatnonzero(sh["L"] == l) for l in range(3)]
    rng = np.random.default_rng(51)
    q = [[rng.choice(by[l]) for l in L] for L, n in (((1, 0, 0, 0), 2600), ((1, 1, 1, 1), 200)) for _ in range(n)]
    plan = eri.Plan(sh, np.array(q, np.int32), bits=0)
    plan.backward(dl=torch.ones(plan.out_values, dtype=torch.float64, device="cuda"))
    before = _device_bytes(plan)
    for _ in range(2):
        plan.backward(density=torch.tensor(W.random_density(plan.nbf, seed=52), device="cuda"))
        assert _device_bytes(plan) - before == 2600 * 3 * 8
