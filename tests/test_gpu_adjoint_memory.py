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
