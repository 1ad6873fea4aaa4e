"""Primitive-parallel kernels (default of small launches): the bits of the
class's other kernels with the same orientation, FP64 values, codes, scales and
packed words, at the edges of their work split: one quartet, workgroups partly
filled, contractions that end anywhere in a turn, several turns of a workgroup."""
import numpy as np
import pytest

from paper_2303_13632_amd import eri, workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

PRIM = 13
# tags of kernels with the default's operation order (in mixed precision the form
# with a slot of lanes, tag 1, rounds FP32 sums elsewhere)
SAME = {"fp64": (0, 1, 2), "mixed": (0,)}


def _outputs(plan, cid, variant):
    v = np.zeros(256, np.int32)
    v[cid] = variant
    plan.set_variants(v)
    out = [t.zero_() for t in plan.alloc(eri=True)]
    plan.compute(*out)
    torch.cuda.synchronize()
    return int(plan.class_tag[cid]), out


def _compare(L, n, k, precision="fp64", forms=((16, False),)):
    cid = W.class_id(*L)
    kw = {"k_fixed": k} if k else {}
    shells, quartets = W.random_class_quartets(*L, n, 7 * n + cid, **kw)
    for bits, packed in forms:
        plan = eri.Plan(shells, quartets, precision=precision, bits=bits, packed=packed)
        tag, got = _outputs(plan, cid, 0)
        assert tag == PRIM
        others = 0
        for variant in range(1, int(plan.class_n_variants[cid])):
            tag, ref = _outputs(plan, cid, variant)
            if tag in SAME[precision]:
                others += 1
                for g, r in zip(got, ref):
                    assert torch.equal(g, r), (L, n, k, bits, packed, variant)
        assert others


@pytest.mark.parametrize("L", [(0, 0, 0, 0), (0, 1, 0, 0), (1, 0, 0, 2), (1, 1, 0, 1), (2, 1, 0, 1), (0, 0, 3, 1),
                               (2, 2, 0, 0), (2, 0, 0, 2)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_lane_per_quartet_classes(L, precision):
    for n, k in ((1, 16), (3, 5), (4, 4), (5, 3), (17, 0), (65, 0), (16385, 0)):
        _compare(L, n, k, precision)
    _compare(L, 67, 0, precision, forms=((3, True), (8, True), (12, True), (24, True), (8, False), (32, False)))


@pytest.mark.parametrize("L", [(1, 1, 1, 1), (2, 1, 2, 1), (2, 2, 2, 2), (3, 2, 3, 2), (2, 2, 1, 0), (3, 0, 2, 0)])
def test_slot_classes(L):
    for n, k in ((1, 16), (3, 5), (2, 2), (17, 0), (257, 0)):
        _compare(L, n, k)
    _compare(L, 19, 0, forms=((3, True), (8, True), (12, True), (24, True), (8, False), (32, False)))


@pytest.mark.parametrize("L,n,k", [((3, 3, 0, 0), 4097, 1), ((0, 0, 2, 3), 4097, 2), ((2, 2, 1, 0), 14337, 1),
                                   ((0, 1, 1, 3), 14337, 2), ((1, 1, 2, 0), 49153, 3)])
def test_lanes_of_large_launches(L, n, k):
    """Above the rule's size a class with a lane-per-quartet form takes it: the values
    are those of the slot kernels, bit for bit."""
    cid = W.class_id(*L)
    shells, quartets = W.random_class_quartets(*L, n, n + cid, k_fixed=k)
    values = []
    for q in (quartets, quartets[: n - 1]):
        plan = eri.Plan(shells, q, bits=16)
        tag, out = _outputs(plan, cid, 0)
        assert (tag == 1) == (len(q) == n)
        values.append(plan.to_user(out[0].cpu().numpy()[: plan.n_eri]))
    assert np.array_equal(values[0][: len(values[1])], values[1])
