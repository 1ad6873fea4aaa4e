"""Column kernels of the Rys plans (default and of small launches): FP64 values,
codes, scales and packed words have the bits of the launch forms that they take the
place of (a lane per quartet, or the table-driven workgroup kernel), for every
class, at one quartet, contractions that end within and at a batch of factors and
of setups, and on both sides of the rule on the launch's size."""
import numpy as np
import pytest

from paper_2303_13632_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
COLUMNS, SMALL = 14, 15


def _compare(precision, shells, quartets, bits=16, packed=False, variants=(1, 2)):
    from paper_2303_13632_amd import eri
    plan = eri.Plan(shells, quartets, precision=precision, bits=bits, packed=packed)
    nv = plan.class_n_variants
    res, tags = [], []
    for v in (0,) + variants:
        plan.set_variants(np.where(nv > v, v, 0).astype(np.int32))
        out = [t.zero_() for t in plan.alloc(eri=True)]
        plan.compute(*out)
        torch.cuda.synchronize()
        res.append(out)
        tags.append(np.array(plan.class_tag))
    here = plan.class_quartets > 0
    for out, tag in zip(res[1:], tags[1:]):
        for got, ref in zip(res[0], out):
            assert torch.equal(got, ref), (precision, bits, packed)
    return tags[0][here], tags[-1][here]


@pytest.mark.parametrize("precision", ["rys", "rys32"])
@pytest.mark.parametrize("form", [(16, False), (12, True), (32, False)])
def test_every_class(precision, form):
    parts = [W.class_case(cid, n_quartets=5, seed=W.SEED_BASE + 17) for cid in range(256)]
    shells, quartets = W.merge(parts)
    first, _ = _compare(precision, shells, quartets, *form)
    assert (first == SMALL).sum() > 100 and (first == COLUMNS).sum() > 60


@pytest.mark.parametrize("L,limit", [((1, 1, 1, 1), 8192), ((2, 0, 1, 0), 8192), ((2, 2, 1, 0), 512), ((3, 3, 1, 0), 512),
                                     ((3, 2, 3, 2), 256), ((3, 3, 3, 3), 256), ((2, 2, 2, 2), 0)])
def test_launch_sizes(L, limit):
    for n, k in ((1, 6), (2, 5), (3, 1), (limit, 2), (limit + 1, 2)):
        if n:
            first, _ = _compare("rys", *W.random_class_quartets(*L, n, 11 * n + sum(L), k_fixed=k), variants=(1,))
            small = n <= limit and (k > 1 or sum(L) > 4)
            assert (first[0] == SMALL) == small, (L, n, k)
