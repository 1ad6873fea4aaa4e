"""The kernel of a Rys class by its launch's size and contractions: which of the two
column kernels or the table-driven one runs on both sides of each limit, every one
with the bits of the table-driven kernel, which stays the class's last variant."""
import numpy as np
import pytest

from paper_2303_13632_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
TABLE, COLUMNS, SMALL = 0, 14, 15

CASES = [("rys", (3, 0, 3, 0), 1000, 1, TABLE), ("rys", (3, 0, 3, 0), 1000, 2, COLUMNS),
         ("rys", (3, 1, 3, 1), 300, 1, TABLE), ("rys", (3, 1, 3, 1), 300, 2, COLUMNS),
         ("rys", (2, 1, 2, 1), 1, 2, COLUMNS), ("rys", (2, 1, 1, 1), 512, 1, SMALL), ("rys", (2, 1, 1, 1), 513, 1, TABLE),
         ("rys", (2, 2, 1, 1), 768, 2, SMALL), ("rys", (2, 2, 1, 1), 769, 2, COLUMNS),
         ("rys", (3, 2, 2, 0), 256, 2, SMALL), ("rys", (3, 2, 2, 0), 257, 2, TABLE), ("rys", (3, 2, 2, 0), 769, 2, COLUMNS),
         ("rys", (2, 0, 3, 2), 257, 2, TABLE), ("rys", (1, 1, 2, 2), 768, 2, SMALL),
         ("rys", (3, 3, 2, 0), 257, 2, COLUMNS), ("rys", (3, 2, 3, 2), 512, 1, SMALL), ("rys", (3, 2, 3, 2), 513, 1, COLUMNS),
         ("rys32", (3, 2, 3, 2), 1024, 1, SMALL), ("rys32", (2, 2, 1, 1), 1024, 2, SMALL),
         ("rys32", (2, 2, 1, 1), 1025, 2, COLUMNS), ("rys32", (3, 0, 2, 2), 1024, 2, TABLE),
         ("rys32", (3, 3, 2, 0), 1025, 2, COLUMNS), ("rys32", (3, 2, 1, 0), 8193, 2, COLUMNS), ("rys32", (0, 1, 3, 3), 700, 2, TABLE),
         ("rys32", (3, 2, 1, 0), 1025, 2, TABLE), ("rys32", (3, 1, 2, 1), 257, 1, COLUMNS)]


@pytest.mark.parametrize("precision,L,n,k,tag", CASES)
def test_kernel_of_a_launch(precision, L, n, k, tag):
    from paper_2303_13632_amd import eri
    plan = eri.Plan(*W.random_class_quartets(*L, n, 7 * n + sum(L) + k, k_fixed=k), precision=precision, bits=16)
    cid = int(np.flatnonzero(plan.class_quartets)[0])
    assert plan.class_tag[cid] == tag
    res = []
    for v in (0, int(plan.class_n_variants[cid]) - 1):
        var = np.zeros(256, np.int32)
        var[cid] = v
        plan.set_variants(var)
        out = [t.zero_() for t in plan.alloc(eri=True)]
        plan.compute(*out)
        torch.cuda.synchronize()
        res.append(out)
    assert plan.class_tag[cid] == TABLE
    for got, ref in zip(*res):
        assert torch.equal(got, ref)
