"""The half-register kernels of the largest classes: which launches take them, by
contraction, size and outputs, and that codes and scales do not depend on it."""
import numpy as np
import pytest

from paper_2303_13632_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,n,k,bits,tag", [((3, 2, 3, 2), 2048, 2, 0, 2), ((3, 2, 3, 2), 2047, 2, 16, 0),
                                            ((3, 2, 3, 2), 8192, 1, 16, 0), ((3, 2, 3, 2), 2048, 1, 0, 0),
                                            ((3, 3, 2, 2), 2048, 2, 0, 6), ((3, 3, 2, 2), 8191, 1, 16, 0),
                                            ((3, 3, 2, 2), 8192, 1, 16, 6), ((3, 3, 2, 2), 8192, 1, 0, 0),
                                            ((2, 2, 3, 3), 8192, 1, 12, 6)])
def test_kernel_of_a_launch(L, n, k, bits, tag):
    from paper_2303_13632_amd import eri
    plan = eri.Plan(*W.random_class_quartets(*L, n, 7 * n + sum(L) + k, k_fixed=k), bits=bits, packed=bits == 12)
    cid = int(np.flatnonzero(plan.class_quartets)[0])
    assert plan.class_tag[cid] == tag
    forms = [(True, 0), (False, 0)] if bits else [(True, 0)]
    for k in range(1, int(plan.class_n_variants[cid])):
        var = np.zeros(256, np.int32)
        var[cid] = k
        plan.set_variants(var)
        if plan.class_tag[cid] in (2, 6):
            forms.append((True, k))
    assert len(forms) > (2 if bits else 1)
    res = []
    for values, k in forms:
        var = np.zeros(256, np.int32)
        var[cid] = k
        plan.set_variants(var)
        out = [t.zero_() if t is not None else None for t in plan.alloc(eri=values)]
        plan.compute(*out)
        torch.cuda.synchronize()
        res.append(out)
    for out in res[1:]:
        for got, ref in zip(res[0], out):
            assert got is None or ref is None or torch.equal(got, ref)
