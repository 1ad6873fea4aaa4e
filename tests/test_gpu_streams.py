"""eri_compute launches its classes on side streams: the same bits as class by
class on one stream, whichever stream the caller uses, from several threads,
and while the call is captured into a graph."""
import threading

import numpy as np
import pytest

from paper_2303_13632_amd import eri, workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _list_plan(seed, bits=16, n=40):
    parts = [W.random_class_quartets(*W.class_of(c), n, seed * 1000 + c) for c in range(0, 256, 7)]
    return eri.Plan(*W.merge(parts), bits=bits)


def _molecule_plan(seed, **kw):
    sh = W.molecule_basis(n_heavy=2, n_h=4, lattice=(3, 2, 1), seed=seed)
    return eri.Plan(sh, None, bits=16, schwarz=1e-10, **kw)


def _by_class(plan):
    out = [t.zero_() for t in plan.alloc(eri=True)]
    for c in range(256):
        if plan.class_quartets[c]:
            plan.compute_class(c, *out)
    torch.cuda.synchronize()
    return [t.cpu().numpy() for t in out]


def _same(got, ref):
    return all(np.array_equal(g.cpu().numpy(), r) for g, r in zip(got, ref))


@pytest.mark.parametrize("make", [_list_plan, _molecule_plan], ids=["list", "screened"])
def test_streams_and_threads(make):
    plans = [make(s) for s in (11, 12, 13)]
    refs = [_by_class(p) for p in plans]
    outs = [[t.zero_() for t in p.alloc(eri=True)] for p in plans]
    torch.cuda.synchronize()
    # results are complete for work ordered on the caller's stream behind the call
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        plans[0].compute(*outs[0])
        copies = [t.clone() for t in outs[0]]
    plans[1].compute(*outs[1])          # the default stream, while the first may still run
    stream.synchronize()
    assert _same(copies, refs[0])
    torch.cuda.synchronize()
    assert _same(outs[1], refs[1])
    failures = []

    def work(k):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            for _ in range(20):
                for t in outs[k]:
                    t.zero_()
                plans[k].compute(*outs[k])
            s.synchronize()
        if not _same(outs[k], refs[k]):
            failures.append(k)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failures


def test_captured():
    """A captured call keeps to the captured stream; its replays, with eager
    calls between them, give the eager bits."""
    plan, other = _list_plan(21), _list_plan(22)
    ref, ref2 = _by_class(plan), _by_class(other)
    out = [t.zero_() for t in plan.alloc(eri=True)]
    out2 = other.alloc(eri=True)
    plan.compute(*out)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        plan.compute(*out)
    for _ in range(3):
        for t in out:
            t.zero_()
        g.replay()
        other.compute(*out2)
        torch.cuda.synchronize()
        assert _same(out, ref) and _same(out2, ref2)


@pytest.mark.parametrize("chunk", [7, 300, 4096, 0])
def test_screened_pieces(chunk):
    """Launch pieces of a screened plan that cut its entries anywhere: every
    slot as in one piece, through eri_compute and eri_compute_noalloc."""
    whole = _molecule_plan(31)
    ref = _by_class(whole)
    small = _molecule_plan(31, chunk_quartets=chunk)
    out = [t.zero_() for t in small.alloc(eri=True)]
    small.compute(*out)
    torch.cuda.synchronize()
    assert _same(out, ref)
    for t in out:
        t.zero_()
    small.compute_noalloc(*out)
    torch.cuda.synchronize()
    assert _same(out, ref)
