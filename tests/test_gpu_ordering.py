"""Calls of one plan that follow each other without a synchronisation: each
gives what it gives alone, on whichever streams they are."""
import numpy as np
import pytest

from paper_2303_13632_amd import eri, workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DELAY = 20_000_000     # cycles that keep a stream busy: some milliseconds


def _list_shells(n=40, seed=5):
    return W.random_shells(10, lmax=2, seed=seed, box=3.0), \
        np.random.default_rng(seed).integers(0, 10, size=(n, 4)).astype(np.int32)


def _plan(kind):
    if kind == "screened":
        return eri.Plan(W.molecule_basis(n_heavy=1, n_h=3, lattice=(2, 2, 1), seed=9), None, bits=0)
    if kind == "long class":
        return eri.Plan(*W.random_class_quartets(1, 0, 0, 0, 2500, 6, k_choices=(1, 2)), bits=0)
    return eri.Plan(*_list_shells(), bits=0)


def _call(plan, kind, seed):
    """A closure that makes one pass on the current stream and returns its outputs."""
    rng = np.random.default_rng(seed)
    if kind == "screened":
        D = torch.tensor(W.random_density(plan.nbf, seed=seed), device="cuda")
        return lambda: plan.backward(density=D)
    if kind == "values":
        def values():
            out = plan.alloc(codes=False)[0].zero_()
            plan.compute(out)
            return (out,)
        return values
    dl = torch.tensor(rng.uniform(-1.0, 1.0, plan.out_values), device="cuda")
    return lambda: plan.backward(dl=dl)


def _near(got, ref):
    for g, r in zip(got, ref):
        assert (g - r).abs().max().item() <= 1e-11 * r.abs().max().item()


@pytest.mark.parametrize("kind", ["list", "screened", "long class", "values"])
def test_set_geometry_behind_the_calls_in_flight(kind):
    """set_geometry after a call on a stream of its own that has not run yet:
    the call is of the old geometry, the next one of the new."""
    plan = _plan(kind)
    call = _call(plan, kind, 3)
    x0 = np.asarray(plan.shells["xyz"]).copy()
    x1 = x0 + np.random.default_rng(4).uniform(-0.2, 0.2, x0.shape)
    refs = []
    for x in (x0, x1):
        plan.set_geometry(xyz=x)
        refs.append(call())
        torch.cuda.synchronize()
    assert (refs[0][0] - refs[1][0]).abs().max().item() > 1e-3 * refs[0][0].abs().max().item()
    plan.set_geometry(xyz=x0)
    stream = torch.cuda.Stream()
    got = []
    with torch.cuda.stream(stream):
        for x in (x1, x0, x1):
            torch.cuda._sleep(DELAY)
            got.append(call())
            plan.set_geometry(xyz=x)
    stream.synchronize()
    for g, r in zip(got, (refs[0], refs[1], refs[0])):
        _near(g, r)


@pytest.mark.parametrize("kind", ["list", "screened", "long class"])
def test_backward_on_two_streams(kind):
    """The adjoint's workspaces belong to the plan: calls on different streams take turns."""
    plan = _plan(kind)
    calls = [_call(plan, kind, s) for s in (11, 12)]
    refs = []
    for call in calls:
        refs.append(call())
        torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    got = []
    for i in range(8):
        with torch.cuda.stream(streams[i % 2]):
            got.append(calls[i % 2]())
    torch.cuda.synchronize()
    for i, g in enumerate(got):
        _near(g, refs[i % 2])
        assert torch.equal(g[2], refs[i % 2][2])


@pytest.mark.parametrize("form", ["screened", "scale blocks"])
def test_compute_on_two_streams(form):
    """Quartet items of a screened plan and staged values of scale blocks likewise."""
    if form == "screened":
        plan = eri.Plan(W.molecule_basis(n_heavy=2, n_h=4, lattice=(3, 2, 1), seed=13), None, bits=16, chunk_quartets=3000)
    else:
        plan = eri.Plan(*W.merge([W.random_class_quartets(*W.class_of(c), 300, c) for c in (0, 85, 98, 170)]), bits=16,
                        scale_block=5)
    ref = [t.zero_() for t in plan.alloc(eri=False)[1:]]
    plan.compute(None, *ref)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    outs = [[t.zero_() for t in plan.alloc(eri=False)[1:]] for _ in range(6)]
    torch.cuda.synchronize()
    for i, out in enumerate(outs):
        with torch.cuda.stream(streams[i % 2]):
            plan.compute(None, *out)
            if form == "screened":
                plan.compute_class(0, None, *out)
            else:
                plan.compute_noalloc(None, *out)
    torch.cuda.synchronize()
    for out in outs:
        assert all(torch.equal(o, r) for o, r in zip(out, ref))


def _many_classes(seed):
    return eri.Plan(*W.merge([W.random_class_quartets(*W.class_of(c), 60, seed * 1000 + c) for c in range(0, 256, 5)]), bits=16)


@pytest.mark.parametrize("form", ["list", "screened"])
def test_beside_a_capture(form):
    """While a stream is being captured (in the mode that forbids the whole
    process unsafe calls), calls on other streams leave the capture whole."""
    plan = _many_classes(1)
    other = _many_classes(2) if form == "list" else \
        eri.Plan(W.molecule_basis(n_heavy=2, n_h=4, lattice=(3, 2, 1), seed=17), None, bits=16)
    refs = []
    for p in (plan, other):
        out = [t.zero_() for t in p.alloc()]
        p.compute_noalloc(*out)          # class after class: the side streams are still to be made or free
        torch.cuda.synchronize()
        refs.append(out)
    out, out2 = ([t.zero_() for t in p.alloc()] for p in (plan, other))
    busy, aside = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, capture_error_mode="global"):
        plan.compute(*out)
        for stream in (busy, aside, busy):
            other.compute(*out2, stream=stream)
    for t in out:
        t.zero_()
    torch.cuda.synchronize()
    for _ in range(2):
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(o, r) for o, r in zip(out, refs[0]))
    assert all(torch.equal(o, r) for o, r in zip(out2, refs[1]))
