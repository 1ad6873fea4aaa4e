"""The work that is timed: what a program that uses this package has it do.

Every case is one pass through the public entry points of
paper_2303_13632_amd.eri on inputs of paper_2303_13632_amd.workloads, with the
plan and the output buffers in hand, as a program that calls the pass again and
again keeps them.  Five paths, each over the range of sizes it is used at:

  list      Plan over a list of quartets, compute(): one class, every class, or
            the mixture of classes of a fragment; every precision, code width
            and output form
  screened  Plan over all Schwarz-screened quartets of a molecule-like basis,
            compute() into codes
  gradient  reverse mode: ERIFunction over a list (forward and backward), or
            backward() with a density over a screened basis
  packed    compute() into the packed n-bit stream, then unpack() to FP64
  recode    compress() and decompress() of FP64 blocks that are already there
"""
import math

import numpy as np
import torch

from paper_2303_13632_amd import eri
from paper_2303_13632_amd import workloads as W

DEVICE = 0


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------
def _list(classes, n, k=0, precision="fp64", bits=16, tune=False):
    """classes: four angular momenta ("0000"), "all" for every class, or
    "fragment"; n: quartets per class (fragment: shells); k: primitives per
    shell, 0 = drawn from 1..3."""
    return {"path": "list", "classes": classes, "n": n, "k": k, "precision": precision, "bits": bits, "tune": tune}


def listed():
    return [
        # the smallest calls: one launch of the cheapest class ...
        dict(_list("0000", 4096, k=3), name="ssss-4k"),
        # ... and the unique quartets of ten shells, s to f: a few quartets in each of many classes
        dict(_list("fragment", 10), name="fragment-10-shells"),
        # one class at a time, as a program that walks a molecule class by class asks for it: middle and high
        # angular momentum
        dict(_list("1111", 65536), name="pppp-64k"),
        dict(_list("2222", 16384), name="dddd-16k"),
        dict(_list("3333", 8192), name="ffff-8k"),
        # every class of s to f shells in one plan, tuned, FP64 values
        dict(_list("all", 1024, bits=0, tune=True), name="all-classes-1k-fp64-out"),
        # the same with the Rys kernels, coded
        dict(_list("all", 256, precision="rys"), name="all-classes-256-rys"),
        # direct and semi-direct SCF: all integrals of a molecule, coded and kept
        {"name": "molecule-48-atoms", "path": "screened", "nx": 4, "ny": 4, "nz": 3, "bits": 16},
        # forces on a small molecule and its exponent gradients
        {"name": "gradient-24-atoms", "path": "gradient", "form": "density", "nx": 4, "ny": 3, "nz": 2, "shells": 0,
         "n": 0},
        # a differentiable loss of a few integrals
        {"name": "gradient-list-256", "path": "gradient", "form": "list", "nx": 0, "ny": 0, "nz": 0, "shells": 12,
         "n": 256},
        # the paper's 12-bit stream written, then read back
        {"name": "packed-12-bits", "path": "packed", "n": 256, "bits": 12},
        # values from elsewhere coded and decoded, blocks of every class's size
        {"name": "recode-128k-blocks", "path": "recode", "blocks": 131072, "bits": 16},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["class", "class", "class", "fragment", "all", "screened", "density", "dl", "packed", "recode"])
    bits = rng.choice([16, 16, 16, 8, 12, 24, 32])
    precision = rng.choice(["fp64", "fp64", "fp64", "mixed", "rys", "rys32"])
    if kind == "class":
        cls = [rng.randrange(4) for _ in range(4)]
        n_eri = math.prod((l + 1) * (l + 2) // 2 for l in cls)
        return _list("".join(map(str, cls)), _log(rng, 1, min(65536, 80_000_000 // n_eri)), rng.choice([0, 0, 1, 3, 5]),
                     precision, rng.choice([bits, bits, 0]))
    if kind == "fragment":
        return _list("fragment", rng.randint(3, 12), 0, precision, bits)
    if kind == "all":
        return _list("all", _log(rng, 3, 256), 0, precision, bits)
    if kind in ("screened", "density"):
        nx, ny = rng.randint(2, 4), rng.randint(1, 3 if kind == "density" else 4)
        nz = rng.randint(1, 2 if kind == "density" else 3)
        if kind == "screened":
            return {"path": "screened", "nx": nx, "ny": ny, "nz": nz, "bits": bits}
        return {"path": "gradient", "form": "density", "nx": nx, "ny": ny, "nz": nz, "shells": 0, "n": 0}
    if kind == "dl":
        return {"path": "gradient", "form": "list", "nx": 0, "ny": 0, "nz": 0, "shells": rng.randint(4, 24),
                "n": _log(rng, 8, 4096)}
    if kind == "packed":
        return {"path": "packed", "n": _log(rng, 3, 256), "bits": rng.randint(2, 32)}
    return {"path": "recode", "blocks": _log(rng, 64, 131072), "bits": rng.randint(2, 32)}


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _redraw(shells, seed, exp_range):
    """The shell set with other exponents (log-uniform, per shell) and coefficients: the angular momenta, the depths
    of contraction and so the sizes of every output stay."""
    rng = np.random.default_rng(seed)
    lo, hi = (np.repeat(np.broadcast_to(r, len(shells["K"])), shells["K"]) for r in exp_range)
    exps = np.exp(rng.uniform(np.log(lo), np.log(hi)))
    return dict(shells, exps=exps, coefs=rng.uniform(0.1, 1.0, size=len(exps)))


def _shells(n, lmax, seed):
    """n shells in a box of 4 Bohr."""
    shells = dict(W.random_shells(n, lmax=lmax, box=4.0), xyz=np.random.default_rng(seed).uniform(0.0, 4.0, (n, 3)))
    return _redraw(shells, seed + 1, (0.1, 100.0))


def _unique(n):
    """Unique quartets of n shells (a >= b, c >= d, ab >= cd)."""
    pairs = [(a, b) for a in range(n) for b in range(a + 1)]
    return np.array([p + r for i, p in enumerate(pairs) for r in pairs[:i + 1]], dtype=np.int32)


def _quartets(case, seed):
    """(shells, quartets) of an explicit list."""
    if case["path"] == "gradient":
        q = np.random.default_rng(case["n"]).integers(0, case["shells"], size=(case["n"], 4))
        return _shells(case["shells"], 2, seed), q.astype(np.int32)
    classes = case.get("classes", "all")
    if classes == "fragment":
        return _shells(case["n"], 3, seed), _unique(case["n"])
    k = case.get("k", 0)
    kw = {"k_fixed": k} if k else {}
    if classes == "all":
        return W.merge([W.random_class_quartets(*W.class_of(c), case["n"], seed * 1000 + c, **kw) for c in range(256)])
    return W.random_class_quartets(*(int(x) for x in classes), case["n"], seed, **kw)


def _basis(case, seed):
    """Molecule-like basis on nx x ny x nz sites, a third of them heavy (the exponents of their shells reach 5000)."""
    sites = case["nx"] * case["ny"] * case["nz"]
    heavy = list(range(0, sites, 3))
    shells = W.molecule_basis(n_heavy=len(heavy), n_h=sites - len(heavy),
                              lattice=(case["nx"], case["ny"], case["nz"]), heavy_sites=heavy)
    move = np.random.default_rng(seed).uniform(-0.3, 0.3, size=(sites, 3))
    shells = dict(shells, xyz=shells["xyz"] + move[shells["atom"]])
    return _redraw(shells, seed + 1, (0.1, np.where(shells["atom"] % 3 == 0, 5000.0, 100.0)))


def _plan(case, seed):
    path = case["path"]
    if path == "screened" or case.get("form") == "density":
        return eri.Plan(_basis(case, seed), None, bits=case.get("bits", 0), device=DEVICE)
    shells, quartets = _quartets(case, seed)
    return eri.Plan(shells, quartets, precision=case.get("precision", "fp64"),
                    bits=0 if path == "gradient" else case["bits"], device=DEVICE, packed=path == "packed")


def _blocks(case):
    """Block sizes of the recode path: the n_ERIQ of random classes."""
    rng = np.random.default_rng(case["blocks"])
    n = np.array([1, 3, 6, 10])
    return np.prod(n[rng.integers(0, 4, size=(case["blocks"], 4))], axis=1)


def _device():
    return torch.device("cuda", DEVICE)


def _unpack_offsets(plan):
    """block_off and word_off (device) of a packed plan's stream, one block per quartet."""
    sizes = np.repeat([W.ncart(a) * W.ncart(b) * W.ncart(c) * W.ncart(d) for a, b, c, d in map(W.class_of, range(256))],
                      plan.class_quartets)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    words = eri.packed_word_offsets(plan.bits, off)
    return torch.from_numpy(off).to(_device()), torch.from_numpy(words).to(_device())


def prepare(case, seed):
    path = case["path"]
    s = {"path": path, "case": case}
    if path == "recode":
        sizes = _blocks(case)
        s["off"] = torch.from_numpy(np.concatenate([[0], np.cumsum(sizes)])).to(_device())
        g = torch.Generator(device=_device()).manual_seed(seed)
        n, blocks = int(sizes.sum()), len(sizes)
        # values of a quartet: one magnitude (1 Ha down to 1e-8) times components of either sign
        scale = torch.exp(-18.0 * torch.rand(blocks, generator=g, device=_device(), dtype=torch.float64))
        s["values"] = torch.randn(n, generator=g, device=_device(), dtype=torch.float64)
        s["values"] *= torch.repeat_interleave(scale, torch.from_numpy(sizes).to(_device()))
        s["codes"] = torch.empty(n, dtype=eri.code_dtype(case["bits"]), device=_device())
        s["scales"] = torch.empty(blocks, dtype=torch.float64, device=_device())
        s["decoded"] = torch.empty(n, dtype=torch.float64, device=_device())
        return s
    plan = s["plan"] = _plan(case, seed)
    if path == "gradient" and case["form"] == "density":
        s["density"] = torch.from_numpy(W.random_density(plan.nbf, seed=seed + 1)).to(_device())
    elif path == "gradient":
        s["centres"] = torch.tensor(plan.shells["xyz"], device=_device())
        s["exps"] = torch.tensor(plan.shells["exps"], device=_device())
        g = torch.Generator(device=_device()).manual_seed(seed + 1)
        s["dl"] = 2.0 * torch.rand(plan.out_values, generator=g, device=_device(), dtype=torch.float64) - 1.0
    else:
        s["eri"], s["codes"], s["scales"] = plan.alloc(eri=plan.bits == 0, codes=plan.bits > 0)
        if path == "screened":
            # a program that follows a geometry keeps buffers with room for every unique quartet
            L = [int(x) for x in plan.shells["L"]]
            pair = [W.ncart(a) * W.ncart(b) for i, a in enumerate(L) for b in L[:i + 1]]
            room, quartets = (sum(pair) ** 2 + sum(x * x for x in pair)) // 2, len(pair) * (len(pair) + 1) // 2
            s["codes"] = torch.zeros(room, dtype=s["codes"].dtype, device=_device())
            s["scales"] = torch.zeros(quartets, dtype=torch.float64, device=_device())
        if case.get("tune"):
            plan.tune(sample_quartets=1024, trials=2)
        if path == "packed":
            s["off"], s["words"] = _unpack_offsets(plan)
    return s


def run(s):
    case, path = s["case"], s["path"]
    if path == "recode":
        eri.compress(case["bits"], s["values"], s["off"], s["codes"], s["scales"])
        eri.decompress(case["bits"], s["codes"], s["scales"], s["off"], s["decoded"])
        return s["codes"], s["scales"], s["decoded"]
    plan = s["plan"]
    if path == "gradient" and case["form"] == "density":
        return plan.backward(density=s["density"])
    if path == "gradient":
        centres, exps = s["centres"].clone().requires_grad_(True), s["exps"].clone().requires_grad_(True)
        values = eri.ERIFunction.apply(centres, exps, plan)
        values.backward(s["dl"])
        return values.detach(), centres.grad, exps.grad
    plan.compute(s["eri"], s["codes"], s["scales"])
    if path == "packed":
        _, values = eri.unpack(case["bits"], s["codes"], s["off"], s["words"], s["scales"], codes=False, values=True)
        return s["codes"], s["scales"], values
    return (s["eri"],) if plan.bits == 0 else (s["codes"], s["scales"])


def work(case):
    """Bytes: the pair and primitive-pair tables and the gradient's inputs read once, the outputs written once.
    FLOPs: the plan's algorithmic count; a gradient needs at least the recurrences and, backwards through them, as
    much again for each of their two inputs."""
    if case["path"] == "recode":
        n = int(_blocks(case).sum())
        wide = 1 if case["bits"] <= 8 else 2 if case["bits"] <= 16 else 4
        return {"bytes": n * (8 + wide) + case["blocks"] * 16 + n * (wide + 8) + case["blocks"] * 16, "flops": 4 * n}
    plan = _plan(case, 0)
    read = 56 * plan.n_pairs + 96 * plan.n_prim_pairs
    flops = float(plan.class_flops.sum())
    if case["path"] == "gradient":
        out = 8 * (3 * len(plan.shells["L"]) + plan.n_prims)
        return {"bytes": read + out + (8 * plan.nbf ** 2 if case["form"] == "density" else 24 * plan.n_eri),
                "flops": 3 * flops}
    out = plan.n_eri * (plan.code_bytes or 8) + (8 * plan.n_quartets if plan.bits else 0)
    if case["path"] == "packed":
        packed = 64 * int(plan.class_word_off[256]) + 8 * plan.n_quartets
        out = 2 * packed + 8 * plan.n_eri
    return {"bytes": read + out, "flops": flops}


# ---------------------------------------------------------------------------
# The same outputs in 64 bits, in torch alone: McMurchie-Davidson (Hermite
# Gaussians), batched over the primitive quartets of a class.  Only the places
# of the values (which quartet comes where) are asked of the plan.
# ---------------------------------------------------------------------------
def _comps(L):
    return [(x, y, L - x - y) for x in range(L, -1, -1) for y in range(L - x, -1, -1)]


def _boys(T, n):
    """F_0..F_n(T) as a list, each with its first derivative -F_{m+1} (the top one included)."""
    with torch.no_grad():
        t = T.detach()
        near, x = t < 1.0, t.clamp(min=1.0)
        a = n + 1.5
        top = torch.special.gammainc(torch.full_like(x, a), x) * math.gamma(a) / (2.0 * x ** a)
        small, term = torch.zeros_like(t), torch.ones_like(t) / (2 * n + 3)
        y = t.clamp(max=1.0)
        for i in range(30):                        # e^-T sum (2T)^i / ((2n+3)(2n+5)...)
            small = small + term
            term = term * 2.0 * y / (2 * n + 5 + 2 * i)
        F = [torch.where(near, small * torch.exp(-y), top)]
        for m in range(n, -1, -1):
            F.insert(0, (2.0 * t * F[0] + torch.exp(-t)) / (2 * m + 1))
    return [F[m] - F[m + 1] * (T - t) for m in range(n + 1)]


def _hermite(la, lb, p, pa, pb):
    """E[i][j] = [E_0, .., E_{i+j}] of one axis (the Gaussian product's factor apart)."""
    h = 0.5 / p
    E = [[None] * (lb + 1) for _ in range(la + 1)]

    def up(e, x):
        out = []
        for t in range(len(e) + 1):
            v = x * e[t] if t < len(e) else 0.0
            if t > 0:
                v = v + h * e[t - 1]
            if t + 1 < len(e):
                v = v + (t + 1) * e[t + 1]
            out.append(v)
        return out

    E[0][0] = [torch.ones_like(p)]
    for i in range(la + 1):
        if i:
            E[i][0] = up(E[i - 1][0], pa)
        for j in range(1, lb + 1):
            E[i][j] = up(E[i][j - 1], pb)
    return E


def _expand(la, lb, p, PA, PB, place):
    """[n, ncart(la) * ncart(lb), len(place)] Hermite expansion of a primitive pair."""
    E = [_hermite(la, lb, p, PA[:, x], PB[:, x]) for x in range(3)]
    zero = torch.zeros_like(p)
    rows = []
    for a in _comps(la):
        for b in _comps(lb):
            ex, ey, ez = (E[x][a[x]][b[x]] for x in range(3))
            rows.append(torch.stack([ex[t] * ey[u] * ez[v] if t < len(ex) and u < len(ey) and v < len(ez) else zero
                                     for t, u, v in place], dim=1))
    return torch.stack(rows, dim=1)


def _hermite_coulomb(L, rho, PQ):
    """R_tuv, t + u + v <= L, as [n, count] and the place of each (t, u, v)."""
    F = _boys(rho * (PQ * PQ).sum(1), L)
    R = {(0, 0, 0): [(-2.0 * rho) ** m * F[m] for m in range(L + 1)]}
    place = [(t, u, s - t - u) for s in range(L + 1) for t in range(s + 1) for u in range(s - t + 1)]
    for k in place[1:]:
        ax = max(range(3), key=lambda x: k[x])
        low = tuple(k[x] - (x == ax) for x in range(3))
        lower = tuple(k[x] - 2 * (x == ax) for x in range(3))
        R[k] = [PQ[:, ax] * R[low][m + 1] + (low[ax] * R[lower][m + 1] if low[ax] else 0.0)
                for m in range(L + 1 - sum(k))]
    return torch.stack([R[k][0] for k in place], dim=1), {k: i for i, k in enumerate(place)}


def _class_values(L, sh, q, chunk):
    """Values [len(q), n_ERIQ] of quartets q of one class; sh: L, K, off (numpy) and xyz, exps, coefs (torch)."""
    la, lb, lc, ld = L
    K = sh["K"][q].astype(np.int64)
    counts = K.prod(axis=1)
    owner = np.repeat(np.arange(len(q)), counts)
    rest = np.arange(len(owner)) - np.repeat(np.cumsum(counts) - counts, counts)
    prim = []
    for s in (3, 2, 1, 0):
        prim.insert(0, sh["off"][q[owner, s]] + rest % K[owner, s])
        rest = rest // K[owner, s]
    dev = sh["xyz"].device
    bra = [(t, u, s - t - u) for s in range(la + lb + 1) for t in range(s + 1) for u in range(s - t + 1)]
    ket = [(t, u, s - t - u) for s in range(lc + ld + 1) for t in range(s + 1) for u in range(s - t + 1)]
    sign = torch.tensor([(-1.0) ** sum(k) for k in ket], dtype=torch.float64, device=dev)
    out = torch.zeros(len(q), math.prod(W.ncart(l) for l in L), dtype=torch.float64, device=dev)
    for lo in range(0, len(owner), chunk):
        own = owner[lo:lo + chunk]
        to = torch.from_numpy(own).to(dev)
        A, B, C, D = (sh["xyz"][torch.from_numpy(q[own, s].astype(np.int64)).to(dev)] for s in range(4))
        idx = [torch.from_numpy(x[lo:lo + chunk]).to(dev) for x in prim]
        a, b, c, d = (sh["exps"][i] for i in idx)
        p, r = a + b, c + d
        f = 1.0
        for l, e, i in zip(L, (a, b, c, d), idx):
            odd = math.prod(range(2 * l - 1, 0, -2))
            f = f * sh["coefs"][i] * (2.0 * e / math.pi) ** 0.75 * (4.0 * e) ** (0.5 * l) / math.sqrt(odd)
        f = f * torch.exp(-a * b / p * ((A - B) ** 2).sum(1) - c * d / r * ((C - D) ** 2).sum(1))
        f = f * 2.0 * math.pi ** 2.5 / (p * r * torch.sqrt(p + r))
        P, Q = (a[:, None] * A + b[:, None] * B) / p[:, None], (c[:, None] * C + d[:, None] * D) / r[:, None]
        R, at = _hermite_coulomb(sum(L), p * r / (p + r), P - Q)
        both = torch.tensor([[at[tuple(x + y for x, y in zip(k, m))] for m in ket] for k in bra], device=dev)
        left = _expand(la, lb, p, P - A, P - B, bra) * f[:, None, None]
        right = (_expand(lc, ld, r, Q - C, Q - D, ket) * sign).transpose(1, 2).contiguous()
        v = torch.bmm(torch.bmm(left, R[:, both]), right)
        out = out.index_add(0, to, v.reshape(len(own), -1))
    return out


def _torch_shells(shells):
    t = {k: torch.tensor(np.asarray(shells[k]), dtype=torch.float64, device=_device())
         for k in ("xyz", "exps", "coefs")}
    return dict(t, K=np.asarray(shells["K"]), off=np.asarray(shells["off"]), L=np.asarray(shells["L"]))


def _cost(q, shells):
    """Rough FLOPs of the torch evaluation of quartets q."""
    L, K = shells["L"][q].astype(np.float64), shells["K"][q].astype(np.float64)
    nb, nk = L[:, 0] + L[:, 1], L[:, 2] + L[:, 3]
    hb, hk = (nb + 1) * (nb + 2) * (nb + 3) / 6, (nk + 1) * (nk + 2) * (nk + 3) / 6
    n = (L + 1) * (L + 2) / 2
    return float((K.prod(1) * (3e4 + 2 * n[:, 0] * n[:, 1] * hk * (hb + n[:, 2] * n[:, 3]))).sum())


def _plan_order(plan):
    """(class, quartets in the order of the outputs) for every class of the plan."""
    return [(c, plan.class_quartet_list(c)) for c in range(256) if plan.class_quartets[c]]


def exact(case, seed):
    if case["path"] == "recode":
        s = prepare(case, seed)
        sizes = _blocks(case)
        # the largest magnitude of every block (padded rows in groups of one size), over the top code
        off, top = s["off"][:-1], torch.empty(len(sizes), dtype=torch.float64, device=_device())
        for n in np.unique(sizes):
            i = torch.from_numpy(np.flatnonzero(sizes == n)).to(_device())
            top[i] = s["values"][off[i, None] + torch.arange(n, device=_device())].abs().amax(1)
        eps = top / (2 ** (case["bits"] - 1) - 1)
        e = torch.repeat_interleave(eps, torch.from_numpy(sizes).to(_device()))
        x = s["values"] / e
        return None, eps, torch.sign(x) * torch.floor(x.abs() + 0.5) * e
    plan = _plan(case, seed)
    grad = case["path"] == "gradient"
    order = _plan_order(plan) if plan.n_quartets <= 2_000_000 else None
    if order is None or sum(_cost(q, plan.shells) for _, q in order) * (8 if grad else 1) > 2e13:
        return None
    sh = _torch_shells(plan.shells)
    if grad:
        return _exact_gradient(case, seed, plan, order, sh)
    values, scales = [], []
    for c, q in order:
        L = W.class_of(c)
        n_eri, m = math.prod(W.ncart(l) for l in L), sum(L)
        v = _class_values(L, sh, q, max(16, int(4e8 / (8 * (3 * n_eri + 40 * (m + 1) ** 3)))))
        if plan.bits:
            scales.append(v.abs().amax(1) / (2 ** (plan.bits - 1) - 1))
        else:
            values.append(v.reshape(-1))
    if plan.bits:
        eps = torch.cat(scales)
        if case["path"] == "screened":
            room = len(plan.shells["L"]) * (len(plan.shells["L"]) + 1) // 2
            eps = torch.cat([eps, eps.new_zeros(room * (room + 1) // 2 - len(eps))])
        return (None, eps, None) if case["path"] == "packed" else (None, eps)
    return (torch.cat(values),)


def _exact_gradient(case, seed, plan, order, sh):
    s = prepare(case, seed)
    centres, exps = sh["xyz"].requires_grad_(True), sh["exps"].requires_grad_(True)
    first = np.concatenate([[0], np.cumsum([W.ncart(int(l)) for l in plan.shells["L"]])])
    gc, ge = torch.zeros_like(centres), torch.zeros_like(exps)
    energy, at, values = 0.0, 0, []
    for c, q in order:
        L = W.class_of(c)
        n = [W.ncart(l) for l in L]
        step = max(1, int(2e6 / (math.prod(n) + 20 * (sum(L) + 1) ** 3)))
        for lo in range(0, len(q), step):
            part = q[lo:lo + step]
            v = _class_values(L, sh, part, 1 << 30)
            if case["form"] == "list":
                bar = s["dl"][at:at + v.numel()].reshape(v.shape)
                values.append(v.detach().reshape(-1))
                at += v.numel()
            else:
                f = [torch.from_numpy(first[part[:, x]][:, None] + np.arange(n[x])).to(_device()) for x in range(4)]
                left = s["density"][f[0][:, :, None], f[1][:, None, :]].reshape(len(part), -1)
                right = s["density"][f[2][:, :, None], f[3][:, None, :]].reshape(len(part), -1)
                a, b, x, y = (part[:, k] for k in range(4))
                same = ((a == x) & (b == y)) | ((a == y) & (b == x))
                w = (1.0 + (a != b)) * (1.0 + (x != y)) * (1.0 + ~same)
                bar = left[:, :, None] * right[:, None, :]
                bar = bar.reshape(v.shape) * torch.from_numpy(w).to(_device())[:, None]
            loss = (v * bar).sum()
            dc, de = torch.autograd.grad(loss, (centres, exps))
            gc, ge, energy = gc + dc, ge + de, energy + loss.detach()
    if case["form"] == "list":
        return torch.cat(values), gc, ge
    return gc, ge, energy.reshape(1)
