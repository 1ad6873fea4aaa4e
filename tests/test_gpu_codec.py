"""Standalone compress / decompress at the edges of their work split: blocks
around one group of four values, around the size that one wavefront takes
(2556), around what a workgroup holds in registers (10240), empty blocks, and
arrays whose base is not aligned to a group."""
import numpy as np
import pytest

import oracle as O
from paper_2303_13632_amd import eri

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

EDGES = [1, 0, 2, 3, 4, 5, 7, 255, 256, 257, 1020, 1023, 1024, 1025, 1027, 2553, 2555, 2556,
         2557, 2559, 2560, 3600, 10000, 10236, 10239, 10240, 10241, 10243, 20001, 1, 1, 0]


@pytest.mark.parametrize("bits", [2, 8, 9, 16, 17, 32])
@pytest.mark.parametrize("shift", [0, 1, 3])
def test_edges(bits, shift):
    """Bit for bit the oracle's compressor; values code * eps exactly."""
    rng = np.random.default_rng(bits * 10 + shift)
    sizes = np.array(EDGES + list(rng.integers(1, 700, size=40)))
    off = np.zeros(len(sizes) + 1, dtype=np.int64)
    off[1:] = np.cumsum(sizes)
    n = int(off[-1])
    x = rng.normal(size=n) * np.repeat(10.0 ** rng.integers(-300, 5, size=len(sizes)), sizes)
    x[off[2]:off[3]] = 0.0
    whole = torch.zeros(n + 8, dtype=torch.float64, device="cuda")
    dx = whole[shift:shift + n]
    dx.copy_(torch.from_numpy(x))
    doff = torch.from_numpy(off).cuda()
    codes = torch.full((n + 8,), 1, dtype=eri.code_dtype(bits), device="cuda")
    out = torch.full((n + 8,), 7.0, dtype=torch.float64, device="cuda")
    c, s = eri.compress(bits, dx, doff, codes=codes[shift:shift + n])
    v = eri.decompress(bits, c, s, doff, out=out[shift:shift + n])
    torch.cuda.synchronize()
    oc, oe = O.compress(bits, x, off)
    assert np.array_equal(c.cpu().numpy().astype(np.int64), oc.astype(np.int64))
    assert np.array_equal(s.cpu().numpy(), oe)
    assert np.array_equal(v.cpu().numpy(), O.decompress(oc, oe, off))
    # nothing outside the blocks is written
    for t, fill in ((codes, 1), (out, 7.0)):
        assert (t[:shift] == fill).all() and (t[shift + n:] == fill).all()


def test_not_finite():
    """NaN does not count in the maximum and codes to 0; an infinite maximum
    gives codes 0 with an infinite scale."""
    x = np.array([np.nan, 1.0, -2.0, 0.5, np.inf, 3.0, -1.0, np.nan, np.nan])
    off = np.array([0, 4, 7, 9], dtype=np.int64)
    c, s = eri.compress(16, torch.from_numpy(x).cuda(), torch.from_numpy(off).cuda())
    c, s = c.cpu().numpy(), s.cpu().numpy()
    assert s[0] == 2.0 * (1.0 / 32767) and np.isinf(s[1]) and s[2] == 0.0
    assert list(c[:4]) == [0, 16384, -32767, 8192] and not c[4:].any()


def _tie_products(n, seed):
    """Pairs (b_max, x) at 16 bits whose product x * (1/eps) rounds to a half in
    FP64 while the exact product lies off it."""
    from fractions import Fraction
    rng = np.random.default_rng(seed)
    out = []
    while len(out) < n:
        b = rng.uniform(0.5, 2.0)
        inv = 1.0 / (b * (1.0 / 32767.0))
        h = float(rng.integers(0, 32766)) + 0.5
        x = h / inv
        if x * inv == h and Fraction(x) * Fraction(inv) != Fraction(h):
            out.append((b, x))
    return out


def test_products_that_round_to_a_half():
    """The code is the rounding of the rounded product (eq. 10), not of a fused
    one: half away from zero, bit for bit the oracle's."""
    pairs = _tie_products(3000, 3)
    x = np.array([v for b, y in pairs for v in (b, y, -y, 0.0)])
    off = np.arange(0, len(x) + 1, 4, dtype=np.int64)
    c, s = eri.compress(16, torch.from_numpy(x).cuda(), torch.from_numpy(off).cuda())
    oc, oe = O.compress(16, x, off)
    assert np.array_equal(s.cpu().numpy(), oe)
    assert np.array_equal(c.cpu().numpy().astype(np.int64), oc.astype(np.int64))
