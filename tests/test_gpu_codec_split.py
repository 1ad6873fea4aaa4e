"""Standalone compress / decompress over the splits that the number of blocks and
their sizes choose: 4, 8 or 16 blocks a workgroup, four small blocks a wavefront
(in quarters, side by side) or one after the other, wavefronts and workgroups
whose last blocks are missing."""
import numpy as np
import pytest

import oracle as O
from paper_2303_13632_amd import eri

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SIZES = {
    "quarters": [0, 1, 2, 3, 4, 5, 7, 36, 57, 59, 60],
    "side by side": [1, 60, 61, 64, 81, 100, 216, 249, 251, 252],
    "mixed": [0, 1, 9, 60, 61, 252, 253, 300, 324],
}
LARGE = [2043, 2044, 2045, 2047, 2553, 2556, 2557, 4087, 4088, 4089, 8191, 8192, 8193, 8195, 10240, 10243, 5121, 1281]


@pytest.mark.parametrize("bits,shift", [(16, 0), (16, 1), (8, 2), (32, 0), (5, 3)])
@pytest.mark.parametrize("kind", sorted(SIZES))
@pytest.mark.parametrize("blocks", [1, 3, 6, 131, 16383, 16384, 16389, 65536, 65549])
def test_splits(blocks, kind, bits, shift):
    """Bit for bit the oracle's compressor; values code * eps exactly."""
    rng = np.random.default_rng(blocks + bits + shift)
    sizes = rng.choice(SIZES[kind], size=blocks)
    if kind == "mixed":
        at = rng.choice(blocks, size=min(blocks, len(LARGE)), replace=False)
        sizes[at] = LARGE[:len(at)]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    n = int(off[-1])
    x = rng.normal(size=n) * np.repeat(10.0 ** rng.integers(-320, 5, size=blocks), sizes)   # 1/eps overflows in some
    dx = torch.zeros(n + 8, dtype=torch.float64, device="cuda")[shift:shift + n]
    dx.copy_(torch.from_numpy(x))
    doff = torch.from_numpy(off).cuda()
    codes = torch.full((n + 8,), 1, dtype=eri.code_dtype(bits), device="cuda")
    scales = torch.full((blocks + 8,), 3.0, dtype=torch.float64, device="cuda")
    out = torch.full((n + 8,), 7.0, dtype=torch.float64, device="cuda")
    c, s = codes[shift:shift + n], scales[:blocks]
    eri.compress(bits, dx, doff, codes=c, scales=s)
    v = eri.decompress(bits, c, s, doff, out=out[shift:shift + n])
    torch.cuda.synchronize()
    oc, oe = O.compress(bits, x, off)
    assert np.array_equal(c.cpu().numpy().astype(np.int64), oc.astype(np.int64))
    assert np.array_equal(s.cpu().numpy(), oe)
    assert np.array_equal(v.cpu().numpy(), O.decompress(oc, oe, off))
    for t, fill in ((codes, 1), (out, 7.0)):
        assert (t[:shift] == fill).all() and (t[shift + n:] == fill).all()
    assert (scales[blocks:] == 3.0).all()
