"""Outer products (K = 1) of signed operands whose digits add up to six while
every entry fits 32 bits (a signed field of b bits may hold no magnitude past
2^(b-2)), on both sides of the bound where C is stored in 64, blocking and
asynchronous, byte for byte against the oracle."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def vector(rng, n, top, b):
    """Signed values of b bits, the largest magnitude `top` at both ends of the
    sign, the rest spread over their lengths."""
    assert 1 << (b - 2) <= top < 1 << (b - 1)
    v = rng.integers(-top, top, size=n, endpoint=True) >> rng.integers(0, b, size=n)
    v[0], v[-1] = top, -top
    return v.astype(np.int64)


# (A bits, B bits): 3 x 3, 4 x 2 and 2 x 4 digits
@pytest.mark.parametrize("ba,bb", [(17, 17), (25, 9), (9, 25)])
@pytest.mark.parametrize("fits", [True, False])
def test_outer_product(ba, bb, fits):
    import paper_1303_0270_amd as c
    rng = np.random.default_rng(10 * ba + bb + fits)
    bt = 5 << (bb - 4)
    at = ((1 << 31) - 1) // bt if fits else (1 << 31) // bt + 1
    assert (at * bt < 1 << 31) == fits
    A, B = vector(rng, 1100, at, ba).reshape(-1, 1), vector(rng, 1103, bt, bb).reshape(1, -1)
    ga, gb = (c.compress(torch.from_numpy(v).cuda()) for v in (A, B))
    assert (ga.bits, gb.bits) == (ba, bb)
    want = oracle.matmul(oracle.compress(A), oracle.compress(B))
    for got in (c.matmul(ga, gb), c.matmul_async(ga, gb).get()):
        assert got.header() == oracle.header(want)
        assert got.payload_bytes() == want.payload_bytes()
