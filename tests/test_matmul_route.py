"""Which way a product of operands past int8 takes: through its operands' digits
(its scratch is then larger than the least that is accepted) or the int64 path.
Host logic only, and the same bytes on the two sides of the line on the GPU."""
import ctypes

import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")


def desc(rows, cols, bits):
    import paper_1303_0270_amd as c
    d = c._lib.Desc()
    d.rows, d.cols, d.vmin, d.vmax = rows, cols, 0, (1 << bits) - 1
    d.bits, d.is_signed, d.words = bits, 0, c.words(rows, cols, bits)
    return d


def by_digits(m, k, n, ba, bb):
    import paper_1303_0270_amd as c
    a, b = desc(m, k, ba), desc(k, n, bb)
    args = (ctypes.byref(a), ctypes.byref(b))
    return c.lib.ccm_matmul_scratch_bytes(*args) > c.lib.ccm_matmul_scratch_least(*args)


# us measured by the int64 path and by digits beside each
@pytest.mark.parametrize("m,k,n,ba,bb", [
    (1 << 20, 4, 4, 12, 12),      # 149 1566
    (1 << 20, 64, 10, 31, 9),     # 305 2525
    (100000, 200, 10, 12, 12),    # 116 194
    (100000, 32, 300, 20, 6),     # 101 226
    (1 << 20, 16, 64, 12, 6),     # 172 392, the narrow form
    (10000, 32, 4096, 24, 24),    # 166 256
    (1000, 32, 128, 12, 6),       # 23 33
    (1000, 97, 128, 8, 8),        # 38 52
    (1100, 1, 1100, 12, 12),      # 40 54 with the packing
])
def test_short_sums_take_int64(m, k, n, ba, bb):
    assert not by_digits(m, k, n, ba, bb)


@pytest.mark.parametrize("m,k,n,ba,bb", [
    (1500, 2000, 1801, 12, 10), (10000, 10001, 33, 17, 6), (100, 200, 10, 12, 12),
    (100000, 1000, 10, 12, 12), (100, 100, 2, 20, 7), (1792, 128, 1792, 9, 16),
    (10000, 300, 300, 31, 9), (1000, 500, 100, 40, 8),
])
def test_long_sums_take_digits(m, k, n, ba, bb):
    assert by_digits(m, k, n, ba, bb)


@pytest.mark.gpu
@pytest.mark.parametrize("ba,bb,signed", [(12, 12, True), (8, 8, False), (31, 9, False),
                                          (40, 8, True), (20, 6, True)])
def test_both_sides_of_the_line(ba, bb, signed):
    """K on both sides of the line at two heights, and the tile edges of the
    digits' side."""
    import paper_1303_0270_amd as c
    rng = np.random.default_rng(ba)
    ways = set()
    for m, k, n in [(97, 64, 130), (97, 161, 130), (129, 255, 65), (260, 65, 3), (31, 193, 257),
                    (5000, 127, 5), (5000, 513, 5), (3000, 65, 40), (257, 130, 129)]:
        lo, hi = (-(1 << (bb - 1)), (1 << (bb - 1)) - 1) if signed else (0, (1 << bb) - 1)
        A = rng.integers(0, 1 << ba, size=(m, k), dtype=np.int64)
        B = rng.integers(lo, hi, size=(k, n), endpoint=True, dtype=np.int64)
        A[0, 0], B[0, 0], B[-1, -1] = (1 << ba) - 1, lo, hi
        ga, gb = (c.compress(torch.from_numpy(v).cuda()) for v in (A, B))
        ways.add(c.matmul_scratch_bytes(ga, gb) > c.matmul_scratch_least(ga, gb))
        want = oracle.matmul(oracle.compress(A), oracle.compress(B))
        got = c.matmul(ga, gb)
        assert got.header() == oracle.header(want), (m, k, n)
        assert got.payload_bytes() == want.payload_bytes(), (m, k, n)
    assert ways == {False, True}
