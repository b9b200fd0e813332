"""Products with at most 64 columns of one digit: the tile of 16 rows a block, its
blocks of 16 columns and the waves' steps of K at their edges, one part of K and
several, four waves a block and eight, and an int8 pair whose scratch has no room
for whole blocks of columns.  Bit exact against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

EDGES = [(1, 128, 15), (15, 129, 16), (16, 1023, 17), (17, 1024, 32), (40, 1025, 47),
         (33, 513, 48), (16, 2100, 49), (9, 300, 63), (70, 1152, 64)]


def bounds(b, signed):
    return (-(1 << (b - 1)), (1 << (b - 1)) - 1) if signed else (0, (1 << b) - 1)


def values(rng, rows, cols, b, signed):
    lo, hi = bounds(b, signed)
    a = rng.integers(lo, hi, size=(rows, cols), endpoint=True, dtype=np.int64)
    a[rng.integers(0, 4, size=a.shape) == 0] = lo
    a.flat[0], a.flat[-1] = hi, lo if signed else hi
    return a


def check(A, B):
    import paper_1303_0270_amd as c
    ga, gb = (c.compress(torch.from_numpy(v).cuda()) for v in (A, B))
    for _ in range(2):
        got = c.matmul(ga, gb)
        want = oracle.matmul(oracle.compress(A), oracle.compress(B))
        assert got.header() == oracle.header(want)
        assert got.payload_bytes() == want.payload_bytes(), (A.shape, B.shape)


@pytest.mark.parametrize("signed", [False, True])
@pytest.mark.parametrize("ba", [1, 2, 3, 4, 7, 8, 9, 12, 16, 17, 20, 24, 25, 31])
def test_edges(ba, signed):
    rng = np.random.default_rng(60 + ba)
    for t, (m, k, n) in enumerate(EDGES):
        bb, sb = ((8, True), (5, False), (1, True), (7, False))[t % 4]
        check(values(rng, m, k, ba, signed), values(rng, k, n, bb, sb))


@pytest.mark.parametrize("ba,m,k,n", [(6, 8193, 140, 20), (17, 8200, 257, 33), (25, 8192, 130, 50)])
def test_tall(ba, m, k, n):
    rng = np.random.default_rng(ba + m)
    check(values(rng, m, k, ba, True), values(rng, k, n, 6, True))


@pytest.mark.parametrize("m,k,n", [(1, 130, 1), (2, 500, 3), (5, 1000, 9), (14, 257, 2)])
def test_int8_pair_with_little_room(m, k, n):
    rng = np.random.default_rng(m)
    check(values(rng, m, k, 7, True), values(rng, k, n, 7, True))
