"""C = A B on the matrix cores for operands wider than a byte (several
base-256 digits per value), at the widths where the digit counts change and
the sizes where tiles, digit groups and K steps end, byte for byte against the
oracle."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def ccm():
    import paper_1303_0270_amd as c
    return c


def bounds(b, signed):
    return (-(1 << (b - 1)), (1 << (b - 1)) - 1) if signed else (0, (1 << b) - 1)


def rand_matrix(rng, rows, cols, b, signed):
    """Uniform over the width, with both extremes present."""
    lo, hi = bounds(b, signed)
    a = rng.integers(lo, hi, size=(rows, cols), endpoint=True, dtype=np.int64)
    a.flat[0] = hi
    a.flat[-1] = lo if signed else hi
    return a


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def assert_product(A, B, **kw):
    c = ccm()
    ga, gb = c.compress(dev(A)), c.compress(dev(B))
    want = oracle.matmul(oracle.compress(A), oracle.compress(B))
    got = c.matmul(ga, gb, **kw)
    assert got.header() == oracle.header(want)
    assert got.payload_bytes() == want.payload_bytes()
    return ga, gb, got


# (A width, signed, B width, signed): every digit count on both sides, each at
# a width that fills its top byte and one that only starts it, the offset
# digits of 8-, 16- and 24-bit unsigned fields, and pairs that need several
# passes (4 x 3, 4 x 4, 5 x 3, 7 x 1 and 8 x 1 digits)
PAIRS = [(8, False, 8, False), (8, False, 8, True), (7, False, 8, False), (9, False, 8, True),
         (8, True, 9, True), (15, False, 16, False), (16, True, 16, True), (17, False, 6, True),
         (3, False, 17, True), (16, False, 24, False), (24, True, 15, False),
         (23, False, 24, True), (24, False, 24, False), (25, False, 5, True),
         (32, False, 16, False), (31, True, 12, False), (4, True, 32, False),
         (12, False, 27, True), (32, True, 20, False), (20, True, 32, False),
         (30, False, 24, True), (28, True, 27, True), (36, True, 18, False),
         (20, False, 35, True), (54, True, 2, False), (2, True, 57, True), (57, True, 1, False)]
# K up to 96 takes the int64 path, longer products the matrix cores
SHAPES = [(1, 1, 1), (31, 96, 32), (1, 97, 1), (33, 129, 31), (97, 128, 130), (129, 127, 65),
          (260, 300, 200)]


@pytest.mark.parametrize("ba,sa,bb,sb", PAIRS)
def test_product_of_digits(ba, sa, bb, sb):
    rng = np.random.default_rng(100 * ba + bb)
    for M, K, N in SHAPES:
        if K * max(map(abs, bounds(ba, sa))) * max(map(abs, bounds(bb, sb))) < 1 << 63:
            assert_product(rand_matrix(rng, M, K, ba, sa), rand_matrix(rng, K, N, bb, sb))


@pytest.mark.parametrize("ba", range(1, 33))
def test_narrow_product_every_width(ba):
    """A narrow B of one digit: every width of A (32 bits goes the other way)
    in both signs, 1 to 129 columns, rows around a block and a wave, K around a
    step and split into parts."""
    rng = np.random.default_rng(3000 + ba)
    shapes = [(1, 1, 1), (33, 63, 2), (127, 129, 31), (129, 128, 33), (70, 257, 64), (40, 1030, 65),
              (130, 700, 128), (31, 64, 129)]
    for i, (M, K, N) in enumerate(shapes):
        sa, sb = bool((i + ba) % 2), bool(i % 3)
        bb = (1, 8, 4, 7)[(i + ba) % 4] if sb else (1, 7, 3, 8)[(i + ba) % 4]
        assert_product(rand_matrix(rng, M, K, ba, sa), rand_matrix(rng, K, N, bb, sb))


@pytest.mark.parametrize("ba,sa,bb,sb", [(8, False, 8, False), (16, True, 8, True),
                                         (9, True, 15, False), (17, False, 16, False)])
@pytest.mark.parametrize("K", [131071, 131072])
def test_longest_sums(ba, sa, bb, sb, K):
    """Every field at an extreme of its width over the longest K whose digit
    sums stay inside int32, and over the first one past it (int64 path)."""
    (alo, ahi), (blo, bhi) = bounds(ba, sa), bounds(bb, sb)
    A = np.empty((3, K), dtype=np.int64)
    A[0], A[1], A[2] = alo, ahi, np.where(np.arange(K) % 2, alo, ahi)
    B = np.empty((K, 2), dtype=np.int64)
    B[:, 0], B[:, 1] = blo, bhi
    assert_product(A, B)


def test_many_tiles_and_small_scratch():
    """Several output tiles in both directions, and the same product through
    the least scratch the C call accepts and through one off a 16-byte
    boundary (the int64 path): the same bytes."""
    rng = np.random.default_rng(77)
    A, B = rand_matrix(rng, 700, 260, 12, False), rand_matrix(rng, 260, 600, 10, True)
    ga, gb, want = assert_product(A, B)
    least_scratch(ga, gb, want)


def test_narrow_product_with_small_scratch():
    """The narrow product through the least scratch and a misaligned one."""
    rng = np.random.default_rng(78)
    A, B = rand_matrix(rng, 300, 520, 17, False), rand_matrix(rng, 520, 33, 6, True)
    least_scratch(*assert_product(A, B))


def least_scratch(ga, gb, want):
    c = ccm()
    least = c.matmul_scratch_least(ga, gb)
    full = c.matmul_scratch_bytes(ga, gb)
    assert least < full
    big = torch.empty(full + 64, dtype=torch.uint8, device="cuda")
    for scratch in (big[:least], big[8: 8 + full]):
        d = c._lib.Desc()
        import ctypes
        args = (ctypes.byref(ga.desc), ctypes.byref(gb.desc))
        s = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
        p = ctypes.c_void_p(scratch.data_ptr())
        assert c.lib.ccm_matmul_plan(*args, ctypes.byref(d), p, scratch.numel(), s) == 0
        m = c.CMatrix(d)
        assert c.lib.ccm_matmul(*args, ctypes.byref(m.desc), p, scratch.numel(), s) == 0
        assert m.header() == want.header() and m.payload_bytes() == want.payload_bytes()
