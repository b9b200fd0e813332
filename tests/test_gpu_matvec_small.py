"""y = A x and A^T x with an element per lane (small and narrow matrices) at the
edges of its loops, and the kernels above the line where it ends.  Whole numbers: equal
to the oracle's, modulo 2^64."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

WIDTHS = (1, 2, 3, 4, 7, 8, 12, 15, 16, 17, 24, 31, 32, 33, 47, 48, 63, 64)


def matrix(rng, rows, cols, b, signed):
    if b == 64:
        lo, hi = -(1 << 63), (1 << 63) - 1
    else:
        lo, hi = (-(1 << (b - 1)), (1 << (b - 1)) - 1) if signed else (0, (1 << b) - 1)
    a = rng.integers(lo, hi, size=(rows, cols), endpoint=True, dtype=np.int64)
    a.reshape(-1)[0] = hi
    a.reshape(-1)[-1] = lo if a.size > 1 else hi
    return a


def check(a, dtype, rng, transposed=False):
    import paper_1303_0270_amd as c
    m = c.compress(torch.from_numpy(a).cuda())
    r = 1 << (31 if dtype == torch.int32 else 62)
    x = rng.integers(-r, r, size=a.shape[0 if transposed else 1], dtype=np.int64)
    xd = torch.from_numpy(x).to(dtype).cuda()
    y = c.matvec_t(m, xd) if transposed else c.matvec(m, xd)
    with np.errstate(over="ignore"):
        want = ((a * x[:, None]).sum(axis=0, dtype=np.int64) if transposed
                else (a * x).sum(axis=1, dtype=np.int64))
    if a.size < 5000 and not transposed:
        assert np.array_equal(want, oracle.matvec(oracle.compress(a), x))
    assert np.array_equal(y.cpu().numpy(), want), (a.shape, m.bits, m.signed, dtype)


@pytest.mark.parametrize("dtype", [torch.int32, torch.int64])
@pytest.mark.parametrize("b", WIDTHS)
def test_small_and_narrow(b, dtype):
    rng = np.random.default_rng(1000 + b)
    shapes = [(1, 1), (5, 1), (3, 63), (4, 64), (9, 65), (6, 128), (7, 129), (2, 256), (3, 257),
              (4, 512), (5, 513), (2, 1024), (3, 1025), (5, 2049), (2, 4097), (2, 8192), (3, 8193),
              (1, 16384), (40, 7), (3001, 130), (20011, 60)]
    for t, (rows, cols) in enumerate(shapes):
        check(matrix(rng, rows, cols, b, bool(t % 2) or b == 64), dtype, rng)


@pytest.mark.parametrize("dtype", [torch.int32, torch.int64])
@pytest.mark.parametrize("b", WIDTHS)
def test_about_the_line(b, dtype):
    """Just below and above the sizes where the wider kernels take over: aligned
    and ragged rows, one column panel and several."""
    rng = np.random.default_rng(1100 + b)
    for t, (rows, cols) in enumerate([(1024, 1024), (1031, 1024), (1029, 1027), (1537, 1024),
                                      (1310, 1203), (530, 8064), (128, 16384), (70, 20011),
                                      (40, 32768), (40, 32771), (513, 3001)]):
        check(matrix(rng, rows, cols, b, bool(t % 2) or b == 64), dtype, rng)


@pytest.mark.parametrize("dtype", [torch.int32, torch.int64])
@pytest.mark.parametrize("b", WIDTHS)
def test_transposed(b, dtype):
    """As many rows as a wave, a block and one pass take, and one more or less;
    the last four on the two sides of the lines."""
    rng = np.random.default_rng(1200 + b)
    for t, (rows, cols) in enumerate([(1, 1), (3, 15), (4, 16), (5, 17), (31, 40), (32, 33),
                                      (33, 100), (64, 31), (65, 257), (511, 19), (513, 30),
                                      (1025, 21), (1536, 50), (1537, 50), (2561, 37), (600, 3600)]):
        check(matrix(rng, rows, cols, b, bool(t % 2) or b == 64), dtype, rng, transposed=True)
