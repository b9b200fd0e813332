"""Products whose right operand is long enough for the wide tiles of its digit
transposition (256 and 128 columns of B), at ragged sizes and with the column
sums of digit offsets.  Sums stay below 2^53, so a float64 product is exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("bits,signed,n", [(1, False, 2048), (3, True, 2049), (4, True, 2303),
                                           (7, False, 2081), (8, False, 2100), (8, True, 2177),
                                           (9, False, 1030), (12, True, 1153), (16, False, 1101),
                                           (16, True, 1024), (20, False, 513)])
@pytest.mark.parametrize("k", [8192, 8070])
def test_wide_tiles(bits, signed, n, k):
    import paper_1303_0270_amd as c
    rng = np.random.default_rng(bits * 10000 + n + k)
    lo, hi = (-(1 << (bits - 1)), (1 << (bits - 1)) - 1) if signed else (0, (1 << bits) - 1)
    m = 130
    a = rng.integers(-128, 128, size=(m, k), dtype=np.int64)
    b = rng.integers(lo, hi, size=(k, n), endpoint=True, dtype=np.int64)
    a[0], a[1, ::2] = 127, -128
    b[:, 0], b[:, -1], b[-1] = hi, lo, hi
    A, B = (c.compress(torch.from_numpy(v).cuda()) for v in (a, b))
    got = c.decompress(c.matmul(A, B)).cpu().numpy()
    want = (a.astype(np.float64) @ b.astype(np.float64)).astype(np.int64)
    assert np.array_equal(got, want)
