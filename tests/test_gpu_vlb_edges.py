"""Method 2 compression at the edges of its passes: quads of four elements on and
off 16-byte boundaries, partial quads and groups, stretches of 128 groups, row
counts around the row scan's steps, and the columns around a wave's step within
a row, against the oracle."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def ccm():
    import paper_1303_0270_amd as c
    return c


def check(A, dtype=torch.int64, offset=0):
    c = ccm()
    t = torch.zeros(A.size + offset, dtype=dtype, device="cuda")[offset:].view(*A.shape)
    t.copy_(torch.from_numpy(A))
    g = c.vlb_compress(t)
    ref = oracle.vlb_compress(A)
    assert (g.vmin, g.vmax, g.k, g.nbits) == (ref.vmin, ref.vmax, ref.k, ref.nbits)
    assert np.array_equal(g.payload_words().numpy().view(np.uint64), ref.payload)
    assert not g.payload[8 * g.words:].cpu().numpy().any()
    starts = oracle.vlb_offsets(ref, 32).astype(np.int64)
    rb = g.row_bits().numpy()
    assert np.array_equal(rb[:-1], starts[:, 0]) and rb[-1] == ref.nbits
    assert np.array_equal(g.group_offsets().numpy(), starts - starts[:, :1])
    ends = np.append(starts.ravel()[1:], ref.nbits)
    assert g.gmax == int((ends - starts.ravel()).max())


def mixed(rng, rows, cols, top, signed):
    """Lengths uniform in 1..top: short pairs, pairs of 32 and 33 bits, and pairs
    past 64."""
    L = rng.integers(1, top + 1, size=(rows, cols))
    v = rng.integers(0, 1 << 62, size=(rows, cols)) & ((np.int64(1) << (L - 1)) - 1)
    v |= np.int64(1) << (L - 1)
    return v * rng.choice([-1, 1], size=v.shape) if signed else v


@pytest.mark.parametrize("dtype,top", [(torch.int64, 62), (torch.int64, 9), (torch.int32, 31)])
@pytest.mark.parametrize("cols", [1, 3, 4, 30, 31, 32, 33, 34, 36, 127, 128, 4095, 4096, 4100])
def test_columns(cols, dtype, top):
    rng = np.random.default_rng(cols + top)
    for rows in (1, 3, 9):
        for signed in (False, True):
            check(mixed(rng, rows, cols, top, signed), dtype, offset=rows % 2)


@pytest.mark.parametrize("rows", [127, 128, 129, 8191, 8192, 8193, 16385])
def test_rows(rows):
    rng = np.random.default_rng(rows)
    check(mixed(rng, rows, 5, 20, True))


def test_long_row():
    """Several steps of a wave along one row, two in the next."""
    rng = np.random.default_rng(3)
    check(mixed(rng, 2, 256 * 32 * 2 + 77, 13, False))
