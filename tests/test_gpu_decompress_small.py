"""Decompression with two elements a lane (up to 2^20 elements) and in groups
above it: every width, around the pairs, the blocks and the line."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("b", range(1, 65))
def test_round_trip(b):
    import paper_1303_0270_amd as c
    rng = np.random.default_rng(700 + b)
    for t, (rows, cols) in enumerate([(1, 1), (1, 2), (3, 1), (7, 73), (16, 32), (19, 27),
                                      (1024, 1024), (1, (1 << 20) + 1), (1025, 1024)]):
        signed = bool(t % 2) or b == 64
        lo, hi = (-(1 << (b - 1)), (1 << (b - 1)) - 1) if signed else (0, (1 << b) - 1)
        a = rng.integers(lo, hi, size=(rows, cols), endpoint=True, dtype=np.int64)
        a.flat[-1], a.flat[0] = lo, hi
        m = c.compress(torch.from_numpy(a).cuda())
        assert a.size == 1 or m.bits == b
        out = torch.full((rows * cols + 2,), 7, dtype=torch.int64, device="cuda")
        c.decompress(m, out[:-2].view(rows, cols))
        got = out.cpu().numpy()
        assert np.array_equal(got[:-2].reshape(rows, cols), a) and (got[-2:] == 7).all()
