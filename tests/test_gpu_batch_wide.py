"""Batched matvec of fields wider than 32 bits: rows of one and of several pieces
of 64 columns, odd and even numbers of rows for the four waves, alone (no buffers
for tiles in the launch) and beside narrower ones.  Equal to the oracle's."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SHAPES = [(1, 1), (1, 64), (4, 3), (5, 64), (8, 63), (9, 64), (130, 17), (1, 65), (3, 127),
          (7, 128), (8, 129), (300, 65), (2, 8192), (140, 333)]


@pytest.mark.parametrize("b", [33, 40, 48, 57, 63, 64])
@pytest.mark.parametrize("mixed", [False, True])
def test_wide_fields(b, mixed):
    import paper_1303_0270_amd as c
    rng = np.random.default_rng(600 + b)
    mats, xs = [], []
    for t, (rows, cols) in enumerate(SHAPES):
        bits = 1 + (t * 5) % 32 if mixed and t % 3 == 0 else b
        signed = bits == 64 or (bool(t % 2) and rows * cols > 1)
        lo, hi = (-(1 << (bits - 1)), (1 << (bits - 1)) - 1) if signed else (0, (1 << bits) - 1)
        a = rng.integers(lo, hi, size=(rows, cols), endpoint=True, dtype=np.int64)
        a.reshape(-1)[0], a.reshape(-1)[-1] = lo, hi
        mats.append(a)
        xs.append(rng.integers(-(1 << 31), 1 << 31, size=cols))
    packed = [c.compress(torch.from_numpy(a).cuda()) for a in mats]
    ys = [torch.full((m.rows,), 7, dtype=torch.int64, device="cuda") for m in packed]
    xd = [torch.from_numpy(x).to(torch.int32).cuda() for x in xs]
    batch = c.Batch(packed)
    batch.set_io(xd, ys)
    batch.run()
    dyn = c.batch.DynBatch(max_mats=32, max_items=4096, slots=2)
    ys2 = [torch.full((m.rows,), 7, dtype=torch.int64, device="cuda") for m in packed]
    dyn.matvec(packed, xd, ys2)
    torch.cuda.synchronize()
    for a, x, y, y2 in zip(mats, xs, ys, ys2):
        want = oracle.matvec(oracle.compress(a), x)
        assert np.array_equal(y.cpu().numpy(), want), a.shape
        assert np.array_equal(y2.cpu().numpy(), want), a.shape
    batch.close()
    dyn.close()
