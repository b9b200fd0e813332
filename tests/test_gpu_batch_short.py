"""Batched matvec of matrices of few rows: tiles whose columns the waves of a block
share (up to two tiles an item), matrices of at most eight long rows of wide fields
on a kernel of their own, and items halved where the list leaves blocks idle.  Equal
to the oracle's."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def ccm():
    import paper_1303_0270_amd as c
    return c


def operands(rng, shapes, b):
    mats, xs = [], []
    for t, (rows, cols) in enumerate(shapes):
        signed = bool(t % 2) and rows * cols > 1
        lo, hi = (-(1 << (b - 1)), (1 << (b - 1)) - 1) if signed else (0, (1 << b) - 1)
        a = rng.integers(lo, hi, size=(rows, cols), endpoint=True, dtype=np.int64)
        a.reshape(-1)[0], a.reshape(-1)[-1] = lo, hi
        mats.append(a)
        r = 1 << (15 if t % 3 else 31)
        x = rng.integers(-r, r, size=cols)
        x[0], x[-1] = r - 1, -r
        xs.append(x)
    return mats, xs


def check(mats, xs, max_items=1 << 14):
    c = ccm()
    packed = [c.compress(torch.from_numpy(a).cuda()) for a in mats]
    xd = [torch.from_numpy(x).to(torch.int32).cuda() for x in xs]
    ys = [torch.full((m.rows,), 7, dtype=torch.int64, device="cuda") for m in packed]
    y2 = [torch.full((m.rows,), 7, dtype=torch.int64, device="cuda") for m in packed]
    batch = c.Batch(packed)
    batch.set_io(xd, ys)
    dyn = c.batch.DynBatch(max_mats=len(mats), max_items=max_items, slots=2)
    for graph in (False, True, True):
        for y in ys + y2:
            y.fill_(7)
        batch.run(use_graph=graph)
        dyn.matvec(packed, xd, y2)
        torch.cuda.synchronize()
        for a, x, got, got2 in zip(mats, xs, ys, y2):
            want = oracle.matvec(oracle.compress(a), x)
            assert np.array_equal(got.cpu().numpy(), want), (a.shape, graph)
            assert np.array_equal(got2.cpu().numpy(), want), (a.shape, "dyn")
    items = batch.info()["items"]
    batch.close()
    dyn.close()
    return items


@pytest.mark.parametrize("b", [1, 3, 4, 8, 12, 13, 16, 17, 20, 24, 25, 31, 32])
def test_few_rows(b):
    shapes = [(r, k) for r, k in zip((1, 2, 7, 8, 9, 15, 16, 17, 31, 32, 33, 1, 8, 9, 5, 16, 32, 3),
                                     (1, 127, 128, 129, 513, 1023, 640, 255, 1030, 8192, 2047, 1024,
                                      1055, 1024, 8191, 8192, 1300, 1023))]
    mats, xs = operands(np.random.default_rng(700 + b), shapes, b)
    check(mats, xs)


@pytest.mark.parametrize("shapes", [[(4, 1100)], [(8, 8192), (1, 1024)]])
def test_only_few_long_rows(shapes):
    """A list that leaves nothing for the tiles."""
    mats, xs = operands(np.random.default_rng(41), shapes, 24)
    assert check(mats, xs) == len(shapes)


def test_halved_items_stay_within_the_workspace():
    c = ccm()
    mats, xs = operands(np.random.default_rng(42), [(300, 8000)], 24)
    for room in (3, 4, 10, 64):  # 128 rows an item: 3 of them
        assert check(mats, xs, max_items=room) == 19  # halved three times: 16 rows
    packed = [c.compress(torch.from_numpy(a).cuda()) for a in mats]
    dyn = c.batch.DynBatch(max_mats=1, max_items=2, slots=2)
    y = torch.empty(300, dtype=torch.int64, device="cuda")
    with pytest.raises(c.CcmError):
        dyn.matvec(packed, [torch.from_numpy(xs[0]).to(torch.int32).cuda()], [y])
    dyn.close()
