"""Batched matvec by tiles of 16 rows: every width at the edges of tiles, steps
and units, x in int16 and in all of int32, and work lists long enough for larger
items and for both ways that blocks get them.  Whole numbers: results are equal
to the oracle's."""
import json

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SHAPES = [(1, 1), (15, 31), (16, 32), (17, 127), (63, 128), (64, 129), (65, 255), (130, 257),
          (33, 512), (16, 513), (5, 1030), (80, 97), (1, 8192), (50, 640)]


def ccm():
    import paper_1303_0270_amd as c
    return c


def fields(rng, rows, cols, b, signed):
    lo, hi = ((-(1 << (b - 1)), (1 << (b - 1)) - 1) if signed else (0, (1 << b) - 1))
    a = rng.integers(lo, hi, size=(rows, cols), endpoint=True, dtype=np.int64)
    a[rng.integers(0, 3, size=a.shape) == 0] = hi
    a.reshape(-1)[0] = lo
    a.reshape(-1)[-1] = hi
    return a


def run(mats, xs, **kw):
    c = ccm()
    packed = [c.compress(torch.from_numpy(a).cuda()) for a in mats]
    batch = c.Batch(packed, **kw)
    ys = [torch.full((m.rows,), 7, dtype=torch.int64, device="cuda") for m in packed]
    batch.set_io([torch.from_numpy(x).to(torch.int32).cuda() for x in xs], ys)
    items = batch.info()["items"]
    for graph in (False, True, True):
        for y in ys:
            y.fill_(7)
        batch.run(use_graph=graph)
        torch.cuda.synchronize()
        for a, x, y in zip(mats, xs, ys):
            want = oracle.matvec(oracle.compress(a), x)
            assert np.array_equal(y.cpu().numpy(), want), (a.shape, graph)
    batch.close()
    return items


@pytest.mark.parametrize("b", range(1, 34))
def test_tiles_of_every_width(b):
    rng = np.random.default_rng(900 + b)
    mats, xs = [], []
    for t, (rows, cols) in enumerate(SHAPES):
        mats.append(fields(rng, rows, cols, b, bool(t % 2) and rows * cols > 1))
        r = 1 << (15 if t % 3 else 31)
        x = rng.integers(-r, r, size=cols)
        x[0], x[-1] = r - 1, -r
        xs.append(x)
    run(mats, xs)


@pytest.mark.parametrize("tile_rows", [1, 5])
def test_long_lists_take_larger_items(tmp_path, tile_rows):
    rng = np.random.default_rng(940 + tile_rows)
    table = tmp_path / "tune.json"
    table.write_text(json.dumps({"widths": {str(b): {"tile_rows": tile_rows}
                                            for b in range(1, 65)}}))
    mats = [fields(rng, 1000 * tile_rows, int(rng.integers(1, 40)), b, False)
            for b in (1, 3, 4, 9, 12, 17, 25, 32, 33, 40)]
    xs = [rng.integers(-(1 << 31), 1 << 31, size=a.shape[1]) for a in mats]
    items = run(mats, xs, tune_json=str(table))
    assert items == 250 * len(mats)  # 10000 of tile_rows would be four or more a block
