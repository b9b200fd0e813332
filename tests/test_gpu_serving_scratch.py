"""The serving loop's matmul scratch: one per stream, within the stream's share of
the arena where the products' full scratch is larger than that, with the same
results."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tight", [False, True])
def test_scratch_stays_within_the_arena(tight):
    import paper_1303_0270_amd as c
    from paper_1303_0270_amd import serve
    pool = [c.generate(200, 3000, 0, 1 << 17, 5, 1), c.generate(100, 500, 0, 1 << 6, 5, 2)]
    reqs = []
    for i in range(12):
        a = pool[i % 2]
        b = c.generate(a.cols, 40 + i, -32, 32, 6, 10 + i)
        reqs.append(serve.Request(i, "mm", i % 2, 0.0, b=b))
    full = max(c.matmul_scratch_bytes(pool[r.mat], r.b) for r in reqs)
    least = max(c.matmul_scratch_least(pool[r.mat], r.b) for r in reqs)
    arena = max(serve.request_footprint(r, pool) for r in reqs) if tight else 1 << 30
    assert least < arena // 2 and (full > arena // 2) == tight
    srv = serve.Server(pool, arena_bytes=arena, streams=2, max_inflight=4)
    sizes = [s.numel() for s in srv._prepare(reqs)]
    assert sizes == [arena // 2 if tight else full] * 2
    srv.run(reqs)
    srv.close()
    for r in reqs:
        want = c.matmul(pool[r.mat], r.b)
        assert r.c.header() == want.header() and r.c.payload_bytes() == want.payload_bytes()
