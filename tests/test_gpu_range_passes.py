"""The range passes the host waits for (compress, get, add): block counts
around the slots they fold into, several threads and streams, and a refusal
under stream capture that leaves the next pass working."""
import threading

import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

# elements one block of the dense range pass takes
BLOCK = 4096


def ccm():
    import paper_1303_0270_amd as c
    return c


@pytest.mark.parametrize("dtype", [torch.int64, torch.int32])
@pytest.mark.parametrize("n", [1, 2, BLOCK, BLOCK + 1, 63 * BLOCK, 64 * BLOCK, 64 * BLOCK + 1,
                               65 * BLOCK, 129 * BLOCK + 7])
def test_extremes_at_either_end(n, dtype):
    c = ccm()
    for at in {0, n // 2, n - 1}:
        for v in (-(1 << 20), (1 << 21) + 3):
            t = torch.full((1, n), 5, dtype=dtype, device="cuda")
            t[0, at] = v
            m = c.compress(t)
            assert (m.vmin, m.vmax) == ((min(v, 5), max(v, 5)) if n > 1 else (v, v))
            assert c.get(m, 0, at) == v
            two = c.add(m, m)
            assert (two.vmin, two.vmax) == (2 * m.vmin, 2 * m.vmax)


def test_threads_and_streams():
    c = ccm()
    bad = []

    def work(i):
        s = torch.cuda.Stream()
        rng = np.random.default_rng(i)
        for k in range(20):
            A = rng.integers(-(1 << (3 + i)), 1 << (3 + i), size=(37 + 50 * k, 41 + i))
            pa = oracle.compress(A)
            with torch.cuda.stream(s):
                m = c.compress(torch.from_numpy(A).cuda())
                d = c.add(m, m)
                ok = m.header() == oracle.header(pa) and m.payload_bytes() == pa.payload_bytes()
                ok = ok and c.get(m, 3, 7) == A[3, 7] and d.vmax == 2 * m.vmax
            if not ok:
                bad.append((i, k))

    ts = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad


def test_refused_under_capture():
    c = ccm()
    A = torch.arange(6, dtype=torch.int64, device="cuda").view(2, 3)
    x = torch.zeros(4, device="cuda")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        x.add_(1)
        with pytest.raises(c.CcmError) as ei:
            c.compress(A)
    assert ei.value.status == -6  # CCM_E_DEVICE
    g.replay()
    assert x.tolist() == [1.0] * 4
    m = c.compress(A)
    assert (m.vmin, m.vmax) == (0, 5) and c.get(m, 1, 2) == 5
