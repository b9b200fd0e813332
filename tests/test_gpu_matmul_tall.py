"""Products with more rows than a launch of one block a row can hold (2^24 of 256
threads): the operands are generated on the device, sampled entries of C are
computed on the host from the generator's values."""
import numpy as np
import pytest

import ccm_workloads as W

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

ROWS = (1 << 24) + 5


# past int8 and within it, each with more columns than the narrow forms take (or,
# in the first, a B that they do not take)
@pytest.mark.parametrize("K,N,ba,bb", [(4, 4, 12, 12), (3, 257, 4, 4)])
def test_more_rows_than_blocks(K, N, ba, bb):
    import paper_1303_0270_amd as c
    sa = W.MatrixSpec(ROWS, K, -(1 << (ba - 1)), 1 << (ba - 1), W.seed_for(9, 0), 5)
    sb = W.MatrixSpec(K, N, -(1 << (bb - 1)), 1 << (bb - 1), W.seed_for(9, 0), 6)
    A, B = (c.generate(s.rows, s.cols, s.lo, s.hi, s.seed, s.stream) for s in (sa, sb))
    C = c.matmul(A, B)
    b = sb.dense()
    rng = np.random.default_rng(3)
    rows = np.concatenate([[0, 63, 64, (1 << 22) - 1, 65535 * 64, 1 << 23, (1 << 24) - 1, 1 << 24,
                            ROWS - 1], rng.integers(0, ROWS, 200)])
    want = np.concatenate([sa.rows_slice(int(r), int(r) + 1) @ b for r in rows])
    ii = np.repeat(rows, N)
    jj = np.tile(np.arange(N), len(rows))
    got, bad = c.gather(C, torch.from_numpy(ii).cuda(), torch.from_numpy(jj).cuda())
    assert not bad and np.array_equal(got.cpu().numpy(), want.reshape(-1))
    assert C.vmin <= want.min() and want.max() <= C.vmax
    del A, B, C
    torch.cuda.empty_cache()
