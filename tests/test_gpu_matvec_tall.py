"""y = A x of narrow matrices on both sides of the rows that a launch of a wave a
row can hold (2^26 of 64 threads): generated on the device, sampled rows computed
on the host from the generator's values."""
import numpy as np
import pytest

import ccm_workloads as W

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [(1 << 26) - 4, (1 << 26) - 3, (1 << 26) + 5])
@pytest.mark.parametrize("dtype", [torch.int32, torch.int64])
def test_more_rows_than_waves(rows, dtype):
    import paper_1303_0270_amd as c
    spec = W.MatrixSpec(rows, 3, -2, 2, W.seed_for(9, 0), 7)
    A = c.generate(rows, 3, spec.lo, spec.hi, spec.seed, spec.stream)
    x = np.array([7, -100003, (1 << 31) - 1])
    y = torch.full((rows,), -1, dtype=torch.int64, device="cuda")
    c.matvec(A, torch.from_numpy(x).to(dtype).cuda(), y=y)
    rng = np.random.default_rng(4)
    at = np.concatenate([[0, 1, (1 << 24) - 1, 1 << 24, (1 << 26) - 5, rows - 1],
                         rng.integers(0, rows, 300)])
    want = np.array([spec.rows_slice(int(r), int(r) + 1)[0] @ x for r in at])
    assert np.array_equal(y[torch.from_numpy(at).cuda()].cpu().numpy(), want)
    del A, y
    torch.cuda.empty_cache()
