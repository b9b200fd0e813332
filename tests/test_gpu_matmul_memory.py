"""Products where memory does not hold the full scratch: the least one serves, a
caller's own is used from the least size on, and one that is too small is replaced.
Allocations are made to fail by size, not by filling the GPU."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def product():
    import paper_1303_0270_amd as c
    rng = np.random.default_rng(21)
    A = rng.integers(0, 1 << 17, size=(300, 900))
    B = rng.integers(-32, 32, size=(900, 40))
    A[0, 0], B[0, 0], B[-1, -1] = (1 << 17) - 1, -32, 31
    ga, gb = (c.compress(torch.from_numpy(v).cuda()) for v in (A, B))
    need, least = c.matmul_scratch_bytes(ga, gb), c.matmul_scratch_least(ga, gb)
    assert least < need
    return c, ga, gb, oracle.matmul(oracle.compress(A), oracle.compress(B)), need, least


def same(got, want):
    assert got.header() == oracle.header(want) and got.payload_bytes() == want.payload_bytes()


def refuse(monkeypatch, refused):
    """torch.empty fails for byte tensors that refused(size) names."""
    real = torch.empty

    def empty(*size, **kw):
        if kw.get("dtype") == torch.uint8 and refused(size[0]):
            raise torch.cuda.OutOfMemoryError(f"refused: {size[0]}")
        return real(*size, **kw)

    monkeypatch.setattr(torch, "empty", empty)


def test_full_scratch_refused(product, monkeypatch):
    c, ga, gb, want, need, least = product
    refuse(monkeypatch, lambda n: n >= need)
    got, scratch = c.matmul_plan(ga, gb)
    assert scratch.numel() == least
    same(c.matmul_pack(ga, gb, got, scratch), want)
    same(c.matmul(ga, gb), want)
    same(c.matmul_async(ga, gb).get(), want)


def test_result_refused_beside_the_full_scratch(product, monkeypatch):
    c, ga, gb, want, need, least = product
    sizes = []

    def refused(n):
        sizes.append(n)
        return len(sizes) == 2  # the result's payload, once

    refuse(monkeypatch, refused)
    got, scratch = c.matmul_plan(ga, gb)
    assert sizes[0] == need and sizes[2] == scratch.numel() == least
    same(c.matmul_pack(ga, gb, got, scratch), want)


def test_nothing_left(product, monkeypatch):
    c, ga, gb, want, need, least = product
    refuse(monkeypatch, lambda n: True)
    for call in (c.matmul, c.matmul_async):
        with pytest.raises(torch.cuda.OutOfMemoryError):
            call(ga, gb)


@pytest.mark.parametrize("extra", [0, 1, 4096])
def test_callers_scratch_is_used(product, extra):
    c, ga, gb, want, need, least = product
    mine = torch.empty(least + extra, dtype=torch.uint8, device="cuda")
    got, scratch = c.matmul_plan(ga, gb, scratch=mine)
    assert scratch is mine
    same(c.matmul_pack(ga, gb, got, scratch), want)
    same(c.matmul_async(ga, gb, scratch=mine).get(), want)


def test_too_small_a_scratch_is_replaced(product):
    c, ga, gb, want, need, least = product
    mine = torch.empty(least - 1, dtype=torch.uint8, device="cuda")
    got, scratch = c.matmul_plan(ga, gb, scratch=mine)
    assert scratch.numel() == need
    same(c.matmul_pack(ga, gb, got, scratch), want)
