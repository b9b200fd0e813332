"""Compression in one pass at a guessed width: the bytes of the two-pass form at
every width, input type and block remainder, and wrong guesses (too narrow, too
wide, the other sign) found wherever the value that refutes them sits."""
import ctypes

import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def ccm():
    import paper_1303_0270_amd as c
    return c


def bounds(b, signed):
    return (-(1 << (b - 1)), (1 << (b - 1)) - 1) if signed else (0, (1 << b) - 1)


def rand_matrix(rng, rows, cols, b, signed):
    lo, hi = bounds(b, signed)
    a = rng.integers(lo, hi, size=(rows, cols), endpoint=True, dtype=np.int64)
    a.flat[0], a.flat[-1] = hi, lo if signed else hi
    return a


def tried(A, bits, signed, dtype, offset=0):
    """ccm_compress_try at the given guess; dense starts `offset` elements into
    its allocation."""
    c = ccm()
    rows, cols = A.shape
    store = torch.zeros(rows * cols + offset, dtype=dtype, device="cuda")
    t = store[offset:].view(rows, cols)
    t.copy_(torch.from_numpy(A))
    payload = torch.full((c.payload_capacity(rows, cols, bits),), 0xA5, dtype=torch.uint8,
                         device="cuda")
    d = c._lib.Desc()
    s = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    code = c._lib.I32 if dtype == torch.int32 else c._lib.I64
    rc = c.lib.ccm_compress_try(ctypes.c_void_p(t.data_ptr()), code, rows, cols, bits, int(signed),
                                ctypes.c_void_p(payload.data_ptr()), ctypes.byref(d), s)
    assert rc == 0
    return d, payload


# one group, a block of 128 or 256 groups and one element either side, several
SHAPES = [(1, 1), (3, 11), (1, 4095), (2, 2048), (1, 4097), (1, 8191), (2, 4096), (1, 8193),
          (71, 331)]


@pytest.mark.parametrize("signed", [False, True])
@pytest.mark.parametrize("b", range(1, 65))
def test_right_guess_every_width(b, signed):
    if b == 64 and not signed:
        return
    c = ccm()
    rng = np.random.default_rng(2 * b + signed)
    for i, (rows, cols) in enumerate(SHAPES):
        A = rand_matrix(rng, rows, cols, b, signed)
        ref = oracle.compress(A)
        if ref.bits != b:  # one element: a signed draw without its negative end
            continue
        types = [torch.int64] + ([torch.int32] if A.min() >= -2**31 and A.max() < 2**31 else [])
        for dt in types:
            d, payload = tried(A, b, signed, dt, offset=i % 2)
            assert d.payload == payload.data_ptr()
            m = c.CMatrix(d, payload)
            assert m.header() == oracle.header(ref) and m.payload_bytes() == ref.payload_bytes()
            assert not payload[8 * m.words:].any()  # zeros to the end of the capacity


@pytest.mark.parametrize("dtype", [torch.int64, torch.int32])
def test_wrong_guess(dtype):
    c = ccm()
    rng = np.random.default_rng(5)
    for rows, cols in ((5, 33), (300, 500)):
        n = rows * cols
        for v in (1 << 12, -1, -(1 << 20), (1 << 30) + 7) + (((1 << 50) + 1,) if dtype == torch.int64
                                                             else ()):
            for at in (0, n // 2, n - 1):
                A = rng.integers(0, 1 << 12, size=(rows, cols))
                A.flat[1] = (1 << 12) - 1
                A.flat[at] = v
                d, _ = tried(A, 12, False, dtype)
                assert not d.payload
                assert (d.vmin, d.vmax) == (A.min(), A.max())
                assert d.bits == oracle.compress(A).bits
        # too wide a guess
        A = rng.integers(0, 1 << 5, size=(rows, cols))
        d, _ = tried(A, 12, True, dtype)
        assert not d.payload and (d.vmin, d.vmax) == (A.min(), A.max())
    # the slots are armed again: the next pass is right
    m = c.compress(torch.from_numpy(A).cuda())
    assert m.payload_bytes() == oracle.compress(A).payload_bytes()


@pytest.mark.parametrize("dtype", [torch.int64, torch.int32])
def test_compress_takes_one_pass_or_two(dtype, monkeypatch):
    """compress() itself: a matrix whose sample has its width, and one whose
    only wide value the sample misses."""
    c = ccm()
    monkeypatch.setattr(c, "_ONEPASS_BYTES", 1 << 20)
    rng = np.random.default_rng(6)
    A = rng.integers(-(1 << 9), 1 << 9, size=(700, 1031))
    for wide in (None, (350, 517)):
        if wide:
            A[wide] = 1 << 25
        ref = oracle.compress(A)
        m = c.compress(torch.from_numpy(A).to(dtype).cuda())
        assert m.header() == oracle.header(ref) and m.payload_bytes() == ref.payload_bytes()


def test_refusals():
    c = ccm()
    t = torch.zeros(64, dtype=torch.int64, device="cuda")
    d = c._lib.Desc()
    p = ctypes.c_void_p(t.data_ptr())
    for dtype, bits, sg in ((0, 33, 0), (1, 65, 1), (1, 0, 0), (1, 64, 0)):
        assert c.lib.ccm_compress_try(p, dtype, 8, 8, bits, sg, p, ctypes.byref(d), None) == -1
    assert c.lib.ccm_compress_try(p, 1, 8, 8, 3, 0, None, ctypes.byref(d), None) == -1
    b = ctypes.c_int32()
    assert c.lib.ccm_compress_guess(p, 1, 0, ctypes.byref(b), ctypes.byref(b), None) == -1
