"""Fixed-point floats: ranges from the floats' own extremes, packing in one pass
at the scale and width of a sample, and decoding straight to floats, against
the oracle."""
import ctypes
import math

import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def ccm():
    import paper_1303_0270_amd as c
    return c


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def packed(v, f):
    return oracle.compress(oracle.quantize(v, f).reshape(v.shape))


def assert_matrix(m, v, f):
    ref = packed(v, f)
    assert m.frac_bits == f and m.bits == ref.bits
    assert (m.vmin, m.vmax) == (ref.vmin, ref.vmax)
    assert m.payload_bytes() == ref.payload_bytes()


# a group, blocks of 128 and 256 groups and one element either side
SHAPES = [(1, 1), (1, 31), (1, 4097), (2, 4096), (1, 8193), (67, 331)]


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("p", [1, 2, 7, 12, 29, 30, 31, 33, 52, 61])
def test_one_pass(dtype, p, monkeypatch):
    c = ccm()
    monkeypatch.setattr(c, "_ONEPASS_BYTES", 0)
    rng = np.random.default_rng(p)
    for rows, cols in SHAPES:
        for offset in (0, 1):
            v = np.ldexp(rng.uniform(-1, 1, (rows, cols)), int(rng.integers(-30, 30))).astype(dtype)
            if offset:
                v = np.abs(v)
            t = torch.zeros(v.size + offset, dtype=torch.from_numpy(v).dtype, device="cuda")
            t = t[offset:].view(rows, cols)  # off a 16-byte boundary for offset 1
            t.copy_(torch.from_numpy(v))
            m = c.compress_float(t, sig_bits=p)
            f = p - math.frexp(float(np.abs(v).max()))[1] if np.abs(v).max() else 0
            assert_matrix(m, v, f)
            for out in (np.float32, np.float64):
                got = c.decompress_float(m, torch.from_numpy(np.zeros(1, out)).dtype)
                q = oracle.quantize(v, f).reshape(-1)
                want = oracle.dequantize(q, f, out).reshape(v.shape)
                assert got.cpu().numpy().tobytes() == want.tobytes()


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_wrong_guess(dtype, monkeypatch):
    """A value the sample misses that changes the scale, the width or the sign."""
    c = ccm()
    monkeypatch.setattr(c, "_ONEPASS_BYTES", 0)
    rng = np.random.default_rng(9)
    base = rng.uniform(0.25, 0.75, (1100, 1031)).astype(dtype)
    for w in (9.0, -0.5, -300.0):
        for at in ((0, 5), (555, 300), (1099, 1030)):
            v = base.copy()
            v[at] = w
            m = c.compress_float(dev(v), sig_bits=10)
            assert_matrix(m, v, 10 - math.frexp(max(0.75, abs(w)) if abs(w) > 1 else
                                                float(np.abs(v).max()))[1])
            assert_matrix(c.compress_float(dev(v), frac_bits=7), v, 7)
    for w in (math.nan, -math.nan, math.inf, -math.inf):
        v = base.copy()
        v[700, 11] = w
        with pytest.raises(c.CcmError) as e:
            c.compress_float(dev(v), sig_bits=10)
        assert e.value.status == c.E_RANGE
        with pytest.raises(c.CcmError) as e:
            c.float_absmax(dev(v))
        assert e.value.status == c.E_RANGE
    v = base.copy()
    v[3, 3] = 2.0 ** 40
    with pytest.raises(c.CcmError) as e:
        c.compress_float(dev(v), frac_bits=22)
    assert e.value.status == c.E_OVERFLOW


@pytest.mark.parametrize("b", list(range(1, 64)))
def test_decode_every_width(b):
    """Packed integers of every width as floats, signed and unsigned."""
    c = ccm()
    rng = np.random.default_rng(b)
    for signed in (False, True):
        lo, hi = ((-(1 << (b - 1)), (1 << (b - 1)) - 1) if signed else (0, (1 << b) - 1))
        for rows, cols in SHAPES:
            a = rng.integers(lo, hi, size=(rows, cols), endpoint=True, dtype=np.int64)
            a.flat[0] = hi
            m = c.compress(dev(a))
            for f in (0, 13, -7, 1100):
                m.frac_bits = f
                for dt, nt in ((torch.float32, np.float32), (torch.float64, np.float64)):
                    got = c.decompress_float(m, dt).cpu().numpy()
                    want = oracle.dequantize(a.reshape(-1), f, nt).reshape(a.shape)
                    assert got.tobytes() == want.tobytes()


def test_column_major_and_stream():
    c = ccm()
    rng = np.random.default_rng(4)
    v = rng.standard_normal((37, 53))
    m = c.compress_float(dev(v), frac_bits=20)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    want = oracle.dequantize(oracle.quantize(v, 20).reshape(-1), 20, np.float64).reshape(v.shape)
    for stream in (None, s):
        t = c.decompress_float(m.T, torch.float64, stream=stream)
        torch.cuda.synchronize()
        assert t.is_contiguous() and np.array_equal(t.cpu().numpy(), want.T)


def test_quantized_range_host():
    c = ccm()
    lo, hi = ctypes.c_int64(), ctypes.c_int64()
    fn = c.lib.ccm_quantized_range
    assert fn(-2.5, 3.5, 0, ctypes.byref(lo), ctypes.byref(hi)) == 0
    assert (lo.value, hi.value) == (-2, 4)  # half to even
    assert fn(-1.0, 1.0, 62, ctypes.byref(lo), ctypes.byref(hi)) == c.E_OVERFLOW
    for bad in ((math.nan, 1.0, 0), (0.0, math.inf, 0), (2.0, 1.0, 0), (0.0, 1.0, 1201)):
        assert fn(*bad, ctypes.byref(lo), ctypes.byref(hi)) == c.E_INVAL
