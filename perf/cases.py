"""Performance cases: the work a program has this library do on one GPU, as
calls of the package's public functions.

A case is a dict of plain values.  ``prepare`` makes what the program holds
before the call (dense inputs, compressed operands, a batch), ``run`` is one
pass, ``work`` the bytes and operations that pass cannot do without: every
input read once, every output written once, packed matrices counted as their
packed bytes.

Operands that a program already holds in compressed form are drawn packed by
``generate``; dense integers and floats are drawn by torch from the seed.
"""
from __future__ import annotations

import math

import torch

import paper_1303_0270_amd as ccm

SWEEP_WIDTHS = (1, 3, 7, 12, 17, 31)


def listed():
    return [
        # The plain method on a small matrix, as a first program runs it: a
        # chain of calls of a few microseconds each, where launches, host waits
        # and marshalling count.
        {"name": "plain_256", "op": "plain", "rows": 256, "cols": 256, "bits": 10, "dtype": "int64"},
        # The bandwidth sweep: y = A x on 16384 x 16384 at six widths.
        {"name": "sweep_16384", "op": "sweep", "rows": 16384, "cols": 16384, "xbits": 16},
        # y = A x off every alignment, with an int64 x over more than 32 bits.
        {"name": "matvec_ragged_i64", "op": "matvec", "rows": 10007, "cols": 9973, "bits": 12,
         "signed": True, "xdtype": "int64", "xbits": 40},
        # y = A^T x (y = A x of a matrix unravelled by column).
        {"name": "matvec_t_7", "op": "matvec_t", "rows": 16384, "cols": 8192, "bits": 7,
         "signed": True, "xdtype": "int32", "xbits": 16},
        # Dense int64 values packed at the width of their own range, as data
        # come in; the largest read from dense memory.
        {"name": "compress_12", "op": "compress", "rows": 16384, "cols": 16384, "bits": 12,
         "signed": False, "dtype": "int64", "order": "C"},
        # A + B of two widths at a ragged shape, re-encoded at the width of the sums.
        {"name": "add_ragged", "op": "add", "rows": 12345, "cols": 6789, "bits": 12, "bits2": 7,
         "signed": True},
        # The dense compressed product, 6-bit by signed 4-bit, 8192^3.
        {"name": "matmul_8192", "op": "matmul", "m": 8192, "k": 8192, "n": 8192, "bits": 6,
         "signed": False, "bits2": 4, "signed2": True},
        # A served request's product: a pool matrix (widths up to 20) by a
        # narrow right operand of a few dozen columns and signed 1..8-bit values.
        {"name": "matmul_served", "op": "matmul", "m": 10000, "k": 10001, "n": 33, "bits": 17,
         "signed": False, "bits2": 6, "signed2": True},
        # A product of two matrices wider than a byte at a middling odd size.
        {"name": "matmul_wide", "op": "matmul", "m": 1500, "k": 2000, "n": 1801, "bits": 12,
         "signed": False, "bits2": 10, "signed2": False},
        # Thousands of matrices of 32..2048 rows and columns and widths 1..24,
        # one matvec each in one graph launch.
        {"name": "batch_4096", "op": "batch", "count": 4096, "lo": 32, "hi": 2048, "bits": 24},
        # Variable length blocks: short bit-lengths (Beta(1, 32)), compressed
        # from dense and multiplied.
        {"name": "vlb_short", "op": "vlb", "rows": 16384, "cols": 8192, "beta": 32.0,
         "signed": False},
        # Floats in fixed point: compressed to 12 significant bits, multiplied by
        # a float vector, and decoded back to float32.
        {"name": "float_12", "op": "float", "rows": 16384, "cols": 8192, "dtype": "float32",
         "sig_bits": 12, "x_sig_bits": 14},
    ]


# ---- drawn cases -----------------------------------------------------------

def _size(rng, lo, hi):
    """Spread over the logarithm of [lo, hi]; a third of the draws multiples of
    128, a third odd."""
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    kind = rng.randrange(3)
    if kind == 0 and n >= 128:
        n = n // 128 * 128
    elif kind == 1:
        n |= 1
    return max(lo, min(hi, n))


def _width(rng):
    return rng.randint(33, 62) if rng.random() < 0.08 else rng.randint(1, 32)


def draw(rng):
    op = rng.choice(("plain", "sweep", "matvec", "matvec", "matvec_t", "compress", "compress",
                     "add", "scale", "decompress", "matmul", "matmul", "served", "served",
                     "batch", "vlb", "float"))
    if op == "plain":
        return {"op": op, "rows": _size(rng, 32, 1024), "cols": _size(rng, 32, 1024),
                "bits": rng.randint(1, 16), "dtype": rng.choice(("int64", "int32"))}
    if op == "sweep":
        n = _size(rng, 1024, 16384)
        return {"op": op, "rows": n, "cols": _size(rng, 1024, 16384), "xbits": 16}
    if op in ("matvec", "matvec_t"):
        xd = rng.choice(("int32", "int32", "int64"))
        return {"op": op, "rows": _size(rng, 64, 16384), "cols": _size(rng, 64, 20000),
                "bits": _width(rng), "signed": rng.random() < 0.5, "xdtype": xd,
                "xbits": rng.choice((16, 31) if xd == "int32" else (16, 31, 40))}
    if op == "compress":
        return {"op": op, "rows": _size(rng, 64, 16384), "cols": _size(rng, 64, 16384),
                "bits": rng.randint(1, 31), "signed": rng.random() < 0.5,
                "dtype": rng.choice(("int64", "int32")), "order": rng.choice("CCCF")}
    if op == "add":
        b = rng.randint(1, 31)
        return {"op": op, "rows": _size(rng, 64, 16384), "cols": _size(rng, 64, 16384),
                "bits": b, "bits2": rng.choice((b, rng.randint(1, 31))),
                "signed": rng.random() < 0.5}
    if op in ("scale", "decompress"):
        return {"op": op, "rows": _size(rng, 64, 16384), "cols": _size(rng, 64, 16384),
                "bits": rng.randint(1, 31), "signed": rng.random() < 0.5,
                "by": rng.randint(2, 99)}
    if op == "matmul":
        b, b2 = rng.randint(1, 16), rng.randint(1, 16)
        top = 4096 if b <= 7 and b2 <= 7 else 1792
        return {"op": op, "m": _size(rng, 48, top), "k": _size(rng, 48, top),
                "n": _size(rng, 48, top), "bits": b, "signed": rng.random() < 0.5,
                "bits2": b2, "signed2": rng.random() < 0.5}
    if op == "served":
        m = _size(rng, 100, 10000)
        return {"op": "matmul", "m": m, "k": m + rng.randint(0, 1), "n": rng.randint(2, 64),
                "bits": rng.randint(1, 20), "signed": False, "bits2": rng.randint(1, 8),
                "signed2": True}
    if op == "batch":
        return {"op": op, "count": _size(rng, 16, 4096), "lo": 32, "hi": 2048,
                "bits": rng.randint(4, 24)}
    if op == "vlb":
        return {"op": op, "rows": _size(rng, 256, 8192), "cols": _size(rng, 256, 16384),
                "beta": rng.choice((1.0, 8.0, 32.0)), "signed": rng.random() < 0.3}
    return {"op": op, "rows": _size(rng, 256, 16384), "cols": _size(rng, 256, 8192),
            "dtype": rng.choice(("float32", "float32", "float64")),
            "sig_bits": rng.randint(6, 20), "x_sig_bits": rng.randint(8, 20)}


# ---- inputs ----------------------------------------------------------------

_DT = {"int32": torch.int32, "int64": torch.int64, "float32": torch.float32,
       "float64": torch.float64}


def _gen(seed, salt=0):
    return torch.Generator(device="cuda").manual_seed(1303 + 1000003 * int(seed) + salt)


def _range(bits, signed):
    if signed:
        return -(1 << (bits - 1)), 1 << (bits - 1)
    return 0, 1 << min(bits, 63)


def _dense(rows, cols, bits, signed, dtype, g):
    lo, hi = _range(bits, signed)
    return torch.randint(lo, hi, (rows, cols), generator=g, dtype=dtype, device="cuda")


def _packed(rows, cols, bits, signed, seed, salt):
    """A compressed matrix of uniform values of the given width."""
    if bits > 32:  # past the packed generator's span: through dense memory
        return ccm.compress(_dense(rows, cols, bits, signed, torch.int64, _gen(seed, salt)))
    lo, hi = _range(bits, signed)
    return ccm.generate(rows, cols, lo, hi, seed=1303027000 + 64 * int(seed) + salt, stream_id=salt)


def _vector(n, bits, dtype, g):
    return torch.randint(-(1 << (bits - 1)), 1 << (bits - 1), (n,), generator=g, dtype=dtype,
                         device="cuda")


def _floats(c, seed):
    """A matrix of values over six decimal orders of magnitude, its largest
    magnitude the same for every seed, and x in [-1, 1)."""
    g, dt = _gen(seed), _DT[c["dtype"]]
    v = torch.rand((c["rows"], c["cols"]), generator=g, dtype=dt, device="cuda")
    v.mul_(2).sub_(1).mul_(0.999)
    e = torch.randint(-20, 1, v.shape, generator=g, dtype=torch.int32, device="cuda")
    v = torch.ldexp(v, e).to(dt)
    v[0, 0], v[-1, -1] = 0.999, -0.999
    x = torch.rand(c["cols"], generator=g, dtype=dt, device="cuda").mul_(2).sub_(1)
    return v, x


def _beta_values(c, seed):
    """int64 values whose bit-lengths are floor(64 u) + 1 with u ~ Beta(1, beta)
    (at most 62), uniform among the values of their length.  Lengths and signs
    are one draw, rolled by the seed, so every seed packs to as many bits."""
    g, fixed, shape = _gen(seed), _gen(0, 9), (c["rows"], c["cols"])
    by = torch.randint(0, 1 << 20, (2,), generator=torch.Generator().manual_seed(seed)).tolist()
    u = torch.rand(shape, generator=fixed, dtype=torch.float32, device="cuda")
    n = (64 * (1 - u.pow(1.0 / c["beta"]))).to(torch.int64).clamp_(0, 61)  # length - 1
    n = n.roll(by, (0, 1))
    del u
    r = torch.randint(0, 1 << 62, shape, generator=g, dtype=torch.int64, device="cuda")
    top = torch.bitwise_left_shift(torch.ones((), dtype=torch.int64, device="cuda"), n)
    del n
    r.bitwise_and_(top - 1).bitwise_or_(top)
    if c["signed"]:
        # odd magnitudes: -2^(L-1) alone would take a bit less than its length
        s = torch.randint(0, 2, shape, generator=fixed, dtype=torch.int64, device="cuda") * 2 - 1
        r.bitwise_or_(1).mul_(s.roll(by, (0, 1)))
    return r


def prepare(case, seed):
    c, op = case, case["op"]
    if op == "plain":
        g = _gen(seed)
        a = _dense(c["rows"], c["cols"], c["bits"], False, _DT[c["dtype"]], g)
        b = _dense(c["rows"], c["cols"], c["bits"], False, _DT[c["dtype"]], g)
        x = torch.randint(0, 1000, (c["cols"],), generator=g, dtype=torch.int64, device="cuda")
        return {"op": op, "a": a, "b": ccm.compress(b), "x": x,
                "at": (c["rows"] // 2, c["cols"] // 3)}
    if op == "sweep":
        ms = [_packed(c["rows"], c["cols"], k, False, seed, 1 + i)
              for i, k in enumerate(SWEEP_WIDTHS)]
        return {"op": op, "ms": ms, "x": _vector(c["cols"], c["xbits"], torch.int32, _gen(seed)),
                "ys": [torch.empty(c["rows"], dtype=torch.int64, device="cuda") for _ in ms]}
    if op in ("matvec", "matvec_t"):
        m = _packed(c["rows"], c["cols"], c["bits"], c["signed"], seed, 1)
        n = c["cols"] if op == "matvec" else c["rows"]
        return {"op": op, "m": m, "x": _vector(n, c["xbits"], _DT[c["xdtype"]], _gen(seed))}
    if op == "compress":
        return {"op": op, "order": c["order"],
                "a": _dense(c["rows"], c["cols"], c["bits"], c["signed"], _DT[c["dtype"]],
                            _gen(seed))}
    if op == "add":
        return {"op": op, "a": _packed(c["rows"], c["cols"], c["bits"], c["signed"], seed, 1),
                "b": _packed(c["rows"], c["cols"], c["bits2"], c["signed"], seed, 2)}
    if op in ("scale", "decompress"):
        return {"op": op, "by": c["by"],
                "a": _packed(c["rows"], c["cols"], c["bits"], c["signed"], seed, 1)}
    if op == "matmul":
        return {"op": op, "a": _packed(c["m"], c["k"], c["bits"], c["signed"], seed, 1),
                "b": _packed(c["k"], c["n"], c["bits2"], c["signed2"], seed, 2)}
    if op == "batch":
        g = torch.Generator().manual_seed(1303 + c["count"])  # the same shapes for every seed
        dims = torch.randint(c["lo"], c["hi"] + 1, (c["count"], 2), generator=g).tolist()
        bits = torch.randint(1, c["bits"] + 1, (c["count"],), generator=g).tolist()
        mats = [_packed(r, k, b, False, seed, 16 + t)
                for t, ((r, k), b) in enumerate(zip(dims, bits))]
        x = _vector(sum(k for _, k in dims), 16, torch.int32, _gen(seed))
        y = torch.empty(sum(r for r, _ in dims), dtype=torch.int64, device="cuda")
        batch = ccm.Batch(mats)
        batch.set_io(x.split([k for _, k in dims]), y.split([r for r, _ in dims]))
        return {"op": op, "batch": batch, "y": y, "x": x}
    if op == "vlb":
        return {"op": op, "a": _beta_values(c, seed),
                "x": _vector(c["cols"], 16, torch.int32, _gen(seed, 1))}
    if op == "float":
        v, x = _floats(c, seed)
        return {"op": op, "v": v, "x": x, "sig": c["sig_bits"], "xsig": c["x_sig_bits"]}
    raise ValueError(op)


# ---- one pass ----------------------------------------------------------------

def _whole(m):
    """A compressed result: its header fields and canonical payload."""
    return {"vmin": m.vmin, "vmax": m.vmax, "bits": m.bits, "payload": m.payload[: 8 * m.words]}


def run(s):
    op = s["op"]
    if op == "plain":
        m = ccm.compress(s["a"])
        v = ccm.get(m, *s["at"])
        y = ccm.matvec(m, s["x"])
        c = ccm.add(m, s["b"])
        t = ccm.scale(c, 7)
        return {"m": _whole(m), "v": v, "y": y, "c": _whole(c), "t": _whole(t),
                "d": ccm.decompress(t)}
    if op == "sweep":
        return [ccm.matvec(m, s["x"], y=y) for m, y in zip(s["ms"], s["ys"])]
    if op == "matvec":
        return ccm.matvec(s["m"], s["x"])
    if op == "matvec_t":
        return ccm.matvec_t(s["m"], s["x"])
    if op == "compress":
        return _whole(ccm.compress(s["a"], order=s["order"]))
    if op == "add":
        return _whole(ccm.add(s["a"], s["b"]))
    if op == "scale":
        return _whole(ccm.scale(s["a"], s["by"]))
    if op == "decompress":
        return ccm.decompress(s["a"])
    if op == "matmul":
        return _whole(ccm.matmul(s["a"], s["b"]))
    if op == "batch":
        s["batch"].run()
        return s["y"]
    if op == "vlb":
        m = ccm.vlb_compress(s["a"])
        y = ccm.vlb_matvec(m, s["x"])
        return {"payload": m.payload[: 8 * m.words], "nbits": m.nbits, "k": m.k, "y": y}
    m = ccm.compress_float(s["v"], sig_bits=s["sig"])
    y = ccm.matvec_float(m, s["x"], x_sig_bits=s["xsig"])
    return {"payload": m.payload[: 8 * m.words], "frac_bits": m.frac_bits, "y": y,
            "d": ccm.decompress_float(m, dtype=s["v"].dtype)}


# ---- exact floating results ----------------------------------------------------

def exact(case, seed):
    """The floats a pass returns, from plain torch in 64 bits (None for the
    whole numbers, which have no rounding)."""
    if case["op"] != "float":
        return None
    v, x = _floats(case, seed)

    def quantized(t, sig):
        t = t.double()
        f = sig - math.frexp(float(t.abs().max()))[1]
        return torch.round(t * 2.0 ** f), f

    q, f = quantized(v, case["sig_bits"])
    xq, g = quantized(x, case["x_sig_bits"])
    y = torch.mv(q, xq) * 2.0 ** -(f + g)
    return {"payload": None, "frac_bits": None, "y": y, "d": q * 2.0 ** -f}


# ---- bytes and operations ---------------------------------------------------------

def _pk(n, bits):
    return n * bits / 8


def work(case):
    c, op = case, case["op"]
    if op == "batch":
        g = torch.Generator().manual_seed(1303 + c["count"])
        dims = torch.randint(c["lo"], c["hi"] + 1, (c["count"], 2), generator=g).tolist()
        bits = torch.randint(1, c["bits"] + 1, (c["count"],), generator=g).tolist()
        n = sum(r * k for r, k in dims)
        return {"bytes": sum(_pk(r * k, b) + 4 * k + 8 * r for (r, k), b in zip(dims, bits)),
                "flops": 2 * n}
    if op == "matmul":
        m, k, n = c["m"], c["k"], c["n"]
        out = min(63, c["bits"] + c["bits2"] + max(0, (k - 1).bit_length() - 1))
        return {"bytes": _pk(m * k, c["bits"]) + _pk(k * n, c["bits2"]) + _pk(m * n, out),
                "flops": 2 * m * n * k}
    r, k = c["rows"], c["cols"]
    n = r * k
    if op == "plain":
        d, b = (8 if c["dtype"] == "int64" else 4), c["bits"]
        return {"bytes": n * d + _pk(n, b) * 6 + _pk(n, b + 1) * 2 + _pk(n, b + 4) * 2
                + 8 * (r + k) + 8 * n, "flops": 4 * n}
    if op == "sweep":
        return {"bytes": sum(_pk(n, b) for b in SWEEP_WIDTHS) + 6 * (4 * k + 8 * r),
                "flops": 12 * n}
    if op in ("matvec", "matvec_t"):
        nx, ny = (k, r) if op == "matvec" else (r, k)
        return {"bytes": _pk(n, c["bits"]) + nx * (4 if c["xdtype"] == "int32" else 8) + 8 * ny,
                "flops": 2 * n}
    if op == "compress":
        return {"bytes": n * (8 if c["dtype"] == "int64" else 4) + _pk(n, c["bits"]), "flops": 0}
    if op == "add":
        out = max(c["bits"], c["bits2"]) + 1
        return {"bytes": _pk(n, c["bits"]) + _pk(n, c["bits2"]) + _pk(n, out), "flops": n}
    if op == "scale":
        out = c["bits"] + c["by"].bit_length()
        return {"bytes": _pk(n, c["bits"]) + _pk(n, out), "flops": n}
    if op == "decompress":
        return {"bytes": _pk(n, c["bits"]) + 8 * n, "flops": 0}
    if op == "vlb":
        # mean length of floor(64 u) + 1, u ~ Beta(1, beta); 6 or 7 bits of length each
        pair = 6 + 0.5 + 64.0 / (1 + c["beta"])
        return {"bytes": 8 * n + 2 * _pk(n, pair) + 4 * k + 8 * r, "flops": 2 * n}
    f = 4 if c["dtype"] == "float32" else 8
    q = c["sig_bits"] + 1
    # floats in, packed out; packed in, y out; packed in, floats out
    return {"bytes": 2 * f * n + 3 * _pk(n, q) + f * k + 8 * r, "flops": 2 * n}
