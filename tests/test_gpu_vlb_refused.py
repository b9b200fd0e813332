"""A Method 2 plan refused for the length of its rows (group offsets of 32 bits) has
ended on the device when it returns: its index can be used on another stream."""
import ctypes

import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def test_refused_plan_has_ended():
    import paper_1303_0270_amd as c
    cols = 1 << 26  # 6 + 62 bits a pair
    dense = torch.full((1, cols), 1 << 61, dtype=torch.int64, device="cuda")
    nidx = int(c.lib.ccm_vlb_index_bytes(1, cols))
    index = torch.empty(nidx, dtype=torch.uint8, device="cuda")
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    for rep in range(8):
        d = c._lib.VlbDesc()
        rc = c.lib.ccm_vlb_compress_plan(
            ctypes.c_void_p(dense.data_ptr()), c._lib.I64, 1, cols,
            ctypes.c_void_p(index.data_ptr()), ctypes.byref(d), ctypes.c_void_p(side.cuda_stream))
        assert rc == c._lib.E_UNSUPPORTED
        index.fill_(0xA5)
        torch.cuda.synchronize()
        assert bool((index == 0xA5).all()), rep
    del dense, index
    torch.cuda.empty_cache()
    a = np.arange(-50, 250).reshape(3, 100)
    m, want = c.vlb_compress(torch.from_numpy(a).cuda()), oracle.vlb_compress(a)
    assert m.nbits == want.nbits
    assert np.array_equal(m.payload_words().numpy().view(np.uint64), want.payload)
