"""Blocks to and from binary16 buffers, vector and general paths: bit-exact
against NumPy's conversion, nothing written past the buffer."""
import numpy as np
import pytest
import torch

from paper_2609_13115_amd import xls
from test_gpu_tiles import box

pytestmark = pytest.mark.gpu


# point counts: a multiple of eight with a short last workgroup, less than one
# workgroup, an odd count, and a multiple of eight in a buffer that is not
# 16-byte aligned
@pytest.mark.parametrize("shape,shift", [((12, 10, 19), 0), ((4, 6, 5), 0), ((7, 9, 11), 0), ((17, 21, 23), 0),
                                         ((12, 10, 19), 3)])
@pytest.mark.parametrize("prec", [xls.XLS_PREC_FP64, xls.XLS_PREC_FP32])
def test_half_buffers(shape, shift, prec):
    print(f"[case] half buffers {shape} shift={shift} prec={prec}", flush=True)
    sd = box(shape, 3, False)
    X = np.random.default_rng(2).standard_normal((sd.nd, 3)) * 10.0 ** np.random.default_rng(3).integers(-9, 5, (sd.nd, 3))
    X[0, 0], X[-1, -1], X[1, 1] = 0.0, 7e4, -65519.0
    X = X.astype(np.float32).astype(np.float64)
    n = sd.nd * 3
    store = torch.full((n + 16,), 3.0, dtype=torch.float16, device="cuda")
    buf = store[shift:shift + n]
    with xls.Subdomain(sd, filter_prec=prec) as s:
        s.xls_subdomain_set_block(X)
        s.xls_subdomain_store_half(buf)
        with np.errstate(over="ignore"):
            want = X.astype(np.float32).astype(np.float16)
        got = store.cpu().numpy()
        assert np.array_equal(got[shift:shift + n].reshape(3, sd.nd).T.view(np.uint16), want.view(np.uint16))
        assert np.all(got[:shift] == 3.0) and np.all(got[shift + n:] == 3.0)
        s.xls_subdomain_load_half(buf)
        assert np.array_equal(s.xls_subdomain_get_block(), want.astype(np.float64))


# blocks past the size from which a lane takes several values: whole vectors, odd
# point counts, an unaligned buffer
@pytest.mark.parametrize("shape,ns,shift", [((32, 32, 40), 30, 0), ((31, 33, 35), 33, 0), ((32, 32, 40), 30, 1)])
@pytest.mark.parametrize("prec", [xls.XLS_PREC_FP64, xls.XLS_PREC_FP32])
def test_half_buffers_of_large_blocks(shape, ns, shift, prec):
    print(f"[case] large half buffers {shape} ns={ns} shift={shift} prec={prec}", flush=True)
    sd = box(shape, ns, False)
    X = np.random.default_rng(5).standard_normal((sd.nd, ns)).astype(np.float32).astype(np.float64)
    n = sd.nd * ns
    store = torch.full((n + 16,), 3.0, dtype=torch.float16, device="cuda")
    buf = store[shift:shift + n]
    want = X.astype(np.float32).astype(np.float16)
    with xls.Subdomain(sd, filter_prec=prec) as s:
        s.xls_subdomain_set_block(X)
        s.xls_subdomain_store_half(buf)
        got = store.cpu().numpy()
        assert np.array_equal(got[shift:shift + n].reshape(ns, sd.nd).T.view(np.uint16), want.view(np.uint16))
        assert np.all(got[:shift] == 3.0) and np.all(got[shift + n:] == 3.0)
        s.xls_subdomain_load_half(buf)
        assert np.array_equal(s.xls_subdomain_get_block(), want.astype(np.float64))
