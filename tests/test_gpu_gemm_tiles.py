"""The large-tile products against NumPy, at the edges of their tiles.

Row tiles of 64 and 128, column tiles of 96 and 128, a k slab that ends short
(odd orders and odd point counts) and orders just past a tile."""
import numpy as np
import pytest

from paper_2609_13115_amd import xls
from test_gpu_tiles import box

pytestmark = pytest.mark.gpu


def rel_err(a, b):
    return float(np.max(np.abs(a - b)) / np.max(np.abs(b)))


# 8211 points: 64-row tiles; 33759 points with 190 or 250 columns: 128-row
# tiles.  The sums have K terms of either sign, so their rounding is about
# sqrt(K) eps of the largest entry and K eps in the worst case; an FP32 block
# stores the rotated block in FP32.
@pytest.mark.parametrize("shape,ns", [((17, 21, 23), 64), ((17, 21, 23), 97), ((17, 21, 23), 129),
                                      ((33, 33, 31), 190), ((33, 33, 31), 250)])
@pytest.mark.parametrize("prec,gprec", [(xls.XLS_PREC_FP64, xls.XLS_PREC_FP64), (xls.XLS_PREC_FP32, xls.XLS_PREC_FP64),
                                        (xls.XLS_PREC_FP32, xls.XLS_PREC_FP32)])
def test_large_tile_products(shape, ns, prec, gprec):
    print(f"[case] large tile products {shape} ns={ns} prec={prec} gemm={gprec}", flush=True)
    sd = box(shape, ns, False)
    rng = np.random.default_rng(11)
    X = rng.standard_normal((sd.nd, ns))
    if prec == xls.XLS_PREC_FP32:
        X = X.astype(np.float32).astype(np.float64)
    Q = rng.standard_normal((ns, ns)) / np.sqrt(ns)
    eps_in = 2.0 ** -24 if gprec == xls.XLS_PREC_FP32 else 2.0 ** -53
    eps_out = 2.0 ** -24 if prec == xls.XLS_PREC_FP32 else 2.0 ** -53
    with xls.Subdomain(sd, filter_prec=prec) as s:
        s.xls_subdomain_set_block(X)
        M, _ = s.xls_subdomain_project(gprec)
        s.xls_subdomain_set_block(X)
        s.xls_subdomain_rotate(Q, gprec)
        out = s.xls_subdomain_get_block()
    assert rel_err(M, X.T @ X) <= 16 * np.sqrt(sd.nd) * eps_in
    assert rel_err(out, X @ Q) <= 16 * np.sqrt(ns) * eps_in + 4 * eps_out


# Split-BF16 products take the edge that issues the less area, whatever leaves
# the compute units less: 128 for orders that fill a tile or two of it, 96 for
# those that it pads less by a tenth.  H_s is averaged with its transpose inside
# diagonal tiles only, so its bits name the edge (an order inside one tile of either
# is averaged whole).
@pytest.mark.parametrize("ns,edge", [(100, 2), (128, 2), (200, 2), (90, 3), (140, 3)])
def test_split_bf16_projection_edge_by_area(ns, edge):
    print(f"[case] split-BF16 edge ns={ns}", flush=True)
    sd = box((33, 32, 34), ns, False)
    X = np.random.default_rng(9).standard_normal((sd.nd, ns))
    got = []
    for plan in (0, edge, 5 - edge):
        with xls.Subdomain(sd, filter_prec=xls.XLS_PREC_FP32) as s:
            s.xls_subdomain_set_block(X)
            s.xls_subdomain_tune_gemm(0, plan, 0)
            got.append(s.xls_subdomain_project(xls.XLS_PREC_BF16X3))
    assert np.array_equal(got[0][1], got[1][1]) and np.array_equal(got[0][0], got[1][0])
    assert ns <= 96 or not np.array_equal(got[0][1], got[2][1])
