"""Lanczos bounds where the recurrence ends early or runs its full length, and
projections of few columns against the same columns among many."""
import numpy as np
import pytest

from oracle import hamiltonian
from paper_2609_13115_amd import xls
from test_gpu_tiles import box

pytestmark = pytest.mark.gpu


# A start vector of `count` eigenvectors spans an invariant space of that size:
# the bounds are its smallest and largest eigenvalue, to the rounding of a few
# dozen products (beta there is rounding too).  More steps than points: k is
# cut to the points, the whole spectrum is found.
@pytest.mark.parametrize("shape,count,k", [((4, 3, 5), 1, 20), ((4, 3, 5), 2, 20), ((6, 5, 7), 5, 12), ((2, 3, 2), 12, 60),
                                           ((1, 1, 1), 1, 20)])
def test_bounds_of_an_invariant_space(shape, count, k):
    print(f"[case] lanczos invariant {shape} count={count} k={k}", flush=True)
    sd = box(shape, 1, False)
    H = hamiltonian.from_subdomain(sd).apply(np.eye(sd.nd))
    lam, U = np.linalg.eigh(0.5 * (H + H.T))
    pick = np.unique(np.linspace(0, sd.nd - 1, count).round().astype(int))
    sd.lanczos_v0 = U[:, pick].sum(axis=1)
    with xls.Subdomain(sd) as s:
        lo, up = s.xls_lanczos_bounds(k)
    tol = 1e-10 * np.abs(lam).max()
    assert abs(lo - lam[pick[0]]) <= tol
    assert abs(up - lam[pick[-1]]) <= tol


# one wavefront per (atom, column) up to 2048 of them, four columns a wavefront
# past that: the same sums in the same order
@pytest.mark.parametrize("prec", [xls.XLS_PREC_FP64, xls.XLS_PREC_FP32])
def test_few_columns_match_many(prec):
    print(f"[case] projection columns prec={prec}", flush=True)
    sd = box((24, 24, 24), 300, True)
    X = np.random.default_rng(4).standard_normal((sd.nd, 300))
    with xls.Subdomain(sd, filter_prec=prec) as s:
        s.xls_subdomain_set_block(X)
        s.xls_subdomain_filter(3, -3.0, 4.0, 45.0)
        many = s.xls_subdomain_get_block()
    for n in (1, 5, 256):
        few = box((24, 24, 24), n, True)
        with xls.Subdomain(few, filter_prec=prec) as s:
            s.xls_subdomain_set_block(X[:, :n])
            s.xls_subdomain_filter(3, -3.0, 4.0, 45.0)
            assert np.array_equal(s.xls_subdomain_get_block(), many[:, :n])


# The counter holds the products of the run: those of the recurrence up to its
# end, however many steps the host had launched by then, and per iteration the
# filter's, one for the projection and one for the residual.  A second call uses
# the kept bounds.
@pytest.mark.parametrize("count", [2, 5])
def test_an_early_end_counts_the_products_that_it_took(count):
    print(f"[case] lanczos products count={count}", flush=True)
    sd = box((6, 5, 7), 3, False)
    H = hamiltonian.from_subdomain(sd).apply(np.eye(sd.nd))
    lam, U = np.linalg.eigh(0.5 * (H + H.T))
    pick = np.unique(np.linspace(0, sd.nd - 1, count).round().astype(int))
    sd.lanczos_v0 = U[:, pick].sum(axis=1)
    with xls.Subdomain(sd) as s:
        s.xls_chefsi_step(6, 1, xls.XLS_BOUNDS_LANCZOS)
        first = s.xls_subdomain_counters()["h_applies"]
        s.xls_chefsi_step(6, 1, xls.XLS_BOUNDS_LANCZOS)
        assert s.xls_subdomain_counters()["h_applies"] == 3 * (6 + 2)
    assert first == count + 3 * (6 + 2)


# Handles of several threads at once, some with a start vector that ends early:
# each stops on its own end.
def test_threads_end_on_their_own_steps():
    import threading
    sd = box((6, 5, 7), 3, False)
    H = hamiltonian.from_subdomain(sd).apply(np.eye(sd.nd))
    lam, U = np.linalg.eigh(0.5 * (H + H.T))
    full = np.random.default_rng(12).standard_normal(sd.nd)
    vectors = [U[:, 0] + U[:, -1], full, U[:, 3] + U[:, 9] + U[:, -1], full]
    got = [[] for _ in vectors]

    def work(i):
        with xls.Subdomain(sd, lanczos_v0=vectors[i]) as s:
            for _ in range(20):
                got[i].append(s.xls_lanczos_bounds(20))

    print("[case] lanczos threads", flush=True)
    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(vectors))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert all(len(g) == 20 and len(set(g)) == 1 for g in got)
    assert got[1][0] == got[3][0]
    tol = 1e-10 * np.abs(lam).max()
    for i, (a, b) in ((0, (0, -1)), (2, (3, -1))):
        assert abs(got[i][0][0] - lam[a]) <= tol and abs(got[i][0][1] - lam[b]) <= tol
