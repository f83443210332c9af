"""Poisson kernels at the edges of their tiles: grids narrower than the
Laplacian's halo, rows past one 64-point tile, a single multigrid level, and
coarsest levels on either side of the one-workgroup end of the V-cycle.
One V-cycle against the oracle's FP64 V-cycle (1e-5: FP32 arithmetic) and
solves against the oracle's solution (both stop at 1e-10 of the right-hand
side; the operator's condition number at these sizes is below 1e3)."""
import numpy as np
import pytest

from oracle import poisson
from paper_2609_13115_amd import xls

pytestmark = pytest.mark.gpu

CASES = [((6, 5, 4), False, 0),       # one level, below the halo
         ((5, 7, 3), True, 0),        # periodic wraps more than once
         ((1, 9, 2), False, 0),
         ((71, 9, 7), False, 0),      # two x tiles; 35 x 4 x 3 does not coarsen
         ((63, 15, 31), False, 0),
         ((130, 20, 8), True, 0),     # ragged last tile, one transfer
         ((63, 47, 31), False, 2),    # coarsest level above the one-workgroup end
         ((72, 40, 24), True, 2),
         ((64, 128, 8), True, 0)]     # 32 x 64 x 4 = 8,192 points: the end's largest level


@pytest.mark.parametrize("n,periodic,levels", CASES)
def test_vcycle_and_solve(n, periodic, levels):
    print(f"[case] poisson edges {n} periodic={periodic} levels={levels}", flush=True)
    h = 0.43
    f = np.random.default_rng(11).standard_normal(int(np.prod(n)))
    if periodic:
        f -= f.mean()
    H = poisson.hierarchy(n, h, periodic, levels or 8)
    z_ref = poisson.vcycle(H, f)
    ref = poisson.solve(f, n, h, periodic, tol=1e-10, max_levels=levels or 8)
    with xls.Poisson(n, h, 0 if periodic else 1, levels) as p:
        z = p.vcycle(f)
        phi, info = p.solve(f, tol=1e-10)
        again, _ = p.solve(f, tol=1e-10)
        zero, info0 = p.solve(np.zeros_like(f))
    assert info[2] == len(H.sizes)
    assert np.linalg.norm(z - z_ref) <= 1e-5 * np.linalg.norm(z_ref)
    assert info[1] <= 1e-10 and abs(info[0] - ref.iters) <= 2
    assert np.linalg.norm(phi - ref.phi) <= 1e-7 * np.linalg.norm(ref.phi)
    assert np.array_equal(phi, again)
    assert info0[0] == 0 and not zero.any()


def test_iteration_limit():
    """max_iter ends the loop with the iterate of that iteration."""
    print("[case] poisson iteration limit", flush=True)
    n, h = (31, 31, 15), 0.43
    f = np.random.default_rng(2).standard_normal(int(np.prod(n)))
    b = 4 * np.pi * f
    with xls.Poisson(n, h, 1) as p:
        for k in (1, 2, 5):
            phi, info = p.solve(f, tol=1e-14, max_iter=k)
            r = b - poisson.apply_A(phi, n, h, False)
            assert info[0] == k
            assert abs(np.linalg.norm(r) / np.linalg.norm(b) - info[1]) <= 1e-10
