"""Dense generalized eigensolver either side of its kernel choices (one
workgroup's tail, register widths of the tridiagonalisation step, reflector
blocks of the back-transform) and on spectra whose eigenvectors have to be
told apart: pairs and groups closer than the cluster gap, down to rounding.

Bounds: backward error of a Householder / inverse-iteration solve, a small
multiple of n eps |T| for eigenvalues and of n eps for orthogonality; 1e-11 as
in the other dense tests covers n = 2,433 twenty times over."""
import numpy as np
import pytest

from paper_2609_13115_amd import xls

pytestmark = pytest.mark.gpu


def check(n, lam_true, cond, seed):
    rng = np.random.default_rng(seed)
    q, _ = np.linalg.qr(rng.standard_normal((n, n)))
    a = (q * lam_true) @ q.T
    b = np.eye(n) + cond * rng.standard_normal((n, n)) / np.sqrt(n)
    H, M = b.T @ (0.5 * (a + a.T)) @ b, b.T @ b
    H, M = 0.5 * (H + H.T), 0.5 * (M + M.T)
    lam, Y = xls.xls_dense_geneig(H, M)
    scale = max(1.0, np.max(np.abs(lam_true)))
    assert np.all(np.diff(lam) >= 0)
    assert np.max(np.abs(lam - np.sort(lam_true))) <= 1e-11 * scale
    assert np.max(np.abs(Y.T @ M @ Y - np.eye(n))) <= 1e-11
    assert np.max(np.abs(H @ Y - (M @ Y) * lam)) <= 1e-11 * scale


@pytest.mark.parametrize("n", [1, 2, 3, 16, 31, 32, 33, 63, 64, 65, 127, 128, 129, 191, 192, 193, 229, 512, 513, 640,
                               641, 900, 901, 1024, 1025, 1152, 1153, 1216, 1217, 1921, 2433])
def test_sizes(n):
    print(f"[case] dense edges n={n}", flush=True)
    check(n, np.sort(np.random.default_rng(n).uniform(-0.4, 0.7, n)), 0.2, n)


# both sides of the widths at which the inverse of the Cholesky factor changes
# its columns per wavefront or leaves the registers
@pytest.mark.parametrize("n", [256, 257, 768, 769, 1280, 1281])
def test_inverse_widths(n):
    test_sizes(n)


@pytest.mark.parametrize("gap", [0.0, 1e-15, 1e-13, 1e-10, 1e-7, 1e-5])
def test_groups_of_close_eigenvalues(gap):
    print(f"[case] dense edges groups gap={gap}", flush=True)
    n = 210
    base = np.repeat(np.linspace(-0.3, 0.6, 10), 21)
    check(n, base + gap * np.tile(np.arange(21), 10), 0.2, 5)


def test_one_wide_cluster():
    """Every gap below the cluster threshold: all vectors in one group."""
    print("[case] dense edges one cluster", flush=True)
    check(300, np.linspace(0.5, 0.6, 300), 0.2, 6)


# Spectra that fall to 1e-14 of the largest state: hundreds of eigenvalues equal
# to rounding, whose vectors come out of inverse iteration nearly parallel.
# Vectors of one cluster are orthogonal to rounding, those of two clusters to eps
# over the gap between them, 1e-3 |T| at least; twice that here.
@pytest.mark.parametrize("n", [300, 480])
def test_states_equal_to_rounding_are_orthogonal(n):
    worst = 0.0
    for seed in range(8):
        print(f"[case] dense edges geometric n={n} seed={seed}", flush=True)
        rng = np.random.default_rng(seed)

        def full(lam):
            q, _ = np.linalg.qr(rng.standard_normal((n, n)))
            a = (q * lam) @ q.T
            return 0.5 * (a + a.T)

        H, M = full(10.0 ** -np.linspace(0, 14, n)), full(np.linspace(0.5, 2, n))
        lam, Y = xls.xls_dense_geneig(H, M)
        worst = max(worst, np.max(np.abs(Y.T @ M @ Y - np.eye(n))))
        assert np.linalg.norm(H @ Y - (M @ Y) * lam) <= 1e-12 * np.linalg.norm(Y)
    assert worst <= 2 * 2.3e-16 / 1e-3
