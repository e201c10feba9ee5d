"""Long rows of a sparse product (a workgroup each): their sums at the edges of
the rounds in flight, more of them than workgroups, and what one costs.

Tolerances: a row of A'z is a sum of up to 8,193 terms in 1,024 lanes, so it
carries less than 64 roundings of its largest partial sum: 1e-13 of the sum of
magnitudes.  Cost: one column of 300,000 entries on top of 1,200,000 in short
rows is a quarter more work in one workgroup; the time of the KKT solves stays
below five times that without it (2.6 times; 9.3 with the row's loads one by one).
"""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2412_19027_amd import hipcone as HC  # noqa: E402
from paper_2412_19027_amd import workloads as W  # noqa: E402


def problem(A, seed=0):
    """min 1/4 |x|^2 + q'x, A x + s = b, s >= 0, with an interior point on both sides."""
    rng = np.random.default_rng(seed)
    m, n = A.shape
    x0, s0, z0 = rng.standard_normal(n), rng.uniform(0.5, 1.5, m), rng.uniform(0.5, 1.5, m)
    P = 0.5 * sp.identity(n, format="csr")
    return W.Problem(n, m, P, -(P @ x0) - A.T @ z0, A, A @ x0 + s0, [(W.NONNEG, m, 0.0)])


@pytest.mark.parametrize("n,m", [(3, 2049), (3, 2817), (3, 3840), (3, 3841), (3, 4096), (3, 5121), (3, 8193), (600, 2100)])
def test_sums(n, m):
    rng = np.random.default_rng(m)
    A = sp.csr_matrix(rng.standard_normal((m, n)))
    g = HC.Solver(problem(A), leaf_blocks=0, equilibrate=0)
    perm = g.iterate()[5]
    g.set_iterate(np.zeros(n), np.ones(m), np.ones(m), 1.0, 1.0)
    x, z, kx, _ = g.test_kkt_ops(1.0, rng.standard_normal(n), rng.standard_normal(m))
    g.close()
    zu = np.empty(m)
    zu[perm] = z
    mag = abs(A).T @ abs(zu) + abs(x)
    assert (np.abs(kx - (0.5 * x + A.T @ zu)) <= 1e-13 * mag + 1e-15).all(), np.abs(kx - (0.5 * x + A.T @ zu)).max()


def test_cost_of_one_long_row():
    rng = np.random.default_rng(1)
    m, n = 300000, 500
    base = sp.random(m, n, density=4.0 / n, random_state=rng, data_rvs=rng.standard_normal, format="csr")
    col = sp.csr_matrix((0.1 * rng.standard_normal(m), (np.arange(m), np.full(m, 3))), shape=(m, n))
    ms = []
    for A in (base, (base + col).tocsr()):
        g = HC.Solver(problem(A), max_iter=4)
        best = np.inf
        for _ in range(3):
            info = g.solve()
            best = min(best, info["solve_kkt_ms"] / info["ir_solves"])
        ms.append(best)
        g.close()
    assert ms[1] <= 5.0 * ms[0], ms
