"""The Schur complement's cone groups against the oracle, at the edges of their
kernels: T = M A of groups below and above the size that takes workgroups, with
more rows than are staged in LDS (a PSD cone of side 32 on few columns), and the
column gather with runs of less than, exactly and more than 64 values, more than
64 rows in a column and columns longer than one LDS chunk.

Tolerance: the one of the KKT-layer tests for symmetric cones, 1e-10 + 5e-13 / mu.
"""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import ipm  # noqa: E402
from paper_2412_19027_amd import hipcone as HC  # noqa: E402
from paper_2412_19027_amd import workloads as W  # noqa: E402


def make(n, blocks, nonneg, row):
    """PSD cones (side, count, entries per row) and nonneg rows of `row` entries."""
    rng = np.random.default_rng(n)
    cones = [(W.NONNEG, nonneg, 0.0)]
    nnz = [row] * nonneg
    s0 = [np.ones(nonneg)]
    for side, count, per in blocks:
        for _ in range(count):
            cones.append((W.PSD, side, 0.0))
            d = side * (side + 1) // 2
            nnz += [per] * d
            B = rng.standard_normal((side, side))
            s0.append(W.svec_encode((B @ B.T / side + np.eye(side))[None]).ravel())
    m = len(nnz)
    cols = np.concatenate([rng.choice(n, k, replace=False) for k in nnz])
    A = sp.csr_matrix((rng.standard_normal(len(cols)), cols, np.concatenate([[0], np.cumsum(nnz)])), shape=(m, n))
    s0 = np.concatenate(s0)
    x0 = rng.standard_normal(n)
    return W.Problem(n, m, sp.identity(n).tocsr(), -x0 - A.T @ s0, A, A @ x0 + s0, cones, name=f"groups_{n}")


CASES = {
    "staged_rows_exceeded": lambda: make(2500, [(32, 1, 2)], 30, 3),
    "two_chunks": lambda: make(5200, [(4, 30, 8), (10, 3, 6)], 300, 64),
    "long_columns": lambda: make(130, [(6, 20, 3), (10, 2, 1)], 400, 65),
    "narrow": lambda: make(64, [(3, 1, 2)], 70, 64),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_schur_of_groups(name):
    prob = CASES[name]()
    o = ipm.Solver(prob)
    g = HC.Solver(prob, leaf_blocks=0)
    perm = g.iterate()[5]
    mu = o.mu()
    kkt = o._kkt([(grp.rows, sc["Hb"]) for grp, sc in zip(o.groups, o.scale(mu, False))])
    g.set_iterate(o.x, o.s[perm], o.z[perm], o.tau, o.kappa)
    Sg, _, _ = g.test_schur(mu, factor=False)
    g.close()
    So = (kkt.P + kkt.delta * sp.identity(prob.n) + kkt.A.T @ kkt.Mbd @ kkt.A).toarray()
    assert np.abs(Sg - So).max() <= (1e-10 + 5e-13 / mu) * np.abs(So).max(), name
