"""Leaf solves against the oracle at the edges of their kernels: leaves of one,
four (a lane each), five and 32 columns (a wave each, columns of L eight at a
time), coupled to none, few or 64 tail columns, mixed in one problem, and for
one right-hand side (a KKT solve) and two (the pairs of a whole solve).

Tolerances: those of the KKT-layer tests for symmetric cones, 1e-10 + 5e-13 / mu,
and 1e-6 for the objectives of whole solves that stop at 1e-8.
"""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import ipm  # noqa: E402
from paper_2412_19027_amd import hipcone as HC  # noqa: E402
from paper_2412_19027_amd import workloads as W  # noqa: E402


def make(leaves, nt):
    """leaves: (columns, coupled tail columns) each; a tail of nt columns that one row couples pairwise."""
    rng = np.random.default_rng(nt)
    n = nt + sum(l for l, _ in leaves)
    rows = []
    for t in range(nt):   # a dense tail: every tail column with 20 others
        rows.append({t: 1.0, **{int(q): 0.1 for q in rng.choice(nt, min(20, nt), replace=False)}})
    c = nt
    for l, cnt in leaves:
        cols = list(range(c, c + l))
        for i in range(l):   # a chain through the leaf
            rows.append({cols[i]: rng.standard_normal(), cols[max(i - 1, 0)]: rng.standard_normal()})
        for a in rng.choice(nt, cnt, replace=False):
            rows.append({int(a): rng.standard_normal(), cols[int(rng.integers(l))]: rng.standard_normal()})
        c += l
    m = len(rows)
    A = sp.lil_matrix((m, n))
    for r, row in enumerate(rows):
        for j, v in row.items():
            A[r, j] = v
    A = A.tocsr()
    x0, s0, z0 = rng.standard_normal(n), rng.uniform(0.5, 1.5, m), rng.uniform(0.5, 1.5, m)
    return W.Problem(n, m, sp.identity(n).tocsr(), -x0 - A.T @ z0, A, A @ x0 + s0, [(W.NONNEG, m, 0.0)], name="leaves")


CASES = {
    "one_column": ([(1, 3)] * 300 + [(1, 0)], 70),
    "edges": ([(4, 2)] * 9 + [(5, 1)] * 5 + [(32, 6), (31, 0), (9, 40)], 90),
    "coupled_to_64": ([(3, 60), (8, 64), (2, 1)], 130),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_leaf_solves(name):
    prob = make(*CASES[name])
    o = ipm.Solver(prob)
    g = HC.Solver(prob, leaf_blocks=1)
    assert g.info()["n_leaves"] > 0, name
    perm = g.iterate()[5]
    mu = o.mu()
    kkt = o._kkt([(grp.rows, sc["Hb"]) for grp, sc in zip(o.groups, o.scale(mu, False))])
    rng = np.random.default_rng(1)
    r1, r2 = rng.standard_normal(prob.n), rng.standard_normal(prob.m)
    xo, zo, _ = kkt.solve(r1, r2, 1e-12, 1e-12, 10)
    g.set_iterate(o.x, o.s[perm], o.z[perm], o.tau, o.kappa)
    xs, zi, _ = g.test_kkt_solve(mu, r1, r2[perm])
    zs = np.empty_like(zi)
    zs[perm] = zi
    tol = 1e-10 + 5e-13 / mu
    assert np.abs(xs - xo).max() <= tol * np.abs(xo).max(), name
    assert np.abs(zs - zo).max() <= tol * np.abs(zo).max(), name
    info = g.solve()
    g.close()
    o.solve()
    assert info["status_name"] == "solved" and o.status == ipm.SOLVED, (name, info)
    assert abs(info["obj_primal"] - o.objective) <= 1e-6 * max(1.0, abs(o.objective)), name
