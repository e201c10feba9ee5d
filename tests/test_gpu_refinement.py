"""The batched refinement's branches against the oracle at the initial point.

Each case takes one way through the row launches: P with a long row (its own
product), P with more entries per row than A' (likewise), a long row of A' (one
workgroup, more entries than its lanes), dense constraint rows (added after the
sparse part), and more lane-per-cone segments than one launch holds together
with PSD and large second-order cones (rows finished by the common launch).

Tolerances: the one of the KKT-layer tests for symmetric cones,
1e-10 + 5e-13 / mu, for the refined solve; for the whole solve both sides stop
at gap and residuals below 1e-8 relative, so the objectives agree to 1e-6.
"""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import ipm  # noqa: E402
from paper_2412_19027_amd import hipcone as HC  # noqa: E402
from paper_2412_19027_amd import workloads as W  # noqa: E402


def rows_of(c):
    return c[1] * (c[1] + 1) // 2 if c[0] == W.PSD else c[1]


def interior(rng, cones):
    """A strictly interior point of the product cone, and one of its dual (self-dual cones)."""
    out = []
    for kind, d, _ in cones:
        if kind == W.SOC:
            v = rng.standard_normal(d)
            v[0] = np.linalg.norm(v[1:]) + 1.0
        elif kind == W.PSD:
            B = rng.standard_normal((d, d))
            v = W.svec_encode((B @ B.T / d + np.eye(d))[None]).ravel()
        else:
            v = rng.uniform(0.5, 1.5, d)
        out.append(v)
    return np.concatenate(out)


def make(name):
    rng = np.random.default_rng(7)
    n = 600
    cones = [(W.NONNEG, 2500, 0.0)] + [(W.SOC, 3, 0.0)] * 100
    P = sp.identity(n) * 0.5
    if name == "segments":
        cones = [(W.NONNEG, 300, 0.0)] + [(W.SOC, d, 0.0) for d in range(2, 16) for _ in range(5)]
        cones += [(W.PSD, 4, 0.0)] * 3 + [(W.PSD, 14, 0.0)] * 2 + [(W.SOC, 40, 0.0)] * 2
    m = sum(rows_of(c) for c in cones)
    A = sp.random(m, n, density=4.0 / n, random_state=rng, data_rvs=rng.standard_normal).tolil()
    if name == "p_row":
        P = P.tolil()
        P[0, :] = 1e-3
        P[0, 0] = 1.0
    elif name == "p_wide":
        P = sp.diags([2.0] + [0.01] * 60, list(range(61)), shape=(n, n))
    elif name == "a_column":
        A[:, 3] = rng.standard_normal((m, 1))
    elif name == "dense_rows":
        A[:5, :] = rng.standard_normal((5, n)) / np.sqrt(n)
    A = A.tocsr()
    x0, s0, z0 = rng.standard_normal(n), interior(rng, cones), interior(rng, cones)
    Pu = sp.triu(P).tocsr()
    q = -(Pu + sp.triu(Pu, 1).T) @ x0 - A.T @ z0
    return W.Problem(n, m, Pu, q, A, A @ x0 + s0, cones, name=name)


@pytest.mark.parametrize("name", ["p_row", "p_wide", "a_column", "dense_rows", "segments"])
@pytest.mark.parametrize("leaf_blocks", [0, 1])
def test_refined_solve_and_whole_solve(name, leaf_blocks):
    prob = make(name)
    o = ipm.Solver(prob)
    g = HC.Solver(prob, leaf_blocks=leaf_blocks)
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
    assert info["status_name"] == "solved" and o.status == ipm.SOLVED, (name, info, o.status)
    assert abs(info["obj_primal"] - o.objective) <= 1e-6 * max(1.0, abs(o.objective)), (name, info, o.objective)
