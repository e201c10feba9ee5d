"""hc_test_kkt_ops runs the refinement's own step: counted as one of its solves
and equal, bit for bit, to the first step of hc_test_kkt_solve (ir_max = 0),
with one unrefined solve's residual as small as the oracle's and the product
equal to the oracle's, through every branch of the step's launches (those of
test_gpu_refinement: long rows, dense rows, P beside A' or by itself, more
segments than a launch holds) and with exponential, power and PSD cones.

Tolerances: the residual that of the KKT-layer tests (50 times the oracle's plus
1e-10 of the right-hand side).  The product: a row of K [x; z] carries the
rounding of its terms, so 1e-12 of the largest sum of |K_ij| |v_j|, plus, for H,
the two sides' independent scalings, 1e-10 + 5e-13 / mu of it (5e-12 with
exponential or power cones).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import ipm  # noqa: E402
from paper_2412_19027_amd import hipcone as HC  # noqa: E402
from paper_2412_19027_amd import workloads as W  # noqa: E402
from tests.test_gpu_refinement import make  # noqa: E402

CASES = {name: (lambda name=name: make(name)) for name in ("p_row", "p_wide", "a_column", "dense_rows", "segments")}
CASES["exp"] = lambda: W.logreg_exp(0, samples=400, features=30)
CASES["psd_pow"] = lambda: W.psd_pow(0, n=250, n_pow=120, n_psd=25, k=4)


@pytest.mark.parametrize("leaf_blocks", [0, 1])
@pytest.mark.parametrize("name", CASES)
def test_hook_runs_the_refinement_step(name, leaf_blocks):
    prob = CASES[name]()
    nonsym = any(c[0] in (W.EXP, W.POW) for c in prob.cones)
    o = ipm.Solver(prob)
    mu = o.mu()
    kkt = o._kkt([(grp.rows, sc["Hb"]) for grp, sc in zip(o.groups, o.scale(mu, False))])
    rng = np.random.default_rng(1)
    r1, r2 = rng.standard_normal(prob.n), rng.standard_normal(prob.m)
    g = HC.Solver(prob, leaf_blocks=leaf_blocks, ir_max=0)
    perm = g.iterate()[5]

    def to_user(v):
        out = np.empty_like(v)
        out[perm] = v
        return out

    g.set_iterate(o.x, o.s[perm], o.z[perm], o.tau, o.kappa)
    before = g.info()["ir_solves"]
    xr, zr, kx, kz = g.test_kkt_ops(mu, r1, r2[perm])
    assert g.info()["ir_solves"] == before + 1, "not the refinement's step"
    x0, z0, st = g.test_kkt_solve(mu, r1, r2[perm])
    g.close()
    assert st["solves"] == 1 and np.array_equal(x0, xr) and np.array_equal(z0, zr)
    zr, kz = to_user(zr), to_user(kz)
    xo, zo = kkt.solve_reg(r1, r2)
    kxo, kzo = kkt.matvec(xo, zo)
    res = max(np.abs(r1 - kx).max(), np.abs(r2 - kz).max())
    res_o = max(np.abs(r1 - kxo).max(), np.abs(r2 - kzo).max())
    assert res <= 50 * res_o + 1e-10 * max(np.abs(r1).max(), np.abs(r2).max()), (res, res_o)
    kxo, kzo = kkt.matvec(xr, zr)
    ax, az = abs(kkt.P) @ abs(xr) + abs(kkt.A).T @ abs(zr), abs(kkt.A) @ abs(xr)
    hz = np.abs(kkt.A @ xr - kzo).max() + np.abs(r2).max()
    assert np.abs(kx - kxo).max() <= 1e-12 * ax.max(), np.abs(kx - kxo).max()
    assert np.abs(kz - kzo).max() <= 1e-12 * az.max() + (1e-10 + (5e-12 if nonsym else 5e-13) / mu) * hz
