"""The Schur column gather where a column just exceeds one LDS chunk (two equal
ones, the last a row short) and where it takes three: the problems and the
tolerance of test_gpu_schur_groups.
"""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import ipm  # noqa: E402
from paper_2412_19027_amd import hipcone as HC  # noqa: E402
from tests.test_gpu_schur_groups import make  # noqa: E402


@pytest.mark.parametrize("n", [5120, 5121, 10243])
def test_schur_of_groups(n):
    prob = make(n, [(4, 30, 8), (10, 3, 6)], 300, 64)
    o = ipm.Solver(prob)
    g = HC.Solver(prob, leaf_blocks=0)
    perm = g.iterate()[5]
    mu = o.mu()
    kkt = o._kkt([(grp.rows, sc["Hb"]) for grp, sc in zip(o.groups, o.scale(mu, False))])
    g.set_iterate(o.x, o.s[perm], o.z[perm], o.tau, o.kappa)
    Sg, _, _ = g.test_schur(mu, factor=False)
    g.close()
    So = (kkt.P + kkt.delta * sp.identity(prob.n) + kkt.A.T @ kkt.Mbd @ kkt.A).tocoo()
    top = np.abs(So.data).max()
    Sg[So.row, So.col] -= So.data   # entry by entry (no duplicates in So), the rest compared with zero
    assert np.abs(Sg).max() <= (1e-10 + 5e-13 / mu) * top, n
