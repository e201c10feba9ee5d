"""PSD cone kernels against the oracle at the edges of their two size classes
(one wave up to side 16, four above; odd sides pair one column with a padding
one), with the directions that take the step length's special ways: none, a
diagonal one (nothing to reflect), minus the point itself (all eigenvalues
equal) and a rank-one one (k - 1 eigenvalues zero).

Tolerances: those of the kernel tests, 1e-12 relative; where the eigenvalues
coincide the oracle's own Cholesky and eigenvalues carry k eps times the
condition number (below 1e3 here), which stays under it.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import cones as C  # noqa: E402
from oracle import ipm  # noqa: E402
from paper_2412_19027_amd import hipcone as HC  # noqa: E402
from tests.test_oracle_cones import spd  # noqa: E402


def T(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


def relerr(a, b):
    a = a.detach().cpu().numpy()
    return np.abs(a - b).max() / max(np.abs(b).max(), 1e-300)


@pytest.mark.parametrize("k", [1, 2, 15, 16, 17, 31, 32])
def test_psd_kernels(k):
    rng = np.random.default_rng(k)
    nc = 9
    s, z = C.svec(spd(nc, k, rng)), C.svec(spd(nc, k, rng))
    H, lam, _ = HC.test_cone_scale(HC.PSD, k, T(s), T(z), 1.0)
    ref = C.psd_scale(s, z, k)
    assert relerr(H, ref["H"]) < 1e-12
    assert np.abs(np.sort(lam.cpu().numpy()[:, :k], 1) - np.sort(ref["lam"], 1)).max() < 1e-12 * ref["lam"].max()
    dsa, dza = 0.3 * rng.standard_normal(s.shape), 0.3 * rng.standard_normal(s.shape)
    out = HC.test_cone_ds(HC.PSD, k, T(s), T(z), T(dsa), T(dza), 0.8, 0.05)
    assert relerr(out, ipm.ds_family(ipm.PSD, s, z, ref, dsa, dza, 0.05, k=k)) < 1e-12
    # step lengths
    v = rng.standard_normal((nc, k))
    zero = np.zeros_like(s)
    diag = C.svec(np.stack([np.diag(d) for d in rng.standard_normal((nc, k)) - 1.0]))
    eye = C.svec(np.stack([np.eye(k)] * nc))
    one = -C.svec(v[:, :, None] * v[:, None, :])
    for x, dx in [(s, 2 * rng.standard_normal(s.shape)), (s, zero), (eye, diag), (s, -2.0 * s), (eye, one), (s, one)]:
        got = HC.test_cone_step(HC.PSD, k, T(x), T(z), T(dx), T(zero), 1.0)
        assert relerr(got, np.minimum(1.0, C.psd_step(x, dx, k))) < 1e-12
    got = HC.test_cone_step(HC.PSD, k, T(s), T(z), T(zero), T(one), 1.0)
    assert relerr(got, np.minimum(1.0, C.psd_step(z, one, k))) < 1e-12
