"""PSD kernels at the ends of the range of doubles: their results are those of
the same data scaled by a power of two, and an entry far below the others
changes no step length.

Tolerance: that of the kernel tests, 1e-12 relative.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import cones as C  # noqa: E402
from paper_2412_19027_amd import hipcone as HC  # noqa: E402
from tests.test_oracle_cones import spd  # noqa: E402
from tests.test_gpu_psd_sides import T, relerr  # noqa: E402


@pytest.mark.parametrize("k", [3, 16, 17, 32])
@pytest.mark.parametrize("tiny", [1e-140, 5e-155, 3e-162, 5e-324])
def test_step_with_a_tiny_column(k, tiny):
    """Column 0 below the diagonal at `tiny`, an eigenvalue -5 in the rest."""
    D = np.diag(np.r_[1.0, -5.0, 2.0 * np.ones(k - 2)])
    D[0, 1:] = D[1:, 0] = tiny
    for i in range(2, k):
        D[1, i] = D[i, 1] = 0.25
    dx, eye = C.svec(D[None]), C.svec(np.eye(k)[None])
    got = HC.test_cone_step(HC.PSD, k, T(eye), T(eye), T(dx), T(0 * dx), 1.0)
    assert relerr(got, -1.0 / np.linalg.eigvalsh(D[1:, 1:]).min()[None]) < 1e-12


@pytest.mark.parametrize("k", [2, 16, 17, 32])
@pytest.mark.parametrize("e", [-560, 560])
def test_step_of_a_scaled_direction(k, e):
    rng = np.random.default_rng(k)
    s, dx = C.svec(spd(3, k, rng)), rng.standard_normal((3, k * (k + 1) // 2))
    got = HC.test_cone_step(HC.PSD, k, T(s), T(s), T(np.ldexp(dx, e)), T(0 * dx), np.inf)
    assert relerr(got * 2.0 ** (e // 2) * 2.0 ** (e // 2), C.psd_step(s, dx, k)) < 1e-12


@pytest.mark.parametrize("k", [2, 15, 16, 17, 32])
@pytest.mark.parametrize("e", [-300, 300])
def test_scaling_of_scaled_points(k, e):
    rng = np.random.default_rng(k)
    s, z = C.svec(spd(3, k, rng)), C.svec(spd(3, k, rng))
    H, lam, _ = HC.test_cone_scale(HC.PSD, k, T(np.ldexp(s, e)), T(np.ldexp(z, e)), 1.0)
    ref = C.psd_scale(s, z, k)
    assert relerr(H, ref["H"]) < 1e-12
    lam = np.ldexp(np.sort(lam.cpu().numpy()[:, :k], 1), -e)
    assert np.abs(lam - np.sort(ref["lam"], 1)).max() < 1e-12 * ref["lam"].max()
