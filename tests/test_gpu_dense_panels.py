"""The FP64 factorisation's panel steps and look-ahead at the edges of their
tiles and rules (through the C-ABI), against A itself.

Tolerance: Cholesky's backward error is at most (n + 1) u max(a_ii) per entry
(u = 2^-53, |L||L'| <= max a_ii row by row); the 64-column blocks solve with
explicit inverses of blocks whose condition is below 8 here, hence 8 (n + 1) u.
"""
import pytest
import torch

from paper_2412_19027_amd import hipcone as HC

pytestmark = pytest.mark.gpu


# one block, a step with and without rows below, an inner panel's last step
# and the update after it, partial last blocks, look-ahead panels of 256
# columns (above 4,096 rows) and of 768 (above 8,192)
@pytest.mark.parametrize("n", [63, 65, 128, 129, 191, 256, 257, 320, 385, 577, 1025, 4096, 4161, 4417, 8257])
def test_factor_backward_error(n):
    g = torch.Generator(device="cuda").manual_seed(n)
    G = torch.randn(n, n, dtype=torch.float64, device="cuda", generator=g)
    A = G @ G.t() / n
    A.diagonal().add_(0.5)
    B = torch.randn(n, 1, dtype=torch.float64, device="cuda", generator=g)
    X, L, hits = HC.test_dense_chol_solve(A, B.clone(), ld=(n + 63) // 64 * 64)
    L = torch.tril(L)
    tol = 8 * (n + 1) * 2.0 ** -53 * A.diagonal().max().item()
    assert hits == 0
    assert (L @ L.t() - A).abs().max().item() <= tol
    # the solve's residual: both triangular solves, each with that bound times |x|'s 1-norm
    assert (A @ X - B).abs().max().item() <= 3 * tol * X.abs().sum().item()


def test_pivot_guard_in_a_panel():
    """A zero pivot past the first block column is replaced and counted."""
    n = 200
    A = torch.eye(n, dtype=torch.float64, device="cuda")
    A[130, 130] = 0.0
    A[131, 131] = -1.0
    B = torch.ones(n, 1, dtype=torch.float64, device="cuda")
    _, L, hits = HC.test_dense_chol_solve(A, B, ld=256)
    assert hits == 2
    d = torch.tril(L).diagonal()
    assert abs(d[130].item() ** 2 - 1e-8) <= 1e-22 and abs(d[131].item() ** 2 - 1e-8) <= 1e-22


@pytest.mark.parametrize("n,nrhs,width", [(1, 1, 0), (127, 2, 0), (128, 1, 0), (129, 3, 0), (257, 2, 1), (640, 4, 64),
                                          (901, 2, 130), (2049, 1, 300)])
def test_triangular_solves(n, nrhs, width):
    """Both passes over 128-row blocks: partial last blocks, one to four
    right-hand sides (in pairs), dense (width 0) and with an envelope that
    leaves blocks uncoupled; two factorisations in a row on new data."""
    for seed in (1, 2):
        g = torch.Generator(device="cuda").manual_seed(10 * n + seed)
        G = torch.randn(n, n, dtype=torch.float64, device="cuda", generator=g)
        i = torch.arange(n, device="cuda")
        if width:
            G = torch.where((i[:, None] - i[None, :]).clamp(min=0) <= width // 2, torch.tril(G), 0.0)
        A = G @ G.t() / (width or n)
        A.diagonal().add_(0.5)
        last = None
        if width:   # rows a column reaches, non-decreasing
            last = torch.clamp(i + width // 2 * 2 + 1, max=n).cpu().numpy()
        B = torch.randn(n, nrhs, dtype=torch.float64, device="cuda", generator=g)
        X, _, hits = HC.test_dense_chol_solve(A, B.clone(), ld=(n + 63) // 64 * 64, last=last)
        tol = 24 * (n + 1) * 2.0 ** -53 * A.diagonal().max().item()
        assert hits == 0
        assert ((A @ X - B).abs().amax(0) <= tol * X.abs().sum(0)).all()
