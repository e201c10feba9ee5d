"""Device workspace of small problems (host-only set-up): what a problem does
not use it does not ask for, so that arenas and the allocation-free call's
static block keep their room.
"""
import ctypes as C
import os

import numpy as np
import pytest
import scipy.sparse as sp

from paper_2412_19027_amd import hipcone as HC
from paper_2412_19027_amd import workloads as W

pytestmark = pytest.mark.skipif(not os.path.exists(HC.LIB_PATH), reason="libhipcone.so not built")


def sizes(prob, precision):
    """Workspace and read-back staging bytes of a set-up handle."""
    h, _keep = HC._setup(prob, HC.default_settings(precision=precision))
    out = []
    for fn in (HC.lib().hc_workspace_bytes, HC.lib().hc_host_stage_bytes):
        b = C.c_size_t()
        assert fn(h, C.byref(b)) == 0
        out.append(b.value)
    HC.lib().hc_destroy(h)
    return out


@pytest.mark.parametrize("blocks,cols", [(1, 1), (10, 4)])
def test_all_columns_in_leaf_blocks(blocks, cols):
    """No dense tail: beside the staged partials (as large on the device) only
    the problem's data, vectors and leaf blocks, 64 KiB and a few hundred bytes
    per variable; the mixed mode has no FP32 factor to add."""
    rng = np.random.default_rng(0)
    A = sp.block_diag([rng.standard_normal((2 * cols, cols)) for _ in range(blocks)], format="csr")
    n, m = A.shape[1], A.shape[0]
    prob = W.Problem(n, m, sp.identity(n).tocsr(), np.zeros(n), A, np.ones(m), [(W.NONNEG, m, 0.0)])
    assert HC.analyze(prob)["n_ordered"] == 0
    work, stage = sizes(prob, "fp64")
    mixed, _ = sizes(prob, "mixed")
    assert work - stage <= (64 << 10) + 1024 * n, (work, stage)
    assert mixed - work <= 4096, (mixed, work)


@pytest.mark.parametrize("n", [8, 64, 200])
def test_mixed_mode_adds_its_fp32_factor(n):
    """The FP32 matrix, its 64 x 64 blocks' inverses and, twice, its 256 x 256
    blocks' inverses, with 8 KiB for vectors and alignment."""
    prob = W.tiny_lp(0, n, 2 * n + 5)
    pad = -(-n // 64) * 64
    work, _ = sizes(prob, "fp64")
    mixed, _ = sizes(prob, "mixed")
    assert mixed - work <= 4 * (pad * pad + pad * 64 + 2 * 256 * 256) + 8192, (mixed, work)
