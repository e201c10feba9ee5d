"""The time split of a solve (info.cone_ms, factor_ms, solve_kkt_ms): the
scalings run the same kernels in FP64 and in mixed precision, so their time per
iteration has to be alike (here: at least half; launches without their kernels'
time are some hundredth of it), whether or not the handle owns its read-back
staging, and the parts stay within the whole.
"""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2412_19027_amd import hipcone as HC  # noqa: E402
from paper_2412_19027_amd import workloads as W  # noqa: E402


@pytest.mark.parametrize("pinned_stage", [False, True])
def test_scaling_time_in_both_precisions(pinned_stage):
    prob = W.psd_mixed(0, n=300, sides=(32,), per_side=60)
    per_it = {}
    for precision in ("fp64", "mixed"):
        g = HC.Solver(prob, precision=precision, max_iter=5, pinned_stage=pinned_stage)
        for _ in range(2):   # the first one loads the kernels
            info = g.solve()
        g.close()
        assert info["iterations"] > 0
        per_it[precision] = info["cone_ms"] / info["iterations"]
        assert info["cone_ms"] + info["factor_ms"] + info["solve_kkt_ms"] <= 1.02 * info["solve_ms"], info
    assert per_it["mixed"] >= 0.5 * per_it["fp64"], per_it
