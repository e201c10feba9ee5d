"""Problems of one batch that share their matrices share a plan and its device
data: each has to come out bitwise as it does alone, also next to problems that
differ in one matrix value, in q, in the settings or in precision, with the
same handle given twice and with results the caller does not ask for."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2412_19027_amd import hipcone as HC  # noqa: E402
from paper_2412_19027_amd import workloads as W  # noqa: E402


def variant(p, seed=None, q=None, last=None):
    b, qv, A = p.b.copy(), p.q.copy(), p.A.copy()
    if seed is not None:
        b[:4] = np.random.default_rng(seed).standard_normal(4)
    if q is not None:
        qv += q
    if last is not None:   # the one value of A that differs
        A.data[len(A.data) // 2 + 1] *= last
    return W.Problem(p.n, p.m, p.P, qv, A, b, p.cones)


def solve(handles, sizes, ask=None):
    res = (HC.hc_result * len(handles))()
    outs = []
    for i, (n, m) in enumerate(sizes):
        v = [np.full(k, np.nan) for k in (n, m, m)]
        outs.append(v)
        if ask is None or ask[i]:
            res[i].x, res[i].s, res[i].z = (a.ctypes.data_as(C.POINTER(C.c_double)) for a in v)
    arr = (C.c_void_p * len(handles))(*[h.value for h in handles])
    st = torch.cuda.current_stream().cuda_stream
    assert HC.lib().hc_solve_batch(arr, len(handles), st, 0, res) == 0
    return res, outs


@pytest.mark.parametrize("stages", [10, 33])
def test_shared_plans_are_bitwise_the_same(stages):
    base = W.mpc_socp(0, 1, stages, 4, 2)
    other = W.mpc_socp(0, 2, stages, 5, 3)
    probs = [(base, {}), (variant(base, 1), {}), (other, {}), (variant(base, 2), {"precision": "mixed"}),
             (variant(base, 3, last=1.01), {}), (variant(base, 4, q=0.5), {}), (variant(base, 5), {"max_iter": 4}),
             (variant(other, 6), {})]
    handles, keep = [], []
    for p, kw in probs:
        h, k = HC._setup(p, HC.default_settings(**kw))
        handles.append(h if isinstance(h, C.c_void_p) else C.c_void_p(h))
        keep.append(k)
    sizes = [(p.n, p.m) for p, _ in probs]
    order = list(range(len(probs))) + [1]
    ask = [i != 2 for i in order[:-1]] + [True]
    res, outs = solve([handles[i] for i in order], [sizes[i] for i in order], ask)
    for j, i in enumerate(order):
        r1, o1 = solve([handles[i]], [sizes[i]])
        for f in ("status", "iterations", "obj_primal", "obj_dual", "res_primal", "res_dual", "n", "m"):
            assert getattr(res[j], f) == getattr(r1[0], f), (j, i, f)
        for a, b in zip(outs[j], o1[0]):
            assert np.isnan(a).all() if not ask[j] else np.array_equal(a, b), (j, i)
    assert res[6].status != res[0].status   # stopped at four iterations
    assert (outs[0][0] != outs[1][0]).any() and (outs[0][0] != outs[4][0]).any()
    for h in handles:
        HC.lib().hc_destroy(h)
