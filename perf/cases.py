"""Performance cases: the conic solves a user of hipcone runs, over the range of
sizes, cone types, precisions and call forms that the library serves.

Every case builds its problem from a seed with the generators of
`paper_2412_19027_amd.workloads`, keeps the handle a program keeps (a set-up and
bound `Solver`, or set-up handles for the batched engine) and times one whole
call: new data where the program has new data, the solve, the solution read back.
Solves run to the default tolerances, or under an iteration budget
(`max_iter`, the anytime use: the iterate after so many steps).
"""
import ctypes as C
import math

import numpy as np
import torch

from paper_2412_19027_amd import hipcone as HC
from paper_2412_19027_amd import workloads as W


def listed():
    return [
        # the smallest call: a dense LP of 50 variables; launches and host round trips are all of it
        {"name": "lp_small", "kind": "lp", "n": 50, "m": 100},
        # a controller's re-solve with a new measured state (new right-hand side), short and long horizon
        {"name": "mpc_short", "kind": "mpc", "T": 20, "nx": 6, "nu": 3},
        {"name": "mpc_long", "kind": "mpc", "T": 100, "nx": 12, "nu": 6},
        # many controllers at once on the batched engine: 16 plants, 16 measured states each
        {"name": "mpc_batch", "kind": "batch", "plants": 16, "states": 16, "T": 40},
        # one Newton system by itself: scaling, factorisation and refined solve at a given interior iterate
        {"name": "kkt_step", "kind": "kkt", "nx": 700, "rank": 20},
        # the factor-model SOCP: a mid-size solve to the default tolerances (odd sizes), the full
        # benchmark size under an iteration budget, and FP32 factors with FP64 refinement
        {"name": "socp_mid", "kind": "socp", "nx": 4983, "rank": 20, "precision": "fp64", "max_iter": 200},
        {"name": "socp_full", "kind": "socp", "nx": 20000, "rank": 20, "precision": "fp64", "max_iter": 5},
        {"name": "socp_mixed", "kind": "socp", "nx": 10000, "rank": 20, "precision": "mixed", "max_iter": 10},
        # l1 logistic regression: 200,000 exponential cones, 100,500 leaf blocks, a dense tail of 500
        {"name": "logreg", "kind": "logreg", "samples": 100000, "features": 500, "max_iter": 10},
        # PSD cones of side 10 with power cones, full configuration
        {"name": "psd_pow", "kind": "psd_pow", "n": 5000, "pow": 20000, "psd": 2000, "side": 10, "max_iter": 8},
        # PSD cones of three sides up to the largest one taken
        {"name": "psd_sides", "kind": "psd_mixed", "n": 2000, "per_side": 30, "max_iter": 8},
        # entropy maximisation: dense inequality rows, exponential cones, leaf blocks
        {"name": "entropy", "kind": "entropy", "n": 2000, "max_iter": 8},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["lp", "mpc", "mpc", "batch", "kkt", "socp", "socp", "logreg", "psd_pow", "psd_mixed", "entropy"])
    if kind == "lp":
        n = _log(rng, 20, 400)
        return {"kind": kind, "n": n, "m": 2 * n + rng.randrange(1, 50)}
    if kind == "mpc":
        return {"kind": kind, "T": _log(rng, 10, 100), "nx": rng.randint(4, 12), "nu": rng.randint(2, 6)}
    if kind == "batch":
        return {"kind": kind, "plants": _log(rng, 1, 16), "states": _log(rng, 1, 24), "T": _log(rng, 10, 60)}
    if kind == "kkt":
        return {"kind": kind, "nx": _log(rng, 60, 900), "rank": rng.randint(3, 24)}
    if kind == "socp":
        return {"kind": kind, "nx": _log(rng, 500, 12000), "rank": rng.randint(5, 24),
                "precision": rng.choice(["fp64", "mixed"]), "max_iter": 8}
    if kind == "logreg":
        return {"kind": kind, "samples": _log(rng, 1000, 100000), "features": _log(rng, 40, 500), "max_iter": 10}
    if kind == "psd_pow":
        f = math.exp(rng.uniform(math.log(0.05), 0.0))
        return {"kind": kind, "n": int(5000 * f), "pow": int(20000 * f), "psd": int(2000 * f),
                "side": rng.randint(3, 10), "max_iter": 8}
    if kind == "psd_mixed":
        per = _log(rng, 3, 30)
        return {"kind": kind, "n": 60 * per + rng.randrange(0, 60), "per_side": per, "max_iter": 8}
    return {"kind": kind, "n": _log(rng, 200, 2500), "max_iter": 8}


def _problem(case, seed):
    k = case["kind"]
    if k == "lp":
        return W.tiny_lp(seed, case["n"], case["m"])
    if k == "mpc":
        return W.mpc_socp(seed, 0, case["T"], case["nx"], case["nu"])
    if k in ("socp", "kkt"):
        nx = case["nx"]
        return W.sparse_socp(seed, nx, case["rank"], nx // 2, 3 * nx // 2, 2 * nx)
    if k == "logreg":
        return W.logreg_exp(seed, case["samples"], case["features"])
    if k == "psd_pow":
        return W.psd_pow(seed, case["n"], case["pow"], case["psd"], case["side"])
    if k == "psd_mixed":
        return W.psd_mixed(seed, case["n"], (8, 20, 32), case["per_side"])
    return W.entropy_max(seed, case["n"])


class _Batch:
    """Set-up handles for hc_solve_batch and the result records with the callers' buffers."""

    def __init__(self, probs):
        L = HC.lib()
        self._destroy = L.hc_destroy
        st = HC.default_settings()
        self.handles = (C.c_void_p * len(probs))()
        self.res = (HC.hc_result * len(probs))()
        self.x, self.s, self.z = (np.zeros(sum(getattr(p, a) for p in probs)) for a in ("n", "m", "m"))
        o = 0, 0

        def ptr(a, t):
            return a.ctypes.data_as(C.POINTER(t))
        for i, p in enumerate(probs):
            f = [np.ascontiguousarray(v, dtype=t) for v, t in (
                (p.P.indptr, np.int64), (p.P.indices, np.int32), (p.P.data, np.float64), (p.q, np.float64),
                (p.A.indptr, np.int64), (p.A.indices, np.int32), (p.A.data, np.float64), (p.b, np.float64))]
            cones = (HC.hc_cone * len(p.cones))(*[HC.hc_cone(int(k), int(d), float(a)) for k, d, a in p.cones])
            t = (C.c_int64, C.c_int32, C.c_double, C.c_double) * 2
            pr = HC.hc_problem(p.n, p.m, *[ptr(v, u) for v, u in zip(f, t)], cones, len(p.cones))
            h = C.c_void_p()
            if L.hc_setup(C.byref(h), C.byref(pr), C.byref(st)) != 0:
                raise RuntimeError(L.hc_last_error(None).decode())
            self.handles[i] = h.value
            r = self.res[i]
            r.x, r.s, r.z = ptr(self.x[o[0]:], C.c_double), ptr(self.s[o[1]:], C.c_double), ptr(self.z[o[1]:], C.c_double)
            o = o[0] + p.n, o[1] + p.m

    def solve(self):
        rc = HC.lib().hc_solve_batch(self.handles, len(self.handles), torch.cuda.current_stream().cuda_stream,
                                     torch.cuda.current_device(), self.res)
        if rc != 0:
            raise RuntimeError(HC.lib().hc_last_error(None).decode())
        return {"x": self.x, "s": self.s, "z": self.z, "objective": np.array([r.obj_primal for r in self.res])}

    def __del__(self):
        for h in self.handles:
            self._destroy(h)


def _plants(case, seed):
    """`states` requests on each of `plants` plants of several sizes; a plant's requests differ in the state."""
    rng = np.random.default_rng(seed)
    probs = []
    for i in range(case["plants"]):
        nx = 4 + (5 * i + 3) % 9
        p = W.mpc_socp(seed, i, case["T"], nx, 2 + (3 * i + 2) % 5)
        for _ in range(case["states"]):
            b = p.b.copy()
            b[:nx] = 3.0 * rng.standard_normal(nx)
            probs.append(W.Problem(p.n, p.m, p.P, p.q, p.A, b, p.cones))
    return probs


def _kkt_data(case, seed):
    """An interior iterate and a right-hand side for the SOCP, in the library's row order (zero, nonneg, then the
    second-order cones by component: component j of every cone, then component j + 1)."""
    p = _problem(case, seed)
    rng = np.random.default_rng(seed + 1)
    nx, nz = case["nx"], case["nx"] // 2 + case["rank"]
    nn, ns = 3 * nx // 2, 2 * nx

    def point():
        u = rng.standard_normal((2, ns))
        t = np.sqrt((u * u).sum(0)) + rng.uniform(0.1, 1.0, ns)
        return np.concatenate([rng.uniform(0.1, 1.0, nn), t, u[0], u[1]])
    s = np.concatenate([np.zeros(nz), point()])
    z = np.concatenate([rng.standard_normal(nz), point()])
    soc = nz + nn + np.arange(3 * ns).reshape(ns, 3).T.ravel()
    rows = np.concatenate([np.arange(nz + nn), soc])
    return dict(p=p, s=s, z=z, x=rng.standard_normal(p.n), r1=rng.standard_normal(p.n), r2=rng.standard_normal(p.m),
                rows=rows, nz=nz, nn=nn, ns=ns, mu=float(s @ z) / (nn + ns + 1))


def prepare(case, seed):
    k = case["kind"]
    if k == "batch":
        return {"kind": k, "batch": _Batch(_plants(case, seed))}
    if k == "kkt":
        d = _kkt_data(case, seed)
        d["solver"] = HC.Solver(d["p"], equilibrate=0)   # the iterate below is the user's, unscaled
        d["solver"].set_iterate(d["x"], d["s"], d["z"], 1.0, 1.0)
        return d | {"kind": k}
    p = _problem(case, seed)
    st = {key: case[key] for key in ("precision", "max_iter") if key in case}
    if st.get("precision") == "fp64":
        del st["precision"]
    b = p.b.copy()
    if k == "mpc":   # the state measured now
        b[:case["nx"]] = 3.0 * np.random.default_rng(seed + 1).standard_normal(case["nx"])
    return {"kind": k, "solver": HC.Solver(p, **st), "b": b}


def run(state):
    k = state["kind"]
    if k == "batch":
        return state["batch"].solve()
    s = state["solver"]
    if k == "kkt":
        x, z, _ = s.test_kkt_solve(state["mu"], state["r1"], state["r2"])
        return {"x": x, "z": z}
    if k == "mpc":
        s.update_data(b=state["b"])
    info = s.solve()
    x, sv, z = s.solution()
    return {"x": x, "s": sv, "z": z, "objective": info["obj_primal"]}


def work(case):
    """Flops: one factorisation and four solves of the Schur complement per iteration (one for a KKT step), dense or
    in its band or blocks as the problem's structure has it, its assembly from A, and the cones' own k x k products.
    Bytes: A, the iterate and the direction once per iteration."""
    k = case["kind"]
    it = min(case.get("max_iter", 200), {"lp": 10, "mpc": 8, "batch": 8, "kkt": 1, "socp": 18}.get(k, 200))
    if k == "lp":
        n, m = case["n"], case["m"]
        nnz, f = n * m, n ** 3 / 3 + n * n * m
    elif k in ("mpc", "batch"):
        T = case["T"]
        c = 1 if k == "mpc" else case["plants"] * case["states"]
        nx, nu = (case["nx"], case["nu"]) if k == "mpc" else (8, 4)
        w = 2 * nx + nu
        n, m = c * ((T + 1) * nx + T * nu), c * ((T + 1) * nx + T * (2 * nu + 3))
        nnz, f = c * T * (nx * (nx + nu + 1) + 2 * nu + 2), n * w * w
    elif k in ("socp", "kkt"):
        nx = case["nx"]
        n, m = nx + case["rank"], 8 * nx + case["rank"]
        nnz, f = 6 * 8 * nx + case["rank"] * nx, n ** 3 / 3
    elif k == "logreg":
        N, F = case["samples"], case["features"]
        n, m = 2 * F + 3 * N, 7 * N + 2 * F
        nnz, f = 16 * N, F ** 3 / 3 + N * 120
    elif k == "psd_pow":
        sd = case["side"] * (case["side"] + 1) // 2
        n, m = case["n"], 3 * case["pow"] + sd * case["psd"]
        nnz, f = 8 * m, n ** 3 / 3 + case["psd"] * sd * sd * 64 + case["psd"] * 40 * case["side"] ** 3
    elif k == "psd_mixed":
        n, m = case["n"], case["per_side"] * (36 + 210 + 528)
        nnz = 8 * m
        f = n ** 3 / 3 + case["per_side"] * sum(64 * (s * (s + 1) // 2) ** 2 + 40 * s ** 3 for s in (8, 20, 32))
    else:
        n, m = 2 * case["n"], 1 + case["n"] // 2 + 3 * case["n"]
        nnz, f = case["n"] ** 2 // 2, case["n"] ** 3 / 3 + case["n"] ** 3 / 2
    solves = 4 * 4 * nnz
    return {"bytes": float(it * (12 * nnz + 8 * (4 * n + 8 * m))), "flops": float(it * (f + solves))}


def _lp_optimum(p):
    """min q'x, Ax + s = b, s >= 0 by Mehrotra's method on dense 64-bit matrices, to rounding."""
    A, b, q = p.A.toarray(), p.b, p.q
    m = p.m
    x = np.linalg.lstsq(A, b, rcond=None)[0]
    s = b - A @ x
    s = s + max(1.0, 1.5 * -s.min())
    z = np.ones(m)
    best = (math.inf,)
    for _ in range(60):
        rd, rp, mu = -(q + A.T @ z), b - A @ x - s, s @ z / m
        gap = max(np.abs(rd).max(), np.abs(rp).max(), mu)
        if gap < best[0]:
            best = (gap, x, s, z)
        if mu < 1e-15:
            break
        S = A.T * (z / s) @ A

        def newton(rc):   # z ds + s dz = rc, A dx + ds = rp, A' dz = rd
            rhs = rd - A.T @ ((rc - z * rp) / s)
            dx = np.linalg.solve(S, rhs)
            dx += np.linalg.solve(S, rhs - S @ dx)
            ds = rp - A @ dx
            return dx, ds, (rc - z * ds) / s

        def step(v, dv):
            return min(1.0, 0.995 * (-v[dv < 0] / dv[dv < 0]).min(initial=math.inf))
        _, ds, dz = newton(-s * z)
        sig = (((s + step(s, ds) * ds) @ (z + step(z, dz) * dz)) / m / mu) ** 3
        dx, ds, dz = newton(sig * mu - s * z - ds * dz)
        a, c = step(s, ds), step(z, dz)
        x, s, z = x + a * dx, s + a * ds, z + c * dz
    return best[1:]


def exact(case, seed):
    """The LP's optimum and the KKT system's solution in 64 bits.  The iterate of an interior-point method after a
    given number of steps, or within its tolerance of the optimum, has no such value."""
    k = case["kind"]
    if k == "lp":
        p = _problem(case, seed)
        x, s, z = _lp_optimum(p)
        return {"x": x, "s": s, "z": z, "objective": float(p.q @ x)}
    if k == "kkt":
        d = _kkt_data(case, seed)
        p, nz, nn, ns = d["p"], d["nz"], d["nn"], d["ns"]
        A = torch.from_numpy(p.A.toarray()[d["rows"]]).cuda()
        P = torch.from_numpy(p.P.toarray()).cuda()
        K = torch.zeros(p.n + p.m, p.n + p.m, dtype=torch.float64, device="cuda")
        K[:p.n, :p.n], K[p.n:, :p.n], K[:p.n, p.n:] = P, A, A.t()
        i = p.n + nz + torch.arange(nn, device="cuda")
        K[i, i] = -torch.from_numpy(d["s"][nz:nz + nn] / d["z"][nz:nz + nn]).cuda()
        s, z = (d[v][nz + nn:].reshape(3, ns) for v in "sz")
        J = np.array([1.0, -1.0, -1.0])[:, None]
        rs, rz = np.sqrt((J * s * s).sum(0)), np.sqrt((J * z * z).sum(0))
        sb, zb = s / rs, z / rz
        w = (sb + J * zb) / (2.0 * np.sqrt((1.0 + (sb * zb).sum(0)) / 2.0))   # Nesterov-Todd point
        H = (rs / rz) * (2.0 * w[:, None] * w[None] - np.diag(J[:, 0])[:, :, None])
        o = p.n + nz + nn + torch.arange(ns, device="cuda")
        for a in range(3):
            for c in range(3):
                K[o + a * ns, o + c * ns] = -torch.from_numpy(H[a, c]).cuda()
        r = torch.from_numpy(np.concatenate([d["r1"], d["r2"]])).cuda()[:, None]
        LU, piv = torch.linalg.lu_factor(K)
        v = torch.linalg.lu_solve(LU, piv, r)
        for _ in range(2):
            v = v + torch.linalg.lu_solve(LU, piv, r - K @ v)
        v = v[:, 0].cpu().numpy()
        return {"x": v[:p.n], "z": v[p.n:]}
    return None
