"""Performance cases of the LQT library: the calls a user's program makes, over the sizes it makes
them with.

Every case is a dict of plain values: what is called (`kind`), the problem's sizes and options, and
how its inputs are drawn.  The kinds are

  solve   lqt.solve into kept outputs and workspace (all stages in one call)
  stages  an element build, lqt.scan_value and a trajectory call, one after another
  dense   lqt.dense_output on the solve's boundary values
  grad    lqt.solve_trajectory and the gradients of a tracking loss on it (forward and backward)
  plan    one launch of a tuned, graph-captured plan over many problems of uneven horizons

Problems are those of the package's workloads: the point mass in nx / 2 axes (`mass`), the random
stable system with constant coefficients (`stable`) or with F(t) sampled (`varying`), with L(t) and
a drift c(t) sampled too where a case says so; references are sums of sinusoids.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2212_11744_amd import lqt
from paper_2212_11744_amd import workloads as W

DTYPES = {"f64": torch.float64, "f32": torch.float32}
HORIZON = 10.0


def _case(kind, system, nx, nu, T, n, dtype="f64", batch=1, **more):
    c = {"kind": kind, "system": system, "nx": nx, "nu": nu, "T": T, "n": n, "dtype": dtype,
         "batch": batch, "L_sampled": False, "drift": False, "lti": False}
    c.update(more)
    return c


def listed():
    return [
        # a short horizon re-solved again and again (receding-horizon control): launches and latency
        {"name": "solve_short", **_case("solve", "mass", 4, 2, 64, 10)},
        # an ordinary planning horizon with time-varying coefficients, odd sizes throughout
        {"name": "solve_varying_odd", **_case("solve", "varying", 3, 2, 20011, 3, L_sampled=True,
                                              drift=True)},
        # the smaller benchmark horizon
        {"name": "solve_2p16", **_case("solve", "mass", 4, 2, 2 ** 16, 4)},
        # the benchmark: a million blocks, FP64 and FP32
        {"name": "solve_2p20", **_case("solve", "mass", 4, 2, 2 ** 20, 4)},
        {"name": "solve_2p20_f32", **_case("solve", "mass", 4, 2, 2 ** 20, 4, "f32")},
        # a caller that knows its problem to be time-invariant says so
        {"name": "solve_lti", **_case("solve", "stable", 4, 2, 200001, 4, lti=True)},
        # a larger state (one wavefront per block): the benchmark's nx = 16 and an odd FP32 size
        {"name": "solve_nx16", **_case("solve", "varying", 16, 4, 2 ** 14, 4)},
        {"name": "solve_nx7_f32", **_case("solve", "stable", 7, 3, 3001, 3, "f32", batch=2,
                                          drift=True)},
        # learning weights and references through the solver: forward and backward, a batch
        {"name": "grad_batch", **_case("grad", "mass", 4, 2, 2 ** 16, 4, batch=16)},
        # the stages called one by one: split blocks, value scan, Method 2 trajectory
        {"name": "stages_method2", **_case("stages", "mass", 4, 2, 100003, 4, build="split",
                                           traj="method2")},
        # values at every integration node, for plots and simulation
        {"name": "dense_2p18", **_case("dense", "mass", 4, 2, 2 ** 18, 4)},
        # a fleet of problems of several sizes and uneven horizons, one graph replay
        {"name": "plan_mix", **_case("plan", "mix", 0, 0, 8192, 4, batch=192)},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "wave", "grad", "stages", "dense", "plan"])
    dtype = rng.choice(["f64", "f64", "f32"])
    n = rng.randint(1, 6)
    if kind == "plan":
        return _case("plan", "mix", 0, 0, _log_int(rng, 600, 6000), 4, batch=rng.randint(12, 160))
    if kind == "wave":  # nx 5 .. 16
        nx = rng.randint(5, 16)
        system = rng.choice(["stable", "varying"])
        return _case("solve", system, nx, rng.randint(1, min(nx, 8)), _log_int(rng, 40, 12000),
                     min(n, 4), dtype, drift=rng.random() < 0.3, L_sampled=rng.random() < 0.2)
    nx = rng.randint(1, 4)
    nu = rng.randint(1, nx)
    system = rng.choice(["mass", "mass", "stable", "varying"])
    if system == "mass":
        nx = 2 * ((nx + 1) // 2)
        nu = nx // 2
    more = {}
    if system != "mass":
        more["drift"] = rng.random() < 0.3
        more["L_sampled"] = rng.random() < 0.2
    if kind == "solve":
        if system == "stable" and rng.random() < 0.5:
            more = {"lti": True}
        return _case("solve", system, nx, nu, _log_int(rng, 16, 700000), n, dtype, **more)
    if kind == "grad":
        batch = rng.choice([1, 3, 16])
        return _case("grad", system, nx, nu, _log_int(rng, 64, 600000 // batch), min(n, 4), dtype,
                     batch, **more)
    if kind == "stages":
        return _case("stages", system, nx, nu, _log_int(rng, 64, 100000), min(n, 4), dtype,
                     build=rng.choice(["backward", "forward", "split"]),
                     traj=rng.choice(["method1", "method2"]), **more)
    return _case("dense", system, nx, nu, _log_int(rng, 64, 200000), min(n, 4), dtype, **more)


# --------------------------------------------------------------------------------------------
# Inputs.
# --------------------------------------------------------------------------------------------
def _sinusoids(rng, ts, axes, terms=4, amp=(0.5, 2.0), freq=(0.1, 1.0), derivative=False):
    """Sums of sinusoids at times ts on the GPU, [ts.size, axes] (and their derivatives)."""
    y = torch.empty(ts.numel(), axes, dtype=torch.float64, device=ts.device)
    dy = torch.empty_like(y) if derivative else None
    for i in range(axes):
        a, f, ph = (rng.uniform(*amp, terms), rng.uniform(*freq, terms),
                    rng.uniform(0, 2 * np.pi, terms))
        col, dcol = torch.zeros_like(ts), torch.zeros_like(ts)
        for k in range(terms):
            w = 2 * np.pi * f[k]
            arg = ts * w + ph[k]
            col += a[k] * torch.sin(arg)
            if derivative:
                dcol += a[k] * w * torch.cos(arg)
        y[:, i] = col
        if derivative:
            dy[:, i] = dcol
    return torch.cat([y, dy], dim=1) if derivative else y


def _problem(case, seed) -> lqt.DeviceProblem:
    """The case's batch of problems on the GPU: small matrices from the package's generators,
    sampled inputs evaluated on the GPU."""
    nx, nu, T, n, B = (case[k] for k in ("nx", "nu", "T", "n", "batch"))
    dtype = DTYPES[case["dtype"]]
    system = case["system"]
    t = torch.linspace(0, HORIZON, T + 1, dtype=torch.float64, device="cuda")
    h = (t[1:] - t[:-1]) / n
    ts = torch.cat([(t[:-1, None] + torch.arange(2 * n, device="cuda") * (h[:, None] / 2)).reshape(-1),
                    t[-1:]])
    to = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=dtype, device="cuda")
    small = {k: [] for k in ("Q", "R", "Qf", "x0")}
    r, c, F, L = [], [], None, None
    for b in range(B):
        rng = np.random.default_rng([seed, b])
        if system == "mass":
            p = W.point_mass(seed * 1000 + b, 1, n, 0.0, HORIZON, d=nx // 2)
            r.append(_sinusoids(rng, ts, nx // 2, derivative=True).to(dtype))
        else:
            p = W.random_stable(seed * 1000 + b, nx, nu, 1, n, 0.0, HORIZON,
                                time_varying=system == "varying")
            r.append(_sinusoids(rng, ts, nx).to(dtype))
        for k in small:
            small[k].append(getattr(p, k))
        if case["drift"]:
            c.append((0.3 * _sinusoids(rng, ts, nx, terms=2)).to(dtype))
        if b == 0:  # constant F and L are shared by a batch; sampled ones are repeated
            F0, L0 = p.F_of_t(np.zeros(1))[0] if p.F_of_t else p.F, p.L
            F1 = (p.F_of_t(np.array([0.5 * np.pi]))[0] - F0) if system == "varying" else None
    if system == "varying":
        F = (to(F0).double() + torch.sin(ts)[:, None, None] * to(F1).double()).to(dtype)
        F = F.expand(B, *F.shape).contiguous()
    else:
        F = to(F0)
    if case["L_sampled"]:
        L = (to(L0).double() * (1 + 0.2 * torch.cos(ts))[:, None, None]).to(dtype)
        L = L.expand(B, *L.shape).contiguous()
    else:
        L = to(L0)
    r = torch.stack(r)
    return lqt.DeviceProblem(
        nx, nu, T, n, B, dtype, t.to(dtype).expand(B, T + 1).contiguous(), F, L,
        *(to(np.stack(small[k])) for k in ("Q", "R")), r.contiguous(), to(np.stack(small["Qf"])),
        r[:, -1].contiguous(), to(np.stack(small["x0"])), torch.stack(c) if c else None,
        system == "varying", bool(case["L_sampled"]), bool(case["lti"]))


def _target(case, seed, t):
    rng = np.random.default_rng([seed, 77])
    ax = max(1, case["nx"] // 2)
    g = _sinusoids(rng, t.double()[0], ax, terms=3, freq=(0.05, 0.5), derivative=True)
    return g[:, :case["nx"]].to(t.dtype).expand(case["batch"], -1, -1).contiguous()


def _mix_horizons(case):
    """The horizons are part of the case, not of its inputs: U{256 .. T}."""
    return np.random.default_rng(case["batch"]).integers(256, case["T"] + 1, size=case["batch"])


def _mix(case, seed):
    """The package's batched mix (its sizes, systems and block length) at these horizons."""
    n, out = case["n"], []
    for i, T in enumerate(int(t) for t in _mix_horizons(case)):
        nx, sub, tf = (2, 4, 8)[i % 3], seed * 1000 + i, T * 10.0 / 1024
        out.append(W.point_mass(sub, T, n, 0.0, tf, d=nx // 2) if i % 2 == 0 else
                   W.random_stable(sub, nx, nx // 2, T, n, 0.0, tf, time_varying=False))
    return out


BUILDS = {"backward": lqt.build_elements, "forward": lqt.build_elements_forward,
          "split": lqt.build_elements_split}
TRAJS = {"method1": (lqt.forward_traj, lqt.CALL_FORWARD_TRAJ),
         "method2": (lqt.forward_traj_method2, lqt.CALL_TRAJ_METHOD2)}


def prepare(case, seed):
    kind = case["kind"]
    if kind == "plan":
        return {"kind": kind, "plan": lqt.BatchedSolve(_mix(case, seed), autotune=True, graph=True)}
    dp = _problem(case, seed)
    st = {"kind": kind, "prob": dp}
    new = lambda *s: torch.empty(dp.batch, *s, dtype=dp.dtype, device="cuda")
    T, nx, nu = dp.T, dp.nx, dp.nu
    if kind == "solve":
        st["out"] = {"S": new(T + 1, nx, nx), "v": new(T + 1, nx), "x": new(T + 1, nx),
                     "u": new(T + 1, nu)}
        st["ws"] = lqt.workspace(dp, lqt.CALL_SOLVE)
    elif kind == "stages":
        st["build"] = BUILDS[case["build"]]
        st["traj"], call = TRAJS[case["traj"]]
        st["elts"] = lqt.empty_elements(dp)
        st["S"], st["v"] = new(T + 1, nx, nx), new(T + 1, nx)
        st["x"], st["u"] = new(T + 1, nx), new(T + 1, nu)
        st["ws"] = [lqt.workspace(dp, c) for c in (lqt.CALL_BUILD, lqt.CALL_SCAN_VALUE, call)]
    elif kind == "dense":
        st["solved"] = lqt.solve(dp)
        nodes = dp.n * T + 1
        st["out"] = {"S": new(nodes, nx, nx), "v": new(nodes, nx), "x": new(nodes, nx),
                     "u": new(nodes, nu)}
        st["ws"] = lqt.workspace(dp, lqt.CALL_BUILD)
    else:
        st["target"] = _target(case, seed, dp.t)
        st["leaves"] = [getattr(dp, k).requires_grad_() for k in ("Q", "R", "r", "x0", "Qf", "rf")]
    return st


def run(st):
    kind = st["kind"]
    if kind == "plan":
        st["plan"].launch()
        return [{k: c[k] for k in ("S", "v", "x", "u")} for c in st["plan"].classes]
    dp = st["prob"]
    if kind == "solve":
        return lqt.solve(dp, st["out"], st["ws"])
    if kind == "stages":
        wb, wv, wt = st["ws"]
        st["build"](dp, st["elts"], wb)
        lqt.scan_value(dp, st["elts"], st["S"], st["v"], wv)
        st["traj"](dp, st["elts"], st["S"], st["v"], st["x"], st["u"], wt)
        return {k: st[k] for k in ("S", "v", "x", "u")}
    if kind == "dense":
        s = st["solved"]
        return lqt.dense_output(dp, s["S"], s["v"], s["x"], st["out"], st["ws"])
    x = lqt.solve_trajectory(*st["leaves"], dp)
    loss = (x - st["target"]).square().sum()
    g = torch.autograd.grad(loss, st["leaves"])
    return {"x": x.detach(), **dict(zip(("Q", "R", "r", "x0", "Qf", "rf"), g))}


# --------------------------------------------------------------------------------------------
# Work a pass cannot do without: every input read once, every output written once, and the
# arithmetic of the sequential method (FMA = 2).
# --------------------------------------------------------------------------------------------
def _rk4_flops(nx, nu, n, drift):
    ns = nx * (nx + 1) // 2
    stage = (2 * nx ** 3 + 4 * nx ** 2 + nx + nx * nx * nu + ns * nu + ns
             + (nx ** 2 if drift else 0) + nx ** 2 * (nx + 1) + 2 * nx ** 2 + 2 * nx + 2 * ns)
    return 2 * 4 * n * stage


def _fold_flops(nx, nu):
    # I + C S, the solve with nx + 1 right-hand sides, S', v', x and u
    return 2 * (3 * nx ** 3 + nx ** 3 + nx ** 2 * (nx + 1) + 6 * nx ** 2 + nx * (nx + nu))


def work(case):
    if case["kind"] == "plan":
        nbytes = flops = 0
        for i, T in enumerate(_mix_horizons(case)):
            nx = (2, 4, 8)[i % 3]
            w = work(_case("solve", "stable", nx, nx // 2, int(T), case["n"]))
            nbytes += w["bytes"]
            flops += w["flops"]
        return {"bytes": nbytes, "flops": flops}
    nx, nu, n = case["nx"], case["nu"], case["n"]
    blocks = case["batch"] * case["T"]
    es = 8 if case["dtype"] == "f64" else 4
    F_s = nx * nx if case["system"] == "varying" else 0
    L_s = nx * nu if case["L_sampled"] else 0
    sample = nx + F_s + L_s + (nx if case["drift"] else 0)
    inputs = 2 * n * sample + 1
    bound = nx * nx + 2 * nx + nu
    build = _rk4_flops(nx, nu, n, case["drift"])
    if case["lti"]:
        build = 2 * 2 * (2 * n + 1) * nx * nx
    per = {"solve": (inputs + bound, build + _fold_flops(nx, nu)),
           "stages": (inputs + bound, build + _fold_flops(nx, nu)),
           "dense": (inputs + bound + n * bound, build + n * _fold_flops(nx, nu)),
           # forward, its adjoint (twice the arithmetic), x and the gradient of r written
           "grad": (inputs + 2 * nx + 2 * n * nx, 3 * (build + _fold_flops(nx, nu)))}
    b, f = per[case["kind"]]
    return {"bytes": es * b * blocks, "flops": f * blocks}


# --------------------------------------------------------------------------------------------
# The same outputs in 64 bits, in plain torch: Theorems 8 and 9 by RK4, Lemma 7 in a recursive
# scan, the closed-loop maps composed in another, and autograd for the gradients.
# --------------------------------------------------------------------------------------------
def _solve_lin(M, B):
    """M^{-1} B by Gauss-Jordan elimination (M = I + C J: no pivoting needed)."""
    m = M.shape[-1]
    eye = torch.eye(m, dtype=torch.bool, device=M.device)
    X = torch.cat([M, B], dim=-1)
    for c in range(m):
        row = X[..., c:c + 1, :] / X[..., c:c + 1, c:c + 1]
        X = torch.where(eye[c][:, None], row, X - X[..., :, c:c + 1] * row)
    return X[..., m:]


def _mv(A, x):
    return (A @ x[..., None])[..., 0]


def _tr(A):
    return A.transpose(-1, -2).contiguous()


def _combine(a, b):
    """Lemma 7: a on the earlier interval, b on the later one; tuples (A, b, C, eta, J)."""
    A1, b1, C1, e1, J1 = a
    A2, b2, C2, e2, J2 = b
    n = A1.shape[-1]
    I = torch.eye(n, dtype=A1.dtype, device=A1.device)
    X = _solve_lin(I + C1 @ J2, torch.cat([A1, C1, (b1 + _mv(C1, e2))[..., None]], -1))
    Y, D, g = X[..., :n], X[..., n:2 * n], X[..., 2 * n]
    Yt = _tr(Y)
    return (A2 @ Y, _mv(A2, g) + b2, A2 @ D @ _tr(A2) + C2, _mv(Yt, e2 - _mv(J2, b1)) + e1,
            Yt @ J2 @ A1 + J1)


def _suffix(e, comb):
    """Suffix products along dim 1 of a tuple of tensors."""
    m = e[0].shape[1]
    if m == 1:
        return e
    h = m // 2
    left, right = tuple(x[:, 0:2 * h:2] for x in e), tuple(x[:, 1:2 * h:2] for x in e)
    pair = comb(left, right)
    if m % 2:
        pair = tuple(torch.cat([p, x[:, -1:]], 1) for p, x in zip(pair, e))
    s = _suffix(pair, comb)
    # odd positions 2 i + 1: their own element and the suffix that begins after it
    k = s[0].shape[1] - 1
    odd = comb(tuple(x[:, :k] for x in right), tuple(x[:, 1:] for x in s)) if k else None
    out = []
    for i, x in enumerate(e):
        o = odd[i] if k else x[:, :0]
        if k < h:
            o = torch.cat([o, x[:, -1:]], 1)
        y = torch.stack([s[i][:, :h], o], 2).flatten(1, 2)
        out.append(torch.cat([y, s[i][:, -1:]], 1) if m % 2 else y)
    return tuple(out)


class _Exact:
    """One batch of problems in float64 (tensors [B, ...])."""

    def __init__(self, dp, rows=slice(None), **over):
        d = lambda x: None if x is None else x.detach().double()
        self.n, self.T, self.nx = dp.n, dp.T, dp.nx
        self.t, self.r, self.Q, self.R, self.Qf, self.rf, self.x0 = (
            d(getattr(dp, k))[rows] for k in ("t", "r", "Q", "R", "Qf", "rf", "x0"))
        self.c = d(dp.c)[rows] if dp.c is not None else None
        self.F = d(dp.F)[rows] if dp.F_sampled else d(dp.F)
        self.L = d(dp.L)[rows] if dp.L_sampled else d(dp.L)
        self.Fs, self.Ls = dp.F_sampled, dp.L_sampled
        for k, v in over.items():
            setattr(self, k, v)
        self.Ri = torch.linalg.inv(self.R.cpu()).to(self.R.device)
        self.h = (self.t[:, 1:] - self.t[:, :-1]) / self.n

    def at(self, j):
        """F, G, c, r at sample 2 n k + j of every block."""
        s = slice(j, j + 2 * self.n * (self.T - 1) + 1, 2 * self.n)
        F = self.F[:, s] if self.Fs else self.F
        L = self.L[:, s] if self.Ls else self.L[None, None]
        G = (L @ self.Ri[:, None]) @ _tr(L)
        return F, G, None if self.c is None else self.c[:, s], self.r[:, s]

    def rk4(self, f, y, sign, j0, n):
        """n RK4 steps of sign * h from sample j0."""
        h = self.h
        hm, hv = (sign * h)[..., None, None], (sign * h)[..., None]
        H = [hm if x.dim() == 4 else hv for x in y]
        step = 2 if sign > 0 else -2
        for m in range(n):
            a, mid, b = j0 + step * m, j0 + step * m + step // 2, j0 + step * (m + 1)
            k1 = f(y, *self.at(a))
            k2 = f([v + 0.5 * e * k for v, e, k in zip(y, H, k1)], *self.at(mid))
            k3 = f([v + 0.5 * e * k for v, e, k in zip(y, H, k2)], *self.at(mid))
            k4 = f([v + e * k for v, e, k in zip(y, H, k3)], *self.at(b))
            y = [v + e * ((p + s) + 2 * (q + r)) / 6
                 for v, e, p, q, r, s in zip(y, H, k1, k2, k3, k4)]
            yield y

    def start(self):
        B, T, n = self.t.shape[0], self.T, self.nx
        z = lambda *s: torch.zeros(B, T, *s, dtype=torch.float64, device=self.t.device)
        A = torch.eye(n, dtype=torch.float64, device=self.t.device).expand(B, T, n, n)
        return [A, z(n), z(n, n), z(n), z(n, n)]

    def back(self, y, F, G, c, r):
        A, _, _, e, J = y
        K = G @ J - F
        w = _mv(G, e) if c is None else _mv(G, e) + c
        Q = self.Q[:, None]
        de = _mv(_tr(K), e) - _mv(Q, r)
        if c is not None:
            de = de + _mv(J, c)
        return A @ K, -_mv(A, w), -(A @ G @ _tr(A)), de, -Q + J @ K - _tr(F) @ J

    def fwd(self, y, F, G, c, r):
        A, b, C, _, _ = y
        Q = self.Q[:, None]
        M = F - C @ Q
        db = _mv(M, b) + _mv(C, _mv(Q, r))
        if c is not None:
            db = db + c
        At = _tr(A)
        return M @ A, db, G + M @ C + C @ _tr(F), _mv(At, _mv(Q, r - b)), At @ Q @ A

    def elements(self, build="backward"):
        n = self.n
        m = {"backward": 0, "split": n // 2, "forward": n}[build]
        f, b = self.start(), self.start()
        for f in self.rk4(self.fwd, f, 1, 0, m):
            pass
        for b in self.rk4(self.back, b, -1, 2 * n, n - m):
            pass
        return tuple(b) if m == 0 else tuple(f) if m == n else _combine(f, b)

    def values(self, el):
        B, n = self.t.shape[0], self.nx
        Qf = self.Qf[:, None]
        z = torch.zeros_like(Qf)
        last = (z, z[..., 0], z, _mv(Qf, self.rf[:, None]), Qf)
        s = _suffix(tuple(torch.cat([x, y], 1) for x, y in zip(el, last)), _combine)
        return s[4], s[3]

    def trajectory(self, el, S, v):
        A, b, C = el[:3]
        I = torch.eye(self.nx, dtype=torch.float64, device=A.device)
        X = _solve_lin(I + C @ S[:, 1:], torch.cat([A, (b + _mv(C, v[:, 1:]))[..., None]], -1))
        P, q = X[..., :-1], X[..., -1]
        rev = lambda e: tuple(x.flip(1) for x in e)
        # reversed in time, prefixes are suffixes whose later part acts first
        comb = lambda a, c: (a[0] @ c[0], _mv(a[0], c[1]) + a[1])
        P, q = rev(_suffix(rev((P, q)), comb))
        x0 = self.x0[:, None]
        return torch.cat([x0, _mv(P, x0) + q], 1)

    def gain(self, j0, step):
        L = self.L[:, j0::step] if self.Ls else self.L[None, None]
        return self.Ri[:, None] @ _tr(L)

    def control(self, S, v, x, step):
        return -_mv(self.gain(0, step), _mv(S, x) - v)

    def solve(self, build="backward"):
        el = self.elements(build)
        S, v = self.values(el)
        x = self.trajectory(el, S, v)
        return S, v, x

    def dense(self):
        S, v, x = self.solve()
        n, T, B = self.n, self.T, self.t.shape[0]

        def f(y, F, G, c, r):
            S, v = y
            Q, Ft = self.Q[:, None], _tr(F)
            P = S @ G
            dv = -_mv(Q, r) - _mv(Ft, v) + _mv(P, v)
            if c is not None:
                dv = dv + _mv(S, c)
            return -Ft @ S - S @ F - Q + P @ S, dv

        Ss, vs, xs = [S[:, :-1]], [v[:, :-1]], [x[:, :-1]]
        back = list(self.rk4(f, [S[:, 1:], v[:, 1:]], -1, 2 * n, n - 1))
        I = torch.eye(self.nx, dtype=torch.float64, device=S.device)
        for (A, b, C, _, _), (Sm, vm) in zip(self.rk4(self.fwd, self.start(), 1, 0, n - 1),
                                             reversed(back)):
            rhs = _mv(A, x[:, :-1]) + b + _mv(C, vm)
            Ss.append(Sm)
            vs.append(vm)
            xs.append(_solve_lin(I + C @ Sm, rhs[..., None])[..., 0])
        join = lambda a, end: torch.cat([torch.stack(a, 2).flatten(1, 2), end[:, -1:]], 1)
        Sd, vd, xd = join(Ss, S), join(vs, v), join(xs, x)
        return {"S": Sd, "v": vd, "x": xd, "u": self.control(Sd, vd, xd, 2)}


def _exact_grad(case, dp, target):
    out = {k: [] for k in ("x", "Q", "R", "r", "x0", "Qf", "rf")}
    per = max(1, 2 ** 18 // case["T"])
    names = ("Q", "R", "r", "x0", "Qf", "rf")
    for b in range(0, case["batch"], per):
        rows = slice(b, b + per)
        leaf = {k: getattr(dp, k).detach()[rows].double().requires_grad_() for k in names}
        E = _Exact(dp, rows, **leaf)
        E.Ri = torch.linalg.inv(leaf["R"].cpu()).to("cuda")
        x = E.solve()[2]
        g = torch.autograd.grad((x - target[rows].double()).square().sum(), list(leaf.values()))
        for k, v in zip(names, g):
            out[k].append(0.5 * (v + v.transpose(-1, -2)) if k in ("Q", "R", "Qf") else v)
        out["x"].append(x.detach())
    return {k: torch.cat(v) for k, v in out.items()}


def _exact_plan(case, seed):
    """Problems of one class together, shorter horizons padded with identity elements."""
    probs, outs = _mix(case, seed), []
    for nx in dict.fromkeys(p.nx for p in probs):
        mem = [p for p in probs if p.nx == nx]
        Tm = max(p.T for p in mem)
        els = []
        to = lambda a: torch.as_tensor(np.asarray(a), dtype=torch.float64, device="cuda")
        for p in mem:
            E = _Exact(lqt.DeviceProblem.from_problems([p]))
            el = E.elements()
            pad = Tm - p.T
            eye = torch.eye(nx, dtype=torch.float64, device="cuda").expand(1, pad, nx, nx)
            els.append(tuple(torch.cat([x, eye if i == 0 else torch.zeros_like(x[:, :1]).expand(
                1, pad, *x.shape[2:])], 1) for i, x in enumerate(el)))
        el = tuple(torch.cat(x) for x in zip(*els))
        Z = _Exact.__new__(_Exact)
        Z.nx = nx
        Z.t = to(np.zeros((len(mem), Tm + 1)))
        Z.Qf, Z.rf, Z.x0, R, L = (to(np.stack([getattr(p, k) for p in mem]))
                                  for k in ("Qf", "rf", "x0", "R", "L"))
        S, v = Z.values(el)
        x = Z.trajectory(el, S, v)
        K = torch.linalg.inv(R.cpu()).to("cuda") @ _tr(L)
        u = -_mv(K[:, None], _mv(S, x) - v)
        outs.append({k: torch.cat([a[i, :p.T + 1] for i, p in enumerate(mem)])
                     for k, a in (("S", S), ("v", v), ("x", x), ("u", u))})
    return outs


def exact(case, seed):
    kind = case["kind"]
    if kind == "plan":
        return _exact_plan(case, seed)
    dp = _problem(case, seed)
    if kind == "grad":
        return _exact_grad(case, dp, _target(case, seed, dp.t))
    with torch.no_grad():
        E = _Exact(dp)
        if kind == "dense":
            return E.dense()
        S, v, x = E.solve(case.get("build", "backward"))
        return {"S": S, "v": v, "x": x, "u": E.control(S, v, x, 2 * dp.n)}
