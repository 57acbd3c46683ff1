"""Workloads of the batched AM optimizer that its performance is measured on.

Each case is one call pattern of a program that plans with this library: a
controller that replans a single trajectory or a few hundred, a planner that
optimizes a thousand or several thousand samples, many uneven problems in one
launch, requests through the replanning server, the plain per-sub-step path,
the set-up of a new problem shape, and the residuals and selection of a batch.
Sizes, horizons and iteration counts are those of the seeded workloads in
`paper_2109_13030_amd.inputs` and of the closed-loop controller in
`paper_2109_13030_amd.mpc`, with odd and ragged ones between them.

`prepare` makes what such a program holds before the call (handle, obstacle
table, state buffers), `run` makes one call from fresh coefficients and the
multipliers of the period before, `exact` computes the same results in 64 bits
with plain torch operations from the equations of the method.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2109_13030_amd import am, inputs, mpc

COEF = ("cx", "cc", "cy", "cs", "cpsi")
STATE = COEF + ("lam", "lam_psi")
FC_TOL = 0.05          # [m] collision tolerance of the selection


def listed():
    return [
        # the smallest request: one straight-line trajectory, the 10 iterations
        # of a control period; latency and launches count
        dict(name="replan_one", kind="solve", B=1, m=5, n=10, q=100, nv=11, K=10, tf=30.0, dtype="f32", flags=0,
             tile=2, moving=True),
        # one period of the closed loop with 200 samples: upload the predicted
        # people, solve, residuals, pick the best, read it back
        dict(name="control_period", kind="period", B=200, m=5, n=10, q=100, nv=11, K=10, tf=10.0),
        # small static scene in FP64, 50 iterations (the c1 workload)
        dict(name="static_f64", kind="solve", B=16, m=3, n=4, q=100, nv=11, K=50, tf=30.0, dtype="f64", flags=0,
             tile=2, moving=False),
        # the headline batch (c2): 1000 samples, 5 circles, 10 moving obstacles,
        # with the launch shape its user tunes and the replanning iteration
        # count (over 100 iterations the method amplifies the last bits of FP32
        # up to 1e4-fold, so two correct results differ in the coefficients)
        dict(name="plan_1000", kind="solve", B=1000, m=5, n=10, q=100, nv=11, K=20, tf=30.0, dtype="f32", flags=0,
             tile=1, moving=True),
        # large batch among 20 moving obstacles (c4)
        dict(name="plan_4096", kind="solve", B=4096, m=5, n=20, q=100, nv=11, K=20, tf=30.0, dtype="f32", flags=0,
             tile=2, moving=True),
        # 64 problems of uneven size in one launch (c3)
        dict(name="uneven_64", kind="multi", problems=64, lo=64, hi=1024, q=100, nv=11, K=20, tf=30.0, dtype="f32"),
        # a planner that validates in FP64, odd horizon, ragged batch
        dict(name="plan_f64", kind="solve", B=501, m=5, n=10, q=127, nv=11, K=20, tf=30.0, dtype="f64", flags=0,
             tile=2, moving=True),
        # long robot (8 circles) in a dense scene, the slack reading, a lower
        # degree and an odd horizon
        dict(name="slack_degree7", kind="solve", B=333, m=8, n=40, q=65, nv=8, K=20, tf=20.0, dtype="f32",
             flags=am.XTILDE_SLACK, tile=2, moving=True),
        # eight robots' requests at once through the server (c5 sizes), the
        # final trajectories read back
        dict(name="serve_burst", kind="serve", requests=8, lo=256, hi=2048, q=100, nv=11, K=20, tf=30.0, dtype="f32"),
        # the per-sub-step path at the headline sizes
        dict(name="plain_1000", kind="plain", B=1000, m=5, n=10, q=100, nv=11, K=10, tf=30.0, dtype="f32", flags=0,
             moving=True),
        # a robot meets a new problem shape: set-up, then its first solve
        dict(name="new_shape", kind="setup", B=200, m=5, n=10, q=100, nv=11, K=10, tf=30.0, dtype="f32"),
        # residuals of a large batch and the choice of its best trajectory
        dict(name="residuals_4096", kind="residuals", B=4096, m=5, n=20, q=100, nv=11, tf=30.0, dtype="f32", flags=0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve"] * 6 + ["multi", "multi", "plain", "plain", "residuals", "residuals", "setup", "serve",
                                       "period"])
    q = rng.choice([100, 100, rng.randint(33, 128)])
    nv = rng.choice([11, 11, 11, 8])
    tf = rng.choice([20.0, 30.0, 30.0])
    dtype = rng.choice(["f32", "f32", "f32", "f64"])
    if kind == "multi":
        lo = _log(rng, 1, 128)
        return dict(kind=kind, problems=_log(rng, 2, 64), lo=lo, hi=lo + _log(rng, 16, 512), q=q, nv=nv,
                    K=rng.randint(5, 20), tf=tf, dtype="f32")
    if kind == "serve":
        lo = _log(rng, 1, 512)
        return dict(kind=kind, requests=rng.randint(1, 8), lo=lo, hi=lo + _log(rng, 64, 1024), q=q, nv=nv,
                    K=rng.randint(5, 20), tf=tf, dtype="f32")
    n = rng.choice([_log(rng, 2, 40), 10, 20])
    m = rng.choice([rng.randint(1, 8), 3, 4, 5, 5])
    if kind == "period":
        return dict(kind=kind, B=_log(rng, 1, 1000), m=m, n=min(n, 20), q=q, nv=nv, K=rng.randint(5, 15), tf=10.0)
    if kind == "setup":
        return dict(kind=kind, B=_log(rng, 1, 400), m=m, n=n, q=q, nv=nv, K=rng.randint(5, 10), tf=tf, dtype=dtype)
    if kind == "residuals":
        return dict(kind=kind, B=_log(rng, 1, 4096), m=m, n=n, q=q, nv=nv, tf=tf, dtype=dtype,
                    flags=rng.choice([0, 0, am.XTILDE_SLACK]))
    # the cost of a drawn solve stays below that of the largest listed one
    flags = rng.choice([0, 0, 0, am.XTILDE_SLACK, am.PSI_NO_UNWRAP, am.Q_CS_ZERO])
    if kind == "plain":
        return dict(kind=kind, B=_log(rng, 1, 2048), m=m, n=n, q=q, nv=nv, K=rng.randint(3, 10), tf=tf, dtype=dtype,
                    flags=am.PLAIN_BF16X3 if dtype == "f32" and rng.random() < 0.25 else flags,
                    moving=rng.random() < 0.7)
    B = _log(rng, 1, 4096 if dtype == "f32" else 600)
    return dict(kind=kind, B=B, m=m, n=n, q=q, nv=nv, K=rng.randint(5, 20 if dtype == "f32" else 50), tf=tf, dtype=dtype,
                flags=flags, tile=rng.choice([1, 2, 2, 4] if dtype == "f32" else [1, 2] if n <= 20 else [1]),
                moving=rng.random() < 0.7)


# ---------------------------------------------------------------- inputs

def _seeds(case, seed, count):
    return [int(s.generate_state(1)[0]) for s in np.random.SeedSequence([13030, int(seed)]).spawn(count)]


def _config(case, m, n, moving=True):
    return inputs.Config("case", batch=1, circles=m, n_obs=n, length=1.5 if moving else 1.2,
                         width=0.5 if moving else 0.6, r_circle=0.25 if moving else 0.3, dynamic=moving, iters=1,
                         q=case["q"], nv=case["nv"], tf=case["tf"])


def _problem(case, seed, m, n, B, moving=True, flags=0):
    """One problem and its initial samples, as device arrays of the case's
    type hold them."""
    kp, ki = _seeds(case, seed, 2)
    pb = inputs.make_problem(_config(case, m, n, moving), kp, flags=flags)
    init = inputs.make_initial(pb, B, ki, 0.5 if B > 1 else 0.0)
    if B == 1:   # one trajectory: the straight line, moved a little by the robot's measured state
        init["cx"][0, 3:-3] += np.random.default_rng(ki).normal(0.0, 0.05, case["nv"] - 6)
    return inputs.as_stored(pb, _multipliers(init, ki, cold=case["kind"] == "serve"), case.get("dtype", "f32"))


def _multipliers(init, seed, cold=False):
    """Multipliers as the previous control period left them (a robot's first
    request starts from zero)."""
    init["lam_psi"] = init.pop("lampsi")
    if not cold:
        rng = np.random.default_rng([seed, 1])
        init["lam"] = rng.normal(0.0, 0.1, init["lam"].shape)
        init["lam_psi"] = rng.normal(0.0, 0.02, init["lam_psi"].shape)
    return init


def _uneven(case, seed, count):
    """Problems of uneven batch, circle and obstacle counts: the sizes follow
    from the case, the scenes and samples from the seed."""
    rng = np.random.default_rng([13030, count, case["lo"], case["hi"], case["q"], case["K"]])
    out = []
    for s in _seeds(case, seed, count):
        B = int(rng.integers(case["lo"], case["hi"] + 1))
        m, n = (5, int(rng.integers(5, 31))) if case["kind"] == "serve" else (int(rng.integers(3, 6)),
                                                                               int(rng.integers(2, 21)))
        out.append(_problem(case, s, m, n, B))
    return out


def _heading_samples(pb, init, seed):
    """Coefficients of a batch in mid-optimization: headings that vary, slack
    copies near their cosine and sine, multipliers of the usual size."""
    rng = np.random.default_rng(seed)
    B, nv = init["cx"].shape
    P = _basis(pb)[0]
    init = dict(init)
    cpsi = rng.normal(0.0, 0.4, (B, nv))
    cpsi[:, :3] = cpsi[:, -3:] = 0.0
    pin = np.linalg.pinv(P)
    psi = cpsi @ P.T
    init["cpsi"] = cpsi
    init["cc"] = (np.cos(psi) + rng.normal(0.0, 0.01, psi.shape)) @ pin.T
    init["cs"] = (np.sin(psi) + rng.normal(0.0, 0.01, psi.shape)) @ pin.T
    init["lam"] = rng.normal(0.0, 1.0, (B, 4 * nv))
    init["lam_psi"] = rng.normal(0.0, 0.1, (B, nv))
    return init


class _States:
    """DeviceStates whose coefficients and multipliers share one buffer (and
    their outputs one each), so that a new start is one device copy."""

    def __init__(self, inits, sizes, case, outputs=True, residuals=True):
        q, dt = case["q"], case["dtype"]
        self.st = [am.DeviceState(i, m, n, q, dtype=dt, outputs=outputs, residuals=residuals)
                   for i, (m, n) in zip(inits, sizes)]
        keys = STATE + (("traj",) if outputs else ()) + (("res",) if residuals else ())
        self.all = {k: torch.cat([s.t[k].reshape(-1) for s in self.st]) for k in keys}
        self.fresh = torch.cat([self.all[k] for k in STATE])
        self.live = self.fresh.clone()
        at = 0
        for k in STATE:
            self.all[k] = self.live[at:at + self.all[k].numel()]
            at += self.all[k].numel()
        for k in keys:
            at = 0
            for s in self.st:
                s.t[k] = self.all[k][at:at + s.t[k].numel()].view(s.t[k].shape)
                at += s.t[k].numel()

    def reset(self):
        self.live.copy_(self.fresh)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "multi":
        probs = _uneven(case, seed, case["problems"])
        return dict(kind=kind, K=case["K"], h=[am.Handle.for_problem(pb, case["dtype"]) for pb, _ in probs],
                    p=[am.DeviceProblem(pb, case["dtype"]) for pb, _ in probs],
                    s=_States([i for _, i in probs], [(len(pb["r"]), len(pb["oa"])) for pb, _ in probs], case),
                    ws=torch.empty(am.multi_workspace_size(len(probs)), dtype=torch.uint8, device="cuda"))
    if kind == "serve":
        probs = _uneven(case, seed, case["requests"])
        return dict(kind=kind, K=case["K"], probs=probs, h=[am.Handle.for_problem(pb, case["dtype"]) for pb, _ in probs],
                    srv=am.Server(256 << 20, idle_spin_us=20000), client=0)
    if kind == "period":
        ctl = mpc.MPC(case["B"], iters=case["K"], horizon=case["tf"], q=case["q"], nv=case["nv"], circles=case["m"],
                      n_obs=case["n"], seed=_seeds(case, seed, 1)[0])
        pb, init = _period_inputs(case, seed, ctl)
        ctl.solve_select(pb, init)   # the first period allocates the state
        warm = {k: torch.as_tensor(init[k], dtype=torch.float32, device="cuda") for k in ("lam", "lam_psi")}
        return dict(kind=kind, ctl=ctl, pb=pb, init=init, warm=warm)
    moving = case.get("moving", True)
    pb, init = _problem(case, seed, case["m"], case["n"], case["B"], moving, case.get("flags", 0))
    p = am.DeviceProblem(pb, case["dtype"])
    if kind == "residuals":
        _, init = inputs.as_stored(pb, _heading_samples(pb, init, _seeds(case, seed, 3)[2]), case["dtype"])
    s = _States([init], [(case["m"], case["n"])], case, outputs=kind != "residuals",
                residuals=kind not in ("residuals", "plain"))
    state = dict(kind=kind, K=case.get("K", 0), pb=pb, p=p, s=s, dtype=case["dtype"])
    if kind == "setup":
        return state
    state["h"] = am.Handle.for_problem(pb, case["dtype"])
    if kind == "solve":
        state["h"].tile = case["tile"]
    elif kind == "plain":
        state["ws"] = torch.empty(am.plain_workspace_size(state["h"], case["B"]), dtype=torch.uint8, device="cuda")
    elif kind == "residuals":
        state["res"] = torch.empty((case["B"], am.NRES), dtype=s.live.dtype, device="cuda")
    return state


def run(state):
    kind = state["kind"]
    if kind == "multi":
        s = state["s"]
        s.reset()
        am.solve_multi(state["h"], state["p"], s.st, state["K"], state["ws"])
        return s.all
    if kind == "serve":
        srv, first = state["srv"], state["client"]
        state["client"] += len(state["probs"])   # other robots: cold multipliers
        tickets = [srv.submit(h, pb, first + i, init["cx"].shape[0], state["K"], init)
                   for i, (h, (pb, init)) in enumerate(zip(state["h"], state["probs"]))]
        return [srv.wait(t, traj=True)[2] for t in tickets]
    if kind == "period":
        ctl = state["ctl"]
        for k, v in state["warm"].items():
            ctl.state.t[k].copy_(v)
        idx, coef, fc = ctl.solve_select(state["pb"], state["init"])
        return {"index": idx, "fc": fc, "coef": {k: v.astype(np.float32) for k, v in coef.items()}, "res": ctl.res}
    s = state["s"]
    if kind == "residuals":
        am.residuals(state["h"], state["p"], s.st[0], out=state["res"])
        idx, cost, fc = am.select_best(state["h"], state["res"], FC_TOL)
        return {"res": state["res"], "index": idx, "cost": cost, "fc": fc}
    s.reset()
    if kind == "setup":
        h = am.Handle.for_problem(state["pb"], state["dtype"])
        am.solve(h, state["p"], s.st[0], state["K"])
        torch.cuda.current_stream().synchronize()
        h.close()
        return s.all
    if kind == "plain":
        am.solve_plain(state["h"], state["p"], s.st[0], state["K"], state["ws"])
    else:
        am.solve(state["h"], state["p"], s.st[0], state["K"])
    return s.all


def _period_inputs(case, seed, ctl):
    """A period of the closed loop: people around a robot that moves at 1 m/s
    along the course, and the samples of that period."""
    s = _seeds(case, seed, 2)[1]
    rng = np.random.default_rng(s)
    crowd = mpc.crowd_scene(mpc.KINDS[int(rng.integers(3))], s)
    pb = ctl.problem(crowd, 0.0, crowd.start + rng.normal(0.0, 0.05, 2), np.array([1.0, 0.0]), np.zeros(2), 0.0, 0.0,
                     0.0)
    init = inputs.make_initial(pb, case["B"], s, 0.5 if case["B"] > 1 else 0.05)
    return inputs.as_stored(pb, _multipliers(init, s), "f32")


# ---------------------------------------------------------------- work

def _solve_work(B, m, n, q, nv, K, es):
    # per iteration: nine channels evaluated and nine contracted, one distance
    # test per (circle, obstacle, t), heading and disc projections, the
    # constant operators; bytes: the state in and out, the obstacle table
    per = 36.0 * nv * q + 12.0 * m * n * q + 80.0 * q + 2.0 * (2 * (2 * nv) ** 2 + nv * nv)
    state = (5 * nv + 5 * nv) * B
    return es * (2.0 * state + 3 * q * B + am.NRES * B + 2 * n * q), B * per * max(K, 1)


def work(case):
    es = 8 if case.get("dtype") == "f64" else 4
    q, nv, kind = case["q"], case["nv"], case["kind"]
    if kind in ("multi", "serve"):
        cnt = case.get("problems") or case["requests"]
        m, n = (4, 11) if kind == "multi" else (5, 17.5)
        b, f = _solve_work(0.5 * (case["lo"] + case["hi"]), m, n, q, nv, case["K"], es)
        return {"bytes": cnt * b, "flops": cnt * f}
    B, m, n = case["B"], case["m"], case["n"]
    b, f = _solve_work(B, m, n, q, nv, case.get("K", 0), es)
    if kind == "plain":   # alpha and d of every (circle, obstacle, t) of every iteration are part of this path
        b += 2.0 * es * B * m * n * q * (case["K"] + 1)
    if kind == "residuals":
        b, f = es * (B * (10 * nv + am.NRES) + 2 * n * q), B * (20.0 * nv * q + 12.0 * m * n * q + 60.0 * q)
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------- 64-bit values

def _basis(pb):
    """Bernstein basis of degree nv-1 and its time derivatives on the grid."""
    q, nv, tf = int(pb["q"]), int(pb["nv"]), float(pb["tf"])
    tau = np.arange(q) / (q - 1.0)

    def bern(d):
        return np.stack([math.comb(d, i) * tau ** i * (1.0 - tau) ** (d - i) for i in range(d + 1)], 1)

    N = nv - 1
    pad = lambda b, l, r: np.pad(b, ((0, 0), (l, r)))  # noqa: E731
    b1, b2 = bern(N - 1), bern(N - 2)
    Pd = N * (pad(b1, 1, 0) - pad(b1, 0, 1)) / tf
    Pdd = N * (N - 1) * (pad(b2, 2, 0) - 2.0 * pad(b2, 1, 1) + pad(b2, 0, 2)) / tf ** 2
    return bern(N), Pd, Pdd


class _Exact:
    """The method's iteration in FP64, in an orthonormal basis of the
    polynomial space (P = U R), written from its equations."""

    def __init__(self, pb):
        dev = "cuda" if torch.cuda.is_available() else "cpu"
        t = lambda v: torch.as_tensor(np.ascontiguousarray(v), dtype=torch.float64, device=dev)  # noqa: E731
        self.t, self.pb = t, pb
        P, Pd, Pdd = _basis(pb)
        U, R = np.linalg.qr(P)
        Ri = np.linalg.inv(R)
        V, W = Pd @ Ri, Pdd @ Ri
        nv, rho = int(pb["nv"]), float(pb["rho"])
        r = np.asarray(pb["r"], float)
        m, n = len(r), len(pb["oa"])
        self.flags = int(pb.get("flags", 0))
        GW = W.T @ W
        I = np.eye(nv)  # noqa: E741
        FtF = np.block([[V.T @ V + GW + m * n * I, n * r.sum() * I], [n * r.sum() * I, (n * (r * r).sum() + 1.0) * I]])
        Q = np.zeros((2 * nv, 2 * nv))
        Q[:nv, :nv] = GW
        if not self.flags & am.Q_CS_ZERO:
            Q[nv:, nv:] = GW
        A = np.stack([U[0], V[0], W[0], U[-1], V[-1], W[-1]])

        def kkt(H, A):
            k = np.block([[H, A.T], [A, np.zeros((6, 6))]])
            inv = np.linalg.inv(k)[:H.shape[0]]
            return t(inv[:, :H.shape[0]]), t(inv[:, H.shape[0]:])

        self.M1, self.H1 = kkt(Q + rho * FtF, np.hstack([A, np.zeros((6, nv))]))
        self.M2, self.H2 = kkt(GW + rho * I, A)
        self.U, self.V, self.W, self.R, self.Ri, self.A = (t(v) for v in (U, V, W, R, Ri, A))
        self.r, self.nv, self.m, self.n = t(r), nv, m, n
        self.ox, self.oy = t(np.reshape(pb["ox"], (n, -1))), t(np.reshape(pb["oy"], (n, -1)))
        self.a = (t(pb["oa"]) + pb["rc"]).view(1, 1, n, 1)
        self.b = (t(pb["ob"]) + pb["rc"]).view(1, 1, n, 1)
        self.bx, self.by, self.bpsi = t(pb["bx"]), t(pb["by"]), t(pb["bpsi"])

    @staticmethod
    def _atan2z(y, x):
        return torch.where((x == 0) & (y == 0), torch.zeros_like(x), torch.atan2(y, x))

    def load(self, init):
        self.z = {k: self.t(init[k]) @ self.R.T for k in COEF}
        lam = self.t(init["lam"]).view(-1, 4, self.nv) @ self.Ri
        self.lam = lam.reshape(lam.shape[0], -1)
        self.lpsi = self.t(init["lam_psi"]) @ self.Ri

    def values(self):
        z, U, V, W = self.z, self.U.T, self.V.T, self.W.T
        return dict(x=z["cx"] @ U, xd=z["cx"] @ V, xdd=z["cx"] @ W, y=z["cy"] @ U, yd=z["cy"] @ V, ydd=z["cy"] @ W,
                    c=z["cc"] @ U, s=z["cs"] @ U, psi=z["cpsi"] @ U, psid=z["cpsi"] @ V, psidd=z["cpsi"] @ W)

    def offsets(self, v, ux, uy):
        r = self.r.view(1, self.m, 1)
        px = (v["x"][:, None] + r * ux[:, None])[:, :, None] - self.ox
        py = (v["y"][:, None] + r * uy[:, None])[:, :, None] - self.oy
        return px, py

    def targets(self, v):
        """Points (a d cos alpha, b d sin alpha) relative to each obstacle
        centre, and the disc targets of velocity and acceleration."""
        slack = self.flags & am.XTILDE_SLACK
        ux, uy = (v["c"], v["s"]) if slack else (torch.cos(v["psi"]), torch.sin(v["psi"]))
        xt, yt = self.offsets(v, ux, uy)
        a, b = self.a, self.b
        if self.flags & am.ALPHA_LITERAL:
            al = self._atan2z(yt, xt)
            ca, sa = torch.cos(al), torch.sin(al)
            d = ((a * xt * ca + b * yt * sa) / (a * a * ca * ca + b * b * sa * sa)).clamp(min=1.0)
            gx, gy = a * d * ca, b * d * sa
        else:
            k = torch.sqrt((xt / a) ** 2 + (yt / b) ** 2)
            f = torch.where(k == 0, torch.zeros_like(k), (1.0 / k).clamp(min=1.0))
            gx, gy = torch.where(k == 0, a.expand_as(k), xt * f), yt * f
        lim = []
        for p, q, top in ((v["xd"], v["yd"], self.pb["vmax"]), (v["xdd"], v["ydd"], self.pb["amax"])):
            h = torch.hypot(p, q)
            f = torch.where(h > top, top / h, torch.ones_like(h))
            lim += [p * f, q * f]
        return gx, gy, lim

    def parts(self, v, g):
        """F^T g of both axes as [B, 4 nv]."""
        gx, gy, lim = g
        out = []
        r = self.r.view(1, self.m, 1, 1)
        for axis, (gg, o, tr) in enumerate(((gx, self.ox, torch.cos(v["psi"])), (gy, self.oy, torch.sin(v["psi"])))):
            tot = gg + o
            pos = lim[axis] @ self.V + lim[2 + axis] @ self.W + tot.sum((1, 2)) @ self.U
            out += [pos, ((r * tot).sum((1, 2)) + tr) @ self.U]
        return torch.cat(out, 1)

    def f_of(self, v):
        """F^T F xi of both axes as [B, 4 nv]."""
        out, sr, mn = [], self.n * self.r.sum(), self.m * self.n
        sr2 = self.n * (self.r * self.r).sum()
        for p, pd, pdd, s in (("x", "xd", "xdd", "c"), ("y", "yd", "ydd", "s")):
            out += [v[pd] @ self.V + v[pdd] @ self.W + (mn * v[p] + sr * v[s]) @ self.U,
                    (sr * v[p] + (sr2 + 1.0) * v[s]) @ self.U]
        return torch.cat(out, 1)

    def solve(self, K):
        nv, rho, z = self.nv, float(self.pb["rho"]), self.z
        v = self.values()
        ftg = self.parts(v, self.targets(v))
        for _ in range(K):
            rhs = (self.lam + rho * ftg).view(-1, 2, 2 * nv)
            xi = rhs @ self.M1.T
            xi[:, 0] += self.H1 @ self.bx
            xi[:, 1] += self.H1 @ self.by
            z["cx"], z["cc"], z["cy"], z["cs"] = xi[:, 0, :nv], xi[:, 0, nv:], xi[:, 1, :nv], xi[:, 1, nv:]
            v = self.values()
            c, s, psi = v["c"], v["s"], v["psi"]
            if self.flags & am.PSI_NO_UNWRAP:
                ph = self._atan2z(s, c)
            else:
                cp, sp = torch.cos(psi), torch.sin(psi)
                ph = psi + self._atan2z(s * cp - c * sp, c * cp + s * sp)
            z["cpsi"] = (self.lpsi + rho * (ph @ self.U)) @ self.M2.T + self.H2 @ self.bpsi
            v = self.values()
            ftg = self.parts(v, self.targets(v))
            self.lam = self.lam - rho * (self.f_of(v) - ftg)
            self.lpsi = self.lpsi - float(self.pb.get("rho_psi", rho)) * ((v["psi"] - ph) @ self.U)

    def residuals(self):
        v = self.values()
        gx, gy, lim = self.targets(v)
        cp, sp = torch.cos(v["psi"]), torch.sin(v["psi"])
        px, py = self.offsets(v, cp, sp)
        B = px.shape[0]
        f2 = ((px - gx) ** 2 + (py - gy) ** 2).reshape(B, -1)
        lev = torch.sqrt((px / self.a) ** 2 + (py / self.b) ** 2).reshape(B, -1)
        o = torch.zeros((B, am.NRES), dtype=torch.float64, device=px.device)
        o[:, 0], o[:, 1] = f2.max(1).values.sqrt(), f2.mean(1).sqrt()
        o[:, 2] = torch.hypot(v["xd"] - lim[0], v["yd"] - lim[1]).max(1).values
        o[:, 3] = torch.hypot(v["xdd"] - lim[2], v["ydd"] - lim[3]).max(1).values
        o[:, 4] = torch.maximum((v["c"] - cp).abs(), (v["s"] - sp).abs()).max(1).values
        dh = self._atan2z(v["s"], v["c"]) - v["psi"]
        o[:, 5] = (dh - 2 * math.pi * torch.floor((dh + math.pi) / (2 * math.pi))).abs().max(1).values
        o[:, 6] = torch.stack([(self.z[k] @ self.A.T - b).abs().max(1).values
                               for k, b in (("cx", self.bx), ("cy", self.by), ("cpsi", self.bpsi))]).max(0).values
        o[:, 7] = (v["xdd"] ** 2 + v["ydd"] ** 2 + v["psidd"] ** 2).sum(1)
        o[:, 8] = lev.min(1).values - 1.0
        o[:, 9] = torch.hypot(v["xd"], v["yd"]).max(1).values - self.pb["vmax"]
        o[:, 10] = torch.hypot(v["xdd"], v["ydd"]).max(1).values - self.pb["amax"]
        return o

    def out(self, res=True):
        v = self.values()
        d = {k: self.z[k] @ self.Ri.T for k in COEF}
        d["lam"] = (self.lam.view(-1, 4, self.nv) @ self.R).reshape(self.lam.shape)
        d["lam_psi"] = self.lpsi @ self.R
        d["traj"] = torch.stack([v["x"], v["y"], v["psi"]], 1)
        if res:
            d["res"] = self.residuals()
        return {k: x.reshape(-1) for k, x in d.items()}


def _best(res, tol):
    r = res.cpu().numpy()
    ok = r[:, 0] <= tol
    i = int(np.argmin(np.where(ok, r[:, 7], np.inf))) if ok.any() else int(np.argmin(r[:, 0]))
    return i, float(r[i, 7]), float(r[i, 0])


def exact(case, seed):
    kind = case["kind"]
    if kind in ("multi", "serve"):
        outs = []
        for pb, init in _uneven(case, seed, case.get("problems") or case["requests"]):
            e = _Exact(pb)
            e.load(init)
            e.solve(case["K"])
            outs.append(e.out())
        if kind == "serve":
            return [o["traj"] for o in outs]
        return {k: torch.cat([o[k] for o in outs]) for k in outs[0]}
    if kind == "period":
        ctl = mpc.MPC(case["B"], iters=case["K"], horizon=case["tf"], q=case["q"], nv=case["nv"], circles=case["m"],
                      n_obs=case["n"], seed=0)
        pb, init = _period_inputs(case, seed, ctl)
        e = _Exact(pb)
        e.load(init)
        e.solve(case["K"])
        o = e.out()
        i, _, fc = _best(o["res"].view(-1, am.NRES), ctl.fc_tol)
        return {"index": None, "fc": fc, "coef": {k: o[k].view(case["B"], -1)[i] for k in COEF}, "res": o["res"]}
    pb, init = _problem(case, seed, case["m"], case["n"], case["B"], case.get("moving", True), case.get("flags", 0))
    e = _Exact(pb)
    if kind == "residuals":
        _, init = inputs.as_stored(pb, _heading_samples(pb, init, _seeds(case, seed, 3)[2]), case["dtype"])
        e.load(init)
        r = e.residuals()
        i, cost, fc = _best(r, FC_TOL)
        return {"res": r, "index": None, "cost": cost, "fc": fc}
    e.load(init)
    e.solve(case["K"])
    return e.out(res=kind != "plain")
