"""Work a user of the batched trajectory-optimisation library has it do.

Every case goes through the public entry points (`Batch.step`, `serve_step` and
`plant_step` inside the closed-loop and hypothesis drivers, `ServeContext`) on
seeded problems of `workload`. A case is a dict of plain values:

  kind "step"    one call over a uniform batch: M solves of n DoF and N knots,
                 `iters` SQP iterations from the resting initial guess;
       "task"    the same with the tip tracking (figure-8) cost;
       "uneven"  a batch whose DoF and horizons differ per solve, replayed as a
                 graph (task: with the tip tracking cost);
       "serve"   `reqs` re-solve requests through a launch context, waited for;
       "loop"    `ticks` closed-loop control ticks over all M instances;
       "forces"  `ticks` hypothesise-and-test ticks, P instances x H forces;
       "plant"   one control period of the RK4 plant for M instances.

A pass starts from the same iterate every time (the trajectories are restored
and the multipliers cleared, as a program does that is handed new problems),
except for "serve", whose instances go on from their last plan. A pass runs the
first SQP iterations (one to three in all) and not those of a solve to
convergence: later the best candidates of the line search tie below the FP32
resolution of the merit, so which one is taken, and with it the rest of the
iterate, hangs on rounding. Each SQP iteration is the same work.
"""
from __future__ import annotations

import numpy as np
import torch

import paper_2510_07625_amd as g
import workload as w
from paper_2510_07625_amd import closed_loop, hypotheses

TOL = 1e-5            # PCG tolerance: the solver's default
TASK_CAP = 1000       # PCG cap with tip tracking (these systems take more than N nx iterations)
MU, BETA, N_ALPHA = 10.0, 2.0, 8   # the solver's defaults


def listed():
    return [
        # One MPC instance out of a served pool asks for its next control: pure latency.
        dict(name="request 7x32", kind="serve", n=7, N=32, M=256, reqs=1, iters=1),
        # A single robot's real-time iteration on the shortest horizon.
        dict(name="rti 6x8 M1", kind="step", n=6, N=8, M=1, iters=1),
        # 512 knots in one real-time iteration, the size quoted for a 10 kHz loop.
        dict(name="rti 6x16 M32", kind="step", n=6, N=16, M=32, iters=1),
        # Many short horizons at once: more solves than compute units.
        dict(name="rti 6x8 M512", kind="step", n=6, N=8, M=512, iters=1),
        # The benchmark's batch: one solve per compute unit.
        dict(name="solve 7x32 M256", kind="step", n=7, N=32, M=256, iters=2),
        # A long, ragged horizon, fewer solves than compute units.
        dict(name="rti 7x100 M50", kind="step", n=7, N=100, M=50, iters=1),
        # The longest horizon, more solves than compute units: the largest call.
        dict(name="rti 6x128 M512", kind="step", n=6, N=128, M=512, iters=1),
        # Tip tracking (figure-8), a real-time iteration.
        dict(name="tip 7x32 M256", kind="task", n=7, N=32, M=256, iters=1),
        # A batch of mixed robots and horizons as one graph replay.
        dict(name="uneven M128", kind="uneven", M=128, iters=2, task=False),
        # Closed-loop MPC: serving step and plant, a real-time iteration per tick.
        dict(name="mpc 7x64 M256", kind="loop", n=7, N=64, M=256, iters=1, ticks=3),
        # Force estimation: 32 instances with 32 hypotheses each.
        dict(name="forces 32x32", kind="forces", n=7, N=32, P=32, H=32, iters=1, ticks=2),
        # The plant of a simulation study on its own.
        dict(name="plant 7 M256", kind="plant", n=7, M=256, substeps=10),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(float(np.exp(rng.uniform(np.log(lo), np.log(hi))))))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "task", "uneven", "serve", "loop", "forces", "plant"])
    n = rng.choice([3, 6, 7])
    N, M, iters = _log_int(rng, 2, 128), _log_int(rng, 1, 512), rng.randint(1, 2)
    # The cost of a call grows with N^2 M iters (the PCG iterations grow with N).
    most = lambda per: max(1, min(M, int(0.7 * 128 * 128 * 512 / (N * N * per))))
    if kind == "step":
        return dict(kind=kind, n=n, N=N, M=most(iters), iters=iters)
    if kind == "task":
        N = min(N, 100)
        return dict(kind=kind, n=n, N=N, M=min(256, most(4)), iters=1)
    if kind == "uneven":
        task = rng.random() < 0.3
        return dict(kind=kind, M=rng.randint(16, 128), iters=1 if task else iters, task=task)
    if kind == "serve":
        pool = max(2, min(256, M))
        return dict(kind=kind, n=n, N=min(N, 64), M=pool, reqs=_log_int(rng, 1, min(32, pool)), iters=1)
    if kind == "loop":
        ticks = rng.randint(1, 2)
        return dict(kind=kind, n=n, N=min(N, 64), M=most(2 * ticks), iters=1, ticks=ticks)
    if kind == "forces":
        return dict(kind=kind, n=rng.choice([6, 7]), N=min(max(N, 8), 32), P=rng.randint(1, 32), H=rng.randint(2, 32),
                    iters=1, ticks=rng.randint(1, 2))
    return dict(kind=kind, n=n, M=_log_int(rng, 1, 1024), substeps=rng.randint(1, 20))


# ---- The problems of a case ---------------------------------------------------
def _solves(case, seed):
    k = case["kind"]
    if k == "uneven":
        return (w.figure8_uneven_batch if case["task"] else w.uneven_batch)(seed, M=case["M"])
    if k == "task":
        return w.figure8_batch(seed, case["M"], n=case["n"], N=case["N"])
    if k == "forces":
        one = [w.chain_solve(seed, p, n=case["n"], N=case["N"]) for p in range(case["P"])]
        return [s for s in one for _ in range(case["H"])]
    return w.chain_batch(seed, case["M"], n=case["n"], N=case.get("N", 8))


def _tracks(case):
    return case["kind"] == "task" or bool(case.get("task"))


def _true_force(case, seed):
    return np.random.default_rng([seed, 5]).normal(0.0, 20.0, (case["P"], 3))


def _torques(case, seed):
    return np.random.default_rng([seed, 6]).normal(0.0, 5.0, (case["M"], case["n"])).astype(np.float32)


def prepare(case, seed):
    k = case["kind"]
    solves = _solves(case, seed)
    params = g.Params(sqp_iters=case.get("iters", 1), pcg_tol=TOL, pcg_max_iter=TASK_CAP if _tracks(case) else 0)
    b = g.Batch.from_solves(solves, params)
    xs, goal, X0, U0 = g.pack_inputs(solves)
    s = dict(case=case, batch=b, xs=xs, goal=goal, X0=X0, U0=U0)
    if k in ("step", "task", "uneven"):
        s["X"], s["U"] = X0.clone(), U0.clone()
    elif k == "serve":
        b.set_trajectories(X0, U0)
        s["ctx"] = g.ServeContext(b, capacity=case["reqs"], n_iters=case["iters"])
        s["h_xs"], s["h_goal"] = xs.cpu().numpy(), goal.cpu().numpy()
        torch.cuda.synchronize()
    elif k == "forces":
        s["x0"], s["g0"] = xs[::case["H"]].contiguous(), goal[::case["H"]].contiguous()
        s["force"] = _true_force(case, seed)
    elif k == "plant":
        s["tau"] = torch.from_numpy(_torques(case, seed)).cuda()
        s["xn"] = torch.empty_like(xs)
    return s


def run(s):
    case, b = s["case"], s["batch"]
    k = case["kind"]
    if k in ("step", "task", "uneven"):
        s["X"].copy_(s["X0"])
        s["U"].copy_(s["U0"])
        b.reset_warm_start()
        b.step(s["xs"], s["goal"], s["X"], s["U"], case["iters"], graph=k == "uneven")
        return {"X": s["X"], "U": s["U"]}
    if k == "serve":
        c, R = s["ctx"], case["reqs"]
        c.slots[:R] = np.arange(R)
        c.xs[:R] = s["h_xs"][:R]
        c.goal[:R] = s["h_goal"][:R]
        c.submit(R, shift=1)
        while not c.done():
            pass
        return {"x1": c.x1[:R].copy(), "u0": c.u0[:R].copy()}
    if k == "plant":
        return {"xn": b.plant_step(s["xs"], s["tau"], h=0.01, substeps=case["substeps"], xn=s["xn"])}
    b.set_trajectories(s["X0"], s["U0"])
    b.reset_warm_start()
    if k == "loop":
        r = closed_loop.run(b, s["xs"], s["goal"], case["ticks"], n_iters=case["iters"], timing=False)
        return {"states": r.states, "controls": r.controls, "plans": b.get_trajectories()}
    r = hypotheses.run(b, case["P"], case["H"], s["x0"], s["g0"], case["ticks"], lambda t: s["force"], sigma=12.0,
                       n_iters=case["iters"])
    return {"states": r.states, "controls": r.controls, "estimates": r.estimates.astype(np.float32),
            "plans": b.get_trajectories()}


# ---- What a pass cannot do without ----------------------------------------------
def _shapes(case):
    """(n, N, solves, SQP iterations, tracking) of every uniform share of the case's SQP work."""
    k = case["kind"]
    if k == "uneven":
        return [(n, N, case["M"] / 12, case["iters"], case["task"]) for n in (3, 6, 7) for N in (16, 32, 64, 128)]
    M = case["P"] * case["H"] if k == "forces" else case["reqs"] if k == "serve" else case["M"]
    return [] if k == "plant" else [(case["n"], case["N"], M, case["iters"] * case.get("ticks", 1), _tracks(case))]


def work(case):
    """Bytes: start states, goals and trajectories in, trajectories and multipliers out. FLOPs: the method's own
    count of an SQP iteration (dynamics and derivatives, Schur complement, PCG, step, line search). The seeded chains take
    about 3 N PCG iterations per SQP iteration, and 7 N with tip tracking."""
    by = fl = 0.0
    for n, N, M, iters, tip in _shapes(case):
        nx = 2 * n
        fd, col = 260.0 * n, 360.0 * n
        pcg = (7 if tip else 3) * N * (4 * (3 * N - 2) * nx * nx + 10 * N * nx)
        fl += M * iters * (N * ((1 + N_ALPHA) * fd + nx * col + 7 * nx ** 3 + 2 * nx * nx * n + 3 * nx * nx) + pcg)
        by += M * (4 * (nx + n) + 2 * 4 * (N * nx + (N - 1) * n) + 2 * 8 * N * nx)
    if case["kind"] in ("plant", "loop", "forces"):
        n, sub = case["n"], case.get("substeps", 10)
        M = case["P"] * (case["H"] + 1) if case["kind"] == "forces" else case["M"]
        M *= case.get("ticks", 1)
        fl += M * sub * 4 * 260.0 * n
        by += M * 4 * (5 * n + 5 * n)
    return {"bytes": by, "flops": fl}


# ---- The same results in 64 bits, in plain torch ---------------------------------
# Vectors of a link frame are triples of tensors; joint i turns about z (even i)
# or y (odd i) and sits at the length of link i - 1 along z of link i - 1.
def _cross(a, b):
    return (a[1] * b[2] - a[2] * b[1], a[2] * b[0] - a[0] * b[2], a[0] * b[1] - a[1] * b[0])


def _add(*v):
    return tuple(sum(x) for x in zip(*v))


def _scale(s, a):
    return tuple(s * x for x in a)


def _turn(i, c, s, v, down):
    """Joint i's rotation of v: to the child frame (down) or to the parent frame."""
    s = -s if down else s
    if i % 2:
        return (c * v[0] + s * v[2], v[1], c * v[2] - s * v[0])
    return (c * v[0] - s * v[1], s * v[0] + c * v[1], v[2])


class _Robots:
    """Chains of one DoF, their parameters broadcast over [M, ...]."""

    def __init__(self, solves, dev, dims):
        t = lambda a: torch.tensor(np.asarray(a, np.float64), device=dev)
        self.n = solves[0].n
        links = t([s.links for s in solves])                                   # [M, n, 5]
        self.link = [[links[:, i, j].reshape((-1,) + (1,) * dims) for j in range(5)] for i in range(self.n)]
        self.g = t([s.gravity for s in solves]).reshape((-1,) + (1,) * dims)
        self.fext = None

    def inverse(self, q, qd, qdd, gravity=True):
        """Newton-Euler recursion; q, qd, qdd: lists of n tensors."""
        n, z = self.n, torch.zeros_like(q[0] + qd[0] + qdd[0] + self.g)
        om, dom, acc = (z, z, z), (z, z, z), (z, z, z + (self.g if gravity else 0.0))
        f, m, rot = [], [], []
        ext = None if self.fext is None or not gravity else tuple(z + x for x in self.fext)
        for i in range(n):
            L, mass, ix, iy, iz = self.link[i]
            r = (0.0, 0.0, self.link[i - 1][0]) if i else (0.0, 0.0, 0.0)
            acc = _add(acc, _cross(dom, r), _cross(om, _cross(om, r)))
            c, s = torch.cos(q[i]), torch.sin(q[i])
            rot.append((c, s))
            om, dom, acc = (_turn(i, c, s, v, True) for v in (om, dom, acc))
            if ext is not None:
                ext = _turn(i, c, s, ext, True)
            e = (0.0, 1.0, 0.0) if i % 2 else (0.0, 0.0, 1.0)
            dom = _add(dom, _scale(qdd[i], e), _cross(om, _scale(qd[i], e)))
            om = _add(om, _scale(qd[i], e))
            com = (0.0, 0.0, 0.5 * L)
            fi = _scale(mass, _add(acc, _cross(dom, com), _cross(om, _cross(om, com))))
            iw, idw = ((ix * v[0], iy * v[1], iz * v[2]) for v in (om, dom))
            f.append(fi)
            m.append(_add(idw, _cross(om, iw), _cross(com, fi)))
        tau, F, T = [None] * n, (z, z, z), (z, z, z)
        if ext is not None:
            F = _scale(-1.0, ext)
            T = _cross((0.0, 0.0, self.link[n - 1][0]), F)
        for i in reversed(range(n)):
            F, T = _add(F, f[i]), _add(T, m[i])
            tau[i] = T[1] if i % 2 else T[2]
            c, s = rot[i]
            F, T = _turn(i, c, s, F, False), _turn(i, c, s, T, False)
            if i:
                T = _add(T, _cross((0.0, 0.0, self.link[i - 1][0]), F))
        return torch.stack(torch.broadcast_tensors(*tau), -1)

    def mass(self, q):
        z = torch.zeros_like(q[0])
        cols = [self.inverse(q, [z] * self.n, [z + float(i == j) for i in range(self.n)], gravity=False)
                for j in range(self.n)]
        return torch.stack(cols, -1)

    def forward(self, q, qd, tau):
        """Accelerations [..., n] for q, qd, tau [..., n]."""
        ql, qdl = list(q.unbind(-1)), list(qd.unbind(-1))
        b = self.inverse(ql, qdl, [torch.zeros_like(ql[0])] * self.n)
        return torch.linalg.solve(self.mass(ql), (tau - b).unsqueeze(-1)).squeeze(-1)

    def tip(self, q):
        """Tip position in the base frame, [..., 3]."""
        z = torch.zeros_like(q[0])
        p = (z, z, z + self.link[self.n - 1][0])
        for i in reversed(range(self.n)):
            c, s = torch.cos(q[i]), torch.sin(q[i])
            p = _turn(i, c, s, p, False)
            if i:
                p = (p[0], p[1], p[2] + self.link[i - 1][0])
        return torch.stack(torch.broadcast_tensors(*p), -1)


def _mv(A, x):
    return (A * x.unsqueeze(-2)).sum(-1)


def _tv(A, x):
    return (A * x.unsqueeze(-1)).sum(-2)


def _columns(f, n, parts):
    """Derivatives of f with respect to every entry of the lists in `parts`, by complex steps."""
    eps, out = 1e-30, []
    for a in range(len(parts)):
        for j in range(n):
            arg = [[x.to(torch.complex128) + (1j * eps if (a, j) == (b, i) else 0.0) for i, x in enumerate(p)]
                   for b, p in enumerate(parts)]
            out.append(f(*arg).imag / eps)
    return torch.stack(out, -1)


class _Sqp:
    """The batched SQP of solves of one shape: Schur complement, stair-preconditioned CG stopped by its own rule."""

    def __init__(self, solves, cap, dev):
        t = lambda a: torch.tensor(np.asarray(a, np.float64), device=dev)
        s0 = solves[0]
        self.n, self.N, self.h, self.cap, self.M = s0.n, s0.N, s0.dt, cap, len(solves)
        self.rob, self.rob_a = _Robots(solves, dev, 1), _Robots(solves, dev, 2)
        Q, QN = t([s.Qd for s in solves]), t([s.QNd for s in solves])
        self.Q = Q[:, None, :].repeat(1, self.N, 1)
        self.Q[:, -1] = QN
        self.R = t([s.Rd for s in solves])[:, None, :]
        self.tip = s0.Wee is not None
        if self.tip:
            self.W = t([s.Wee for s in solves])[:, None, :].repeat(1, self.N, 1)
            self.W[:, -1] = t([s.WeeN for s in solves])
            self.pref = t([s.pref for s in solves])

    def forces(self, fext):
        """External tip forces [M, 3] in the dynamics."""
        for r, d in ((self.rob, 1), (self.rob_a, 2)):
            r.fext = tuple(fext[:, c].reshape((-1,) + (1,) * d) for c in range(3))

    def merit(self, rob, xs, xg, X, U):
        """Merit of trajectories [M, (candidates,) N, nx]."""
        n, ex = self.n, X.dim() - 3
        up = lambda a: a.reshape(a.shape[:1] + (1,) * ex + a.shape[1:])
        q, qd = X[..., :-1, :n], X[..., :-1, n:]
        acc = rob.forward(q, qd, U)
        c = torch.cat([q + self.h * qd, qd + self.h * acc], -1) - X[..., 1:, :]
        J = 0.5 * (up(self.Q) * (X - up(xg[:, None])) ** 2).sum((-1, -2)) + 0.5 * (up(self.R) * U ** 2).sum((-1, -2))
        if self.tip:
            p = rob.tip(list(X[..., :n].unbind(-1)))
            J = J + 0.5 * (up(self.W) * (p - up(self.pref)) ** 2).sum((-1, -2))
        return J + MU * (c.abs().sum((-1, -2)) + (X[..., 0, :] - up(xs)).abs().sum(-1))

    def iterate(self, xs, xg, X, U, lam):
        """One SQP iteration; X [M, N, nx], U [M, N-1, n], lam [M, N, nx]."""
        n, N, h, M = self.n, self.N, self.h, self.M
        nx, dev = 2 * n, X.device
        q, qd = X[:, :-1, :n], X[:, :-1, n:]
        ql, qdl = list(q.unbind(-1)), list(qd.unbind(-1))
        acc = self.rob.forward(q, qd, U)
        accl = list(acc.unbind(-1))
        Mi = torch.linalg.inv(self.rob.mass(ql))
        dtau = _columns(lambda a, b: self.rob.inverse(a, b, accl), n, [ql, qdl])        # [M, N-1, n, 2n]
        eye = torch.eye(n, dtype=torch.float64, device=dev)
        A = torch.zeros(M, N - 1, nx, nx, dtype=torch.float64, device=dev)
        A[..., :n, :n], A[..., :n, n:] = eye, h * eye
        A[..., n:, :] = -h * (Mi.unsqueeze(-1) * dtau.unsqueeze(-3)).sum(-2)
        A[..., n:, n:] += eye
        B = torch.zeros(M, N - 1, nx, n, dtype=torch.float64, device=dev)
        B[..., n:, :] = h * Mi
        e = torch.cat([q + h * qd, qd + h * acc], -1) - X[:, 1:]
        c0 = xs - X[:, 0]
        gx, gu = self.Q * (X - xg[:, None]), self.R * U
        H = torch.diag_embed(self.Q)
        if self.tip:
            xl = list(X[..., :n].unbind(-1))
            Jt = _columns(self.rob.tip, n, [xl])                                          # [M, N, 3, n]
            r = self.rob.tip(xl) - self.pref
            gx[..., :n] += _tv(Jt, self.W * r)
            H[..., :n, :n] += (Jt.unsqueeze(-1) * (self.W.unsqueeze(-1) * Jt).unsqueeze(-2)).sum(-3)
        Hi = torch.linalg.inv(H)
        AH = (A.unsqueeze(-1) * Hi[:, :-1].unsqueeze(-3)).sum(-2)                          # A_k Q_k^-1
        D = Hi.clone()
        D[:, 1:] += (AH.unsqueeze(-2) * A.unsqueeze(-3)).sum(-1)
        BR = B / self.R.unsqueeze(-2)
        D[:, 1:] += (BR.unsqueeze(-2) * B.unsqueeze(-3)).sum(-1)
        gam = _mv(Hi, gx)
        gam[:, 0] += c0
        gam[:, 1:] += e - _mv(AH, gx[:, :-1]) - _mv(BR, gu)
        Di = torch.linalg.inv(D)
        del D

        def off(v):                                                                       # off-diagonal blocks of S~
            o = torch.zeros_like(v)
            o[:, 1:] -= _mv(AH, v[:, :-1])
            o[:, :-1] -= _tv(AH, v[:, 1:])
            return o

        Dg = Hi.clone()
        Dg[:, 1:] += (AH.unsqueeze(-2) * A.unsqueeze(-3)).sum(-1) + (BR.unsqueeze(-2) * B.unsqueeze(-3)).sum(-1)
        S = lambda v: _mv(Dg, v) + off(v)

        def P(v):
            zv = _mv(Di, v)
            return zv - _mv(Di, off(zv))

        dot = lambda a, b: (a * b).sum((1, 2))
        stop = TOL * TOL * dot(gam, P(gam))
        r = gam - S(lam)
        u = P(r)
        eta, p = dot(r, u), u.clone()
        for _ in range(self.cap or N * nx):
            on = eta > stop
            if not bool(on.any()):
                break
            sp = S(p)
            al = torch.where(on, eta / dot(p, sp), 0.0)[:, None, None]
            lam, r = lam + al * p, r - al * sp
            u = P(r)
            new = torch.where(on, dot(r, u), eta)
            p = torch.where(on[:, None, None], u + (new / eta)[:, None, None] * p, p)
            eta = new
        gx, gu = gx - lam, gu.clone()
        gx[:, :-1] += _tv(A, lam[:, 1:])
        gu += _tv(B, lam[:, 1:])
        dX, dU = -_mv(Hi, gx), -gu / self.R
        al = torch.tensor([BETA ** -i for i in range(N_ALPHA)], dtype=torch.float64, device=dev)[None, :, None, None]
        Xa, Ua = X[:, None] + al * dX[:, None], U[:, None] + al * dU[:, None]
        m = self.merit(self.rob_a, xs, xg, Xa, Ua)
        best = torch.argmin(m, 1)
        pick = torch.arange(M, device=dev)
        return Xa[pick, best], Ua[pick, best], lam

    def shifted(self, *v):
        return [torch.cat([a[:, 1:], a[:, -1:]], 1) for a in v]


def _rk4(rob, x, tau, h, substeps):
    n, d = rob.n, h / substeps
    f = lambda y: torch.cat([y[..., n:], rob.forward(y[..., :n], y[..., n:], tau)], -1)
    for _ in range(substeps):
        k1 = f(x)
        k2 = f(x + 0.5 * d * k1)
        k3 = f(x + 0.5 * d * k2)
        x = x + d / 6.0 * (k1 + 2.0 * k2 + 2.0 * k3 + f(x + d * k3))
    return x


def exact(case, seed):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    solves, k = _solves(case, seed), case["kind"]
    t = lambda a: torch.tensor(np.asarray(a, np.float32), device=dev).double()     # inputs as the call gets them
    start = lambda ss: (t([s.xs for s in ss]), t([np.r_[s.qgoal, np.zeros(s.n)] for s in ss]),
                        t([s.X0 for s in ss]), t([s.U0 for s in ss]))
    if k == "plant":
        xs = start(solves)[0]
        return {"xn": _rk4(_Robots(solves, dev, 0), xs, t(_torques(case, seed)), 0.01, case["substeps"])}
    cap = TASK_CAP if _tracks(case) else 0
    if k in ("step", "task", "uneven"):
        n_max, N_max = max(s.n for s in solves), max(s.N for s in solves)
        X = torch.zeros(len(solves), N_max, 2 * n_max, dtype=torch.float64)
        U = torch.zeros(len(solves), N_max - 1, n_max, dtype=torch.float64)
        for n, N in sorted({(s.n, s.N) for s in solves}):
            at = [i for i, s in enumerate(solves) if (s.n, s.N) == (n, N)]
            sub = [solves[i] for i in at]
            q = _Sqp(sub, cap, dev)
            xs, xg, x, u = start(sub)
            lam = torch.zeros_like(x)
            for _ in range(case["iters"]):
                x, u, lam = q.iterate(xs, xg, x, u, lam)
            for j, i in enumerate(at):
                X[i, :N, :2 * n], U[i, :N - 1, :n] = x[j].cpu(), u[j].cpu()
        return {"X": X, "U": U}
    if k == "serve":
        solves = solves[:case["reqs"]]
    q = _Sqp(solves, cap, dev)
    xs, xg, x, u = start(solves)
    lam = torch.zeros_like(x)
    if k == "serve":
        x, u, lam = q.shifted(x, u, lam)
        for _ in range(case["iters"]):
            x, u, lam = q.iterate(xs, xg, x, u, lam)
        return {"x1": x[:, 1], "u0": u[:, 0]}
    ticks, states, controls = case["ticks"], [], []
    if k == "loop":
        plant, now = _Robots(solves, dev, 0), xs
        states.append(now)
        for _ in range(ticks):
            x, u, lam = q.shifted(x, u, lam)
            for _ in range(case["iters"]):
                x, u, lam = q.iterate(now, xg, x, u, lam)
            controls.append(u[:, 0])
            now = _rk4(plant, now, u[:, 0], 0.01, 10)
            states.append(now)
        return {"states": torch.stack(states), "controls": torch.stack(controls), "plans": (x, u)}
    P, H = case["P"], case["H"]
    off = torch.tensor(hypotheses.offsets(H) * 12.0, device=dev)
    est, force = torch.zeros(P, 3, dtype=torch.float64, device=dev), t(_true_force(case, seed))
    first, every = _Robots(solves[::H], dev, 0), _Robots(solves, dev, 0)
    now = xs[::H]
    states.append(now)
    ests = [est]
    for _ in range(ticks):
        guess = (est[:, None] + off[None]).reshape(P * H, 3)
        q.forces(guess)
        now_h = now.repeat_interleave(H, 0)
        x, u, lam = q.shifted(x, u, lam)
        for _ in range(case["iters"]):
            x, u, lam = q.iterate(now_h, xg, x, u, lam)
        ctrl = u[::H, 0]
        first.fext, every.fext = tuple(force.unbind(-1)), tuple(guess.unbind(-1))
        pred = _rk4(every, now_h, ctrl.repeat_interleave(H, 0), 0.01, 10)
        now = _rk4(first, now, ctrl, 0.01, 10)
        d = (pred.reshape(P, H, -1) - now[:, None]).norm(dim=-1)
        est = est + off[torch.argmin(d, 1)]
        controls.append(ctrl)
        states.append(now)
        ests.append(est)
    return {"states": torch.stack(states), "controls": torch.stack(controls), "estimates": torch.stack(ests),
            "plans": (x, u)}
