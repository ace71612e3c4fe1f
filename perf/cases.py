"""Performance cases of the bundle-adjustment library: the work a program has
it do, through the Python binding of the C ABI, over the range of sizes, data
types and options it is used with.

Kinds of case (the "kind" field):

  solve   a whole Levenberg-Marquardt solve of one graph that the program has
          built (gba_prepare): reset, gba_solve, cameras and points read back
  step    one linearisation and damped step (gba_eval_step) of such a graph
  serve   local-BA requests submitted to a running server and collected
  vi      a whole visual-inertial solve (gba_vi_solve; host arrays in and out)
  preint  IMU preintegration of all intervals of a trajectory

Scenes are drawn by the package's seeded generators from the seed alone.  The
mixed-precision modes store steps and vectors in FP32, and programs that
choose them keep their maps in single precision: their results are taken as
float32 here (a step's entries are FP32 values already); FP64 results stay
float64.
"""
import math

import numpy as np
import torch

from paper_2509_26581_amd import gba, synth, synth_vi

_PREC = {"fp64": gba.GBA_FP64, "fp32": gba.GBA_MIXED_FP32, "bf16": gba.GBA_MIXED_BF16}
_GYRO_NOISE, _ACC_NOISE, _GYRO_WALK, _ACC_WALK = 1.7e-4, 2e-3, 2e-5, 3e-3


def listed():
    return [
        # a test-sized ring of cameras with squared loss: launches and host
        # round trips are all of it
        dict(name="solve_small_fp64", kind="solve", prec="fp64", n_cams=10, n_pts=500, track="u3-8",
             huber=False, solver="schur", trials=10, tol=1e-8),
        # a few hundred cameras: an object or a street block, odd sizes
        dict(name="solve_mid_fp32", kind="solve", prec="fp32", n_cams=203, n_pts=30011, track="g4",
             huber=True, solver="schur", trials=10, tol=1e-6),
        # the benchmark configuration: 1,000 cameras, ~1M observations
        dict(name="solve_1k_fp32", kind="solve", prec="fp32", n_cams=1000, n_pts=200000, track="g4",
             huber=True, solver="schur", trials=20, tol=1e-6),
        # the same system in plain FP64, one damped step
        dict(name="step_1k_fp64", kind="step", prec="fp64", n_cams=1000, n_pts=200000, track="g4",
             huber=True, solver="schur", lam=1e-4, tol=1e-8),
        # the whole damped system with recomputed Jacobians (minimum memory)
        dict(name="solve_full_fp64", kind="solve", prec="fp64", n_cams=120, n_pts=12007, track="g4",
             huber=True, solver="full-dynamic", trials=6, tol=1e-8),
        # more cameras than a workgroup's sums hold: the at-scale
        # configuration's shape at 0.4 of its size, BF16 Jacobian copy
        dict(name="step_4k_bf16", kind="step", prec="bf16", n_cams=4000, n_pts=400000, track="g7",
             huber=True, solver="schur", lam=1e-4, tol=1e-6),
        # one local-BA window at a time: the latency of a tracking thread
        dict(name="serve_one_fp32", kind="serve", prec="fp32", n_req=1, k_lo=18, k_hi=18, p_lo=3001,
             p_hi=3001, trials=10),
        # a burst of the benchmark's local-BA stream: throughput
        dict(name="serve_burst_fp32", kind="serve", prec="fp32", n_req=48, k_lo=5, k_hi=40, p_lo=500,
             p_hi=20000, trials=10),
        # a sliding visual-inertial window in FP64
        dict(name="vi_window_fp64", kind="vi", prec="fp64", n_kf=31, n_pts=2503, solver="schur",
             trials=5, tol=1e-8, max_pcg=200),
        # the paper's whole-system form on a medium trajectory
        dict(name="vi_full_fp64", kind="vi", prec="fp64", n_kf=300, n_pts=45001, solver="full",
             trials=4, tol=1e-6, max_pcg=100),
        # the benchmark's long trajectory: 2,000 keyframes, ~2.07M stereo
        # observations, FP32 storage of the products' array
        dict(name="vi_2k_fp32", kind="vi", prec="fp32", n_kf=2000, n_pts=300000, solver="schur",
             trials=5, tol=1e-6, max_pcg=100),
        # the IMU of that trajectory: 200 Hz, 0.25 s between keyframes
        dict(name="preint_2k", kind="preint", n=1999, rate=200),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "step", "serve", "serve", "vi", "vi", "preint"])
    if kind in ("solve", "step"):
        n_cams = _log_int(rng, 6, 1800 if kind == "step" else 1000)
        track = "u3-8" if n_cams < 16 else rng.choice(["u3-8", "g4", "g7"])
        mean = {"u3-8": 5.5, "g4": 5.0, "g7": 8.0}[track]
        n_pts = _log_int(rng, 30 * n_cams, min(200 * n_cams, 1.0e6 / mean))
        prec = rng.choice(["fp64", "fp32", "fp32", "bf16"] if kind == "step" else ["fp64", "fp32"])
        case = dict(kind=kind, prec=prec, n_cams=n_cams, n_pts=n_pts, track=track,
                    huber=rng.random() < 0.8, solver="schur", tol=1e-8 if prec == "fp64" else 1e-6)
        if kind == "solve":
            case["trials"] = rng.randint(8, 15)
            if n_cams <= 200 and prec == "fp64" and rng.random() < 0.4:
                case["solver"] = rng.choice(["full", "full-dynamic"])
                case["trials"] = 6
        else:
            case["lam"] = 10.0 ** rng.uniform(-5.0, -3.0)
        return case
    if kind == "serve":
        if rng.random() < 0.5:
            k, p = _log_int(rng, 5, 40), _log_int(rng, 500, 20000)
            return dict(kind="serve", prec="fp32", n_req=1, k_lo=k, k_hi=k, p_lo=p, p_hi=p, trials=10)
        return dict(kind="serve", prec="fp32", n_req=rng.randint(2, 48), k_lo=5, k_hi=40, p_lo=500,
                    p_hi=_log_int(rng, 2000, 20000), trials=10)
    if kind == "vi":
        n_kf = _log_int(rng, 10, 1500)
        return dict(kind="vi", prec=rng.choice(["fp64", "fp32"]), n_kf=n_kf,
                    n_pts=int(n_kf * rng.uniform(60, 150)), solver=rng.choice(["schur", "schur", "full"]),
                    trials=rng.randint(3, 6), tol=1e-8 if n_kf <= 60 else 1e-6,
                    max_pcg=200 if n_kf <= 60 else 100)
    return dict(kind="preint", n=_log_int(rng, 9, 4000), rate=rng.choice([100, 200, 400]))


# ------------------------------------------------------------------ inputs
def _scene(case, seed):
    """A bundle-adjustment scene whose first two cameras are held at their
    true values (the gauge, as in the local-BA requests)."""
    t = case["track"]
    track = ("uniform", 3, 8) if t == "u3-8" else ("geometric", 1.0 / int(t[1:]))
    sc = synth.make_scene(dict(n_cams=case["n_cams"], n_pts=case["n_pts"],
                               layout="ring" if case["n_cams"] <= 16 else "sphere", track=track,
                               loss=synth.HUBER if case["huber"] else synth.SQUARED, delta=1.0,
                               trials=case.get("trials", 1), pcg_max_iters=100, pcg_tol=case["tol"]),
                          seed=seed)
    sc.cams0[:2] = sc.cams_true[:2]
    fixed = np.zeros(case["n_cams"], bool)
    fixed[:2] = True
    return sc, fixed


def _requests(case, seed):
    """The requests of a burst: their sizes are the case's (log-uniform in its
    ranges), their scenes the seed's."""
    rng = np.random.default_rng(case["n_req"])
    size = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))  # noqa: E731
    reqs = []
    for k in range(case["n_req"]):
        n_kf, n_pts = size(case["k_lo"], case["k_hi"]), size(case["p_lo"], case["p_hi"])
        reqs.append(synth.make_local_request(100_003 * (seed % 20_011) + k, k_range=(n_kf, n_kf),
                                             np_range=(n_pts, n_pts), trials=case["trials"]))
    return reqs


def _rotation(phi):
    """Rotation matrices of rotation vectors (n, 3)."""
    th = np.linalg.norm(phi, axis=1)[:, None, None]
    K = np.zeros((len(phi), 3, 3))
    K[:, 0, 1], K[:, 0, 2], K[:, 1, 2] = -phi[:, 2], phi[:, 1], -phi[:, 0]
    K -= K.transpose(0, 2, 1)
    ths = np.where(th > 0, th, 1.0)
    return np.eye(3) + np.sin(ths) / ths * K + (1 - np.cos(ths)) / ths ** 2 * (K @ K)


def _rotvec(R):
    """Rotation vectors (n, 3) of rotation matrices."""
    v = 0.5 * np.stack([R[:, 2, 1] - R[:, 1, 2], R[:, 0, 2] - R[:, 2, 0], R[:, 1, 0] - R[:, 0, 1]], 1)
    s = np.linalg.norm(v, axis=1)
    c = 0.5 * (np.trace(R, axis1=1, axis2=2) - 1)
    return v * (np.arctan2(s, c) / np.where(s > 0, s, 1.0))[:, None]


def _vi_inputs(case, seed):
    sc = synth_vi.make_vi_scene(seed=seed, n_kf=case["n_kf"], n_pts=case["n_pts"], window=3)
    K = sc.n_kf
    rng = np.random.default_rng(seed + 1)
    pert = rng.normal(0, 1, (K, 9)) * np.repeat([0.01, 0.05, 0.05], 3)
    pert[0] = 0.0
    R0 = sc.R_true @ _rotation(pert[:, :3])
    states = np.concatenate([_rotvec(R0), sc.p_true + pert[:, 3:6], sc.v_true + pert[:, 6:9],
                             sc.bg_true, sc.ba_true], axis=1)
    pts = sc.pts + rng.normal(0, 0.05, sc.pts.shape)
    m = sc.gyro.shape[1]
    imu = dict(off=np.arange(K, dtype=np.int64) * m, gyro=sc.gyro.reshape(-1, 3),
               acc=sc.acc.reshape(-1, 3), dt=sc.imu_dt,
               bias0=np.concatenate([sc.bg_true[:-1], sc.ba_true[:-1]], axis=1))
    return sc, states, pts, imu


def _imu_inputs(case, seed):
    """IMU samples as a moving body gives them: rates and accelerations that
    vary over seconds, gravity, biases and noise; about 0.25 s an interval,
    with a dropped or an extra sample now and then."""
    rng = np.random.default_rng(seed)
    n, dt = case["n"], 1.0 / case["rate"]
    m = np.full(n, case["rate"] // 4) + rng.integers(-1, 2, n)
    off = np.concatenate([[0], np.cumsum(m)]).astype(np.int64)
    t = np.arange(off[-1])[:, None] * dt
    f, ph = rng.uniform(0.1, 1.5, (2, 3)), rng.uniform(0, 6.28, (2, 3))
    gyro = 0.4 * np.sin(f[0] * t + ph[0]) + rng.normal(0, _GYRO_NOISE / np.sqrt(dt), (len(t), 3))
    acc = (1.5 * np.sin(f[1] * t + ph[1]) + np.array([0, 0, 9.81]) +
           rng.normal(0, _ACC_NOISE / np.sqrt(dt), (len(t), 3)))
    bias0 = np.concatenate([rng.normal(0, 0.01, (n, 3)), rng.normal(0, 0.05, (n, 3))], axis=1)
    return off, gyro, acc, dt, bias0


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("solve", "step"):
        sc, fixed = _scene(case, seed)
        opts = gba.options(pcg_max_iters=100, pcg_tol=case["tol"],
                           solver=gba.GBA_SOLVER_SCHUR if case["solver"] == "schur" else gba.GBA_SOLVER_FULL,
                           jacobian=gba.GBA_JACOBIAN_DYNAMIC if case["solver"] == "full-dynamic"
                           else gba.GBA_JACOBIAN_ANALYTIC)
        g = gba.Graph.from_arrays(sc.cams0, sc.pts0, sc.cam_idx, sc.pt_idx, sc.obs, loss=sc.loss,
                                  delta=sc.delta, precision=_PREC[case["prec"]], options=opts,
                                  cam_fixed=fixed, use_torch=True)
        gba.gba_prepare(g.h)
        return dict(case=case, graph=g)
    if kind == "serve":
        srv = gba.Server(precision=_PREC[case["prec"]], budget_bytes=1 << 30, max_slots=64)
        return dict(case=case, server=srv, reqs=_requests(case, seed))
    if kind == "vi":
        sc, states, pts, imu = _vi_inputs(case, seed)
        pre = gba.gba_vi_preintegrate(0, imu["off"], imu["gyro"], imu["acc"], imu["dt"], imu["bias0"],
                                      _GYRO_NOISE, _ACC_NOISE)
        opts = gba.vi_options(pcg_max_iters=case["max_pcg"], pcg_tol=case["tol"],
                              solver=gba.GBA_SOLVER_SCHUR if case["solver"] == "schur" else gba.GBA_SOLVER_FULL,
                              precision=_PREC[case["prec"]])
        return dict(case=case, args=(states, pts, sc.st_kf, sc.st_pt, sc.st_obs, sc.intr, pre), opts=opts)
    return dict(case=case, args=_imu_inputs(case, seed))


def _taken(case, a):
    return a if case["prec"] == "fp64" else np.asarray(a).astype(np.float32)


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "solve":
        g = state["graph"]
        gba.gba_reset(g.h)
        rep = g.solve(case["trials"])
        return dict(cams=_taken(case, g.cameras()), pts=_taken(case, g.points()),
                    cost=_taken(case, rep.final_cost))
    if kind == "step":
        g = state["graph"]
        dc, dp, _ = gba.gba_eval_step(g.h, case["lam"], g.n_cams, g.n_pts)
        return dict(dcam=_taken(case, dc), dpt=_taken(case, dp))
    if kind == "serve":
        srv = state["server"]
        tickets = [srv.submit(r) for r in state["reqs"]]
        res = [srv.poll(t) for t in tickets]
        return dict(cams=_taken(case, np.concatenate([r["cams"] for r in res])),
                    pts=_taken(case, np.concatenate([r["pts"] for r in res])),
                    cost=_taken(case, np.array([r["report"]["final_cost"] for r in res])))
    if kind == "vi":
        st, pts, rep, _ = gba.gba_vi_solve(0, *state["args"], case["trials"], sigma_px=1.0,
                                           huber_delta2=7.815, sigma_gw=_GYRO_WALK, sigma_aw=_ACC_WALK,
                                           options=state["opts"])
        return dict(states=_taken(case, st), pts=_taken(case, pts), cost=_taken(case, rep["final_cost"]))
    return gba.gba_vi_preintegrate(0, *state["args"], _GYRO_NOISE, _ACC_NOISE)


def work(case):
    """Bytes and operations of one pass.  Every trial has to read each
    observation (pixels and the two indices), read and write the parameters,
    and evaluate residuals and Jacobians (about 500 operations an edge, with
    its block sums); every PCG iteration multiplies by J and its transpose
    (96 operations an edge for 2 x 12 entries), of which a well-conditioned
    step takes about ten."""
    kind = case["kind"]
    if kind in ("solve", "step"):
        mean = {"u3-8": 5.5, "g4": 5.0, "g7": 8.0}[case["track"]]
        ne, trials = case["n_pts"] * mean, case.get("trials", 1)
        return dict(bytes=trials * (24 * ne + 2 * 8 * (9 * case["n_cams"] + 3 * case["n_pts"])),
                    flops=trials * ne * (500 + 10 * 96))
    if kind == "serve":
        pts = math.sqrt(case["p_lo"] * case["p_hi"]) * case["n_req"]
        ne = 5.0 * pts
        return dict(bytes=case["trials"] * (24 * ne + 2 * 24 * pts), flops=case["trials"] * ne * (500 + 10 * 96))
    if kind == "vi":
        ne = 6.9 * case["n_pts"]
        return dict(bytes=case["trials"] * (32 * ne + 2 * 8 * (15 * case["n_kf"] + 3 * case["n_pts"])
                                            + 8 * 148 * case["n_kf"]),
                    flops=case["trials"] * ne * (400 + case["max_pcg"] / 2 * 72))
    samples = case["n"] * case["rate"] / 4
    return dict(bytes=48 * samples + 8 * (6 + 148) * case["n"], flops=samples * 2500)


# ------------------------------------------------- exact values, in 64 bits
def _dev():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _t(a, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a), device=_dev()).to(dtype)


def _project(c, x):
    """BAL camera c (9,) of point x (3,)."""
    w = c[:3]
    th2 = (w * w).sum()
    th = torch.sqrt(th2)
    wx = torch.linalg.cross(w, x)
    P = x + torch.sin(th) / th * wx + 2 * torch.sin(th / 2) ** 2 / th2 * torch.linalg.cross(w, wx) + c[3:6]
    p = -P[:2] / P[2]
    n = (p * p).sum()
    return c[6] * (1 + c[7] * n + c[8] * n * n) * p


class _Ba:
    """One bundle-adjustment problem: cost, linear system and damped step by
    the plain Schur complement (dense and factored for few cameras, conjugate
    gradients to rounding for many)."""

    def __init__(self, ci, pi, uv, fixed, huber, nc, npt):
        order = np.lexsort((ci, pi))
        self.ci, self.pi = _t(ci[order], torch.int64), _t(pi[order], torch.int64)
        self.uv, self.free = _t(uv[order]), _t(~fixed)
        self.huber, self.nc, self.np = huber, nc, npt

    def residual(self, cams, pts):
        return torch.vmap(_project)(cams[self.ci], pts[self.pi]) - self.uv

    def weight(self, r):
        s = (r * r).sum(1)
        q = torch.sqrt(s)
        if not self.huber:
            return 0.5 * s.sum(), torch.ones_like(s)
        return 0.5 * torch.where(s > 1, 2 * q - 1, s).sum(), torch.where(s > 1, 1 / q, torch.ones_like(s))

    def cost(self, cams, pts):
        return float(self.weight(self.residual(cams, pts))[0])

    def linearise(self, cams, pts):
        r = self.residual(cams, pts)
        _, w = self.weight(r)
        sw = torch.sqrt(w)[:, None]
        jc, jp = torch.vmap(torch.func.jacfwd(_project, argnums=(0, 1)))(cams[self.ci], pts[self.pi])
        self.r = sw * r
        self.jc = sw[:, :, None] * jc * self.free[self.ci][:, None, None]
        self.jp = sw[:, :, None] * jp
        z = lambda *s: torch.zeros(*s, dtype=torch.float64, device=r.device)  # noqa: E731
        self.hcc = z(self.nc, 9, 9).index_add_(0, self.ci, self.jc.mT @ self.jc)
        self.hpp = z(self.np, 3, 3).index_add_(0, self.pi, self.jp.mT @ self.jp)
        self.bc = z(self.nc, 9).index_add_(0, self.ci, (self.jc.mT @ self.r[:, :, None])[..., 0])
        self.bp = z(self.np, 3).index_add_(0, self.pi, (self.jp.mT @ self.r[:, :, None])[..., 0])

    def step(self, lam):
        damp = lambda H: H + lam * torch.diag_embed(torch.diagonal(H, dim1=1, dim2=2).clamp(1e-6, 1e32))  # noqa: E731
        A, C = damp(self.hcc), damp(self.hpp)
        Ci = torch.linalg.inv(C)
        W = self.jc.mT @ self.jp                                     # (edges, 9, 3)
        camsum = lambda e: torch.zeros_like(self.bc).index_add_(0, self.ci, e)  # noqa: E731
        ptsum = lambda e: torch.zeros_like(self.bp).index_add_(0, self.pi, e)  # noqa: E731
        mv = lambda M, v: (M * v[:, None, :]).sum(-1)  # noqa: E731
        rhs = -self.bc + camsum(mv(W, mv(Ci, self.bp)[self.pi]))
        if 9 * self.nc <= 2000:
            S = torch.block_diag(*A)
            L = torch.linalg.cholesky(Ci)
            Y = W @ L[self.pi]
            chunk = max(1, 40_000_000 // (27 * self.nc))
            for j0 in range(0, self.np, chunk):
                n = min(chunk, self.np - j0)
                sel = (self.pi >= j0) & (self.pi < j0 + n)
                D = torch.zeros(self.nc * n, 9, 3, dtype=torch.float64, device=S.device)
                D.index_add_(0, self.ci[sel] * n + self.pi[sel] - j0, Y[sel])
                D = D.view(self.nc, n, 9, 3).permute(0, 2, 1, 3).reshape(9 * self.nc, 3 * n)
                S -= D @ D.mT
            dc = torch.cholesky_solve(rhs.reshape(-1, 1), torch.linalg.cholesky(S)).view(-1, 9)
        else:
            blk = A.clone().index_add_(0, self.ci, -(W @ Ci[self.pi] @ W.mT))
            M = torch.linalg.inv(blk)
            x, r = torch.zeros_like(rhs), rhs.clone()
            z = mv(M, r)
            p, rz, r0 = z.clone(), (r * z).sum(), float((r * r).sum())
            for k in range(2000):
                t = mv(Ci, ptsum(mv(W.mT, p[self.ci])))
                q = mv(A, p) - camsum(mv(W, t[self.pi]))
                a = rz / (p * q).sum()
                x += a * p
                r -= a * q
                if k % 10 == 9 and float((r * r).sum()) <= 1e-24 * r0:
                    break
                z = mv(M, r)
                rz, old = (r * z).sum(), rz
                p = z + rz / old * p
            dc = x
        dp = -mv(Ci, self.bp + ptsum(mv(W.mT, dc[self.ci])))
        return dc, dp

    def solve(self, cams, pts, trials):
        F, lam, nu, fresh = self.cost(cams, pts), 1e-4, 2.0, True
        for _ in range(trials):
            if fresh:
                self.linearise(cams, pts)
            dc, dp = self.step(lam)
            y = (self.jc * dc[self.ci][:, None, :]).sum(-1) + (self.jp * dp[self.pi][:, None, :]).sum(-1)
            L = -float((self.bc * dc).sum() + (self.bp * dp).sum() + 0.5 * (y * y).sum())
            Fn = self.cost(cams + dc, pts + dp)
            fresh = L > 0 and Fn < F
            if fresh:
                cams, pts = cams + dc, pts + dp
                lam *= max(1 / 3, 1 - (2 * (F - Fn) / L - 1) ** 3)
                F, nu = Fn, 2.0
            else:
                lam, nu = lam * nu, nu * 2
        return cams, pts, F


def _exact_preint(off, gyro, acc, dt, bias0):
    """The deltas, bias Jacobians and covariance of every interval, the
    intervals side by side."""
    n = len(off) - 1
    m = np.diff(off)
    eye = np.broadcast_to(np.eye(3), (n, 3, 3))
    dR, dv, dp = eye.copy(), np.zeros((n, 3)), np.zeros((n, 3))
    JRg, Jvg, Jva, Jpg, Jpa = (np.zeros((n, 3, 3)) for _ in range(5))
    cov = np.zeros((n, 9, 9))
    T = lambda a: np.swapaxes(a, 1, 2)  # noqa: E731

    def hat(v):
        K = np.zeros((len(v), 3, 3))
        K[:, 0, 1], K[:, 0, 2], K[:, 1, 2] = -v[:, 2], v[:, 1], -v[:, 0]
        return K - T(K)

    for s in range(int(m.max()) if n else 0):
        on = np.flatnonzero(m > s)
        w = (gyro[off[on] + s] - bias0[on, :3]) * dt
        a = acc[off[on] + s] - bias0[on, 3:]
        R, E, K = dR[on], _rotation(w), hat(w)
        t2 = (w * w).sum(1)[:, None, None]
        t = np.sqrt(t2)
        small = t2 < 1e-6
        ts = np.where(small, 1.0, t)
        Jr = (np.eye(3) - np.where(small, 0.5 - t2 / 24, (1 - np.cos(ts)) / ts ** 2) * K +
              np.where(small, 1 / 6 - t2 / 120, (ts - np.sin(ts)) / ts ** 3) * (K @ K))
        Ra, Rax = (R @ a[:, :, None])[..., 0], R @ hat(a)
        A = np.broadcast_to(np.eye(9), (len(on), 9, 9)).copy()
        A[:, :3, :3], A[:, 3:6, :3], A[:, 6:, :3] = T(E), -Rax * dt, -0.5 * Rax * dt * dt
        A[:, 6:, 3:6] = np.eye(3) * dt
        Bg, Ba = np.zeros((len(on), 9, 3)), np.zeros((len(on), 9, 3))
        Bg[:, :3], Ba[:, 3:6], Ba[:, 6:] = Jr * dt, R * dt, 0.5 * R * dt * dt
        cov[on] = (A @ cov[on] @ T(A) + _GYRO_NOISE ** 2 / dt * Bg @ T(Bg) + _ACC_NOISE ** 2 / dt * Ba @ T(Ba))
        RJ = Rax @ JRg[on]
        Jpa[on] += Jva[on] * dt - 0.5 * R * dt * dt
        Jpg[on] += Jvg[on] * dt - 0.5 * RJ * dt * dt
        Jva[on] -= R * dt
        Jvg[on] -= RJ * dt
        JRg[on] = T(E) @ JRg[on] - Jr * dt
        dp[on] += dv[on] * dt + 0.5 * Ra * dt * dt
        dv[on] += Ra * dt
        dR[on] = R @ E
    flat = lambda a: a.reshape(n, -1)  # noqa: E731
    return np.concatenate([(dt * m)[:, None], flat(dR), dv, dp, flat(JRg), flat(Jvg), flat(Jva), flat(Jpg),
                           flat(Jpa), bias0, flat(0.5 * (cov + T(cov)))], axis=1)


def _hat(v):
    z = torch.zeros_like(v[0])
    return torch.stack([torch.stack([z, -v[2], v[1]]), torch.stack([v[2], z, -v[0]]), torch.stack([-v[1], v[0], z])])


def _exp_small(v):
    """Exp of a rotation vector well below one radian (to rounding)."""
    K = _hat(v)
    E = torch.eye(3, dtype=v.dtype, device=v.device)
    for k in range(12, 0, -1):
        E = torch.eye(3, dtype=v.dtype, device=v.device) + K @ E / k
    return E


def _inertial(u, Ri, Rj, si, sj, pre):
    """Inertial residual (9) of two keyframes (states p, v, bg, ba) perturbed
    by u = (dtheta_i, dp_i, dv_i, dbg_i, dba_i, dtheta_j, dp_j, dv_j)."""
    g = torch.tensor([0.0, 0.0, -9.81], dtype=u.dtype, device=u.device)
    m = lambda k: pre[k:k + 9].view(3, 3)  # noqa: E731
    dt = pre[0]
    Ri, Rj = Ri @ (torch.eye(3, dtype=u.dtype, device=u.device) + _hat(u[:3])), \
        Rj @ (torch.eye(3, dtype=u.dtype, device=u.device) + _hat(u[15:18]))
    pi, vi, bg, ba = (si + u[3:15]).view(4, 3)
    pj, vj = (sj[:6] + u[18:24]).view(2, 3)
    dbg, dba = bg - pre[61:64], ba - pre[64:67]
    E = (m(1) @ _exp_small(m(16) @ dbg)).T @ Ri.T @ Rj
    v = 0.5 * torch.stack([E[2, 1] - E[1, 2], E[0, 2] - E[2, 0], E[1, 0] - E[0, 1]])
    s2 = (v * v).sum()
    f = 1 + s2 / 6 * (1 + s2 * 9 / 20 * (1 + s2 * 25 / 42 * (1 + s2 * 49 / 72 * (1 + s2 * 81 / 110))))
    rv = Ri.T @ (vj - vi - g * dt) - (pre[10:13] + m(25) @ dbg + m(34) @ dba)
    rp = Ri.T @ (pj - pi - vi * dt - 0.5 * g * dt * dt) - (pre[13:16] + m(43) @ dbg + m(52) @ dba)
    return torch.cat([f * v, rv, rp])


def _stereo(u, R, p, X, intr):
    """Prediction (u_l, v_l, u_r) with (dtheta, dp, dX) = u."""
    Xc = (R @ (torch.eye(3, dtype=u.dtype, device=u.device) + _hat(u[:3]))).T @ (X + u[6:] - p - u[3:6])
    ul = intr[0] * Xc[0] / Xc[2] + intr[2]
    return torch.stack([ul, intr[1] * Xc[1] / Xc[2] + intr[3], ul - intr[0] * intr[4] / Xc[2]])


def _exact_vi(case, seed):
    sc, states, pts, imu = _vi_inputs(case, seed)
    K, N = sc.n_kf, len(pts)
    off = imu["off"]
    pre = _t(_exact_preint(off, imu["gyro"], imu["acc"], imu["dt"], imu["bias0"]))
    om = torch.linalg.inv(pre[:, 67:].view(-1, 9, 9))
    ob = torch.cat([(1 / (s * s * pre[:, :1])).expand(-1, 3) for s in (_GYRO_WALK, _ACC_WALK)], 1)
    kf, pt, obs, intr = _t(sc.st_kf, torch.int64), _t(sc.st_pt, torch.int64), _t(sc.st_obs), _t(sc.intr)
    R, s, X = _t(_rotation(states[:, :3])), _t(states[:, 3:]), _t(pts)
    d2 = 7.815
    z9, z24 = torch.zeros(len(kf), 9, dtype=R.dtype, device=R.device), torch.zeros(K - 1, 24, dtype=R.dtype, device=R.device)
    st, ine = torch.vmap(_stereo, (0, 0, 0, 0, None)), torch.vmap(_inertial)

    def terms(R, s, X):
        r = st(z9, R[kf], s[kf, :3], X[pt], intr) - obs
        q = (r * r).sum(1)
        out = q > d2
        w = torch.where(out, math.sqrt(d2) / torch.sqrt(q), torch.ones_like(q))
        ri = ine(z24, R[:-1], R[1:], s[:-1], s[1:], pre)
        rb = s[1:, 6:] - s[:-1, 6:]
        F = 0.5 * torch.where(out, 2 * math.sqrt(d2) * torch.sqrt(q) - d2, q).sum() + \
            0.5 * (ri * (om @ ri[:, :, None])[..., 0]).sum() + 0.5 * (ob * rb * rb).sum()
        return float(F), r, w, ri, rb

    F, lam, nu, fresh = terms(R, s, X)[0], 1e-4, 2.0, True
    f = torch.arange(K - 1, device=R.device)
    for _ in range(case["trials"]):
        if fresh:
            _, r, w, ri, rb = terms(R, s, X)
            J = torch.vmap(torch.func.jacfwd(_stereo), (0, 0, 0, 0, None))(z9, R[kf], s[kf, :3], X[pt], intr)
            J = J * torch.sqrt(w)[:, None, None]
            r = r * torch.sqrt(w)[:, None]
            Ji = torch.vmap(torch.func.jacfwd(_inertial))(z24, R[:-1], R[1:], s[:-1], s[1:], pre)
            J[kf == 0, :, :6] = 0
            Ji[0, :, :15] = 0
            zk = lambda *n: torch.zeros(*n, dtype=R.dtype, device=R.device)  # noqa: E731
            Hk, bk = zk(K * K, 15, 15), zk(K, 15)
            Jk = torch.cat([J[:, :, :6], zk(len(kf), 3, 9)], 2)
            Hk.index_add_(0, kf * (K + 1), Jk.mT @ Jk)
            bk.index_add_(0, kf, (Jk.mT @ r[:, :, None])[..., 0])
            Jb = zk(K - 1, 6, 30)
            Jb[:, range(6), range(9, 15)] = -1.0
            Jb[:, range(6), range(24, 30)] = 1.0
            Jb[0, :, :15] = 0
            Jt = torch.cat([torch.cat([Ji, zk(K - 1, 9, 6)], 2), Jb], 1)         # (K-1, 15, 30)
            O = torch.cat([torch.cat([om, zk(K - 1, 9, 6)], 2), torch.cat([zk(K - 1, 6, 9), torch.diag_embed(ob)], 2)], 1)
            H30 = Jt.mT @ O @ Jt
            g30 = (Jt.mT @ O @ torch.cat([ri, rb], 1)[:, :, None])[..., 0]
            for a in range(2):
                bk.index_add_(0, f + a, g30[:, 15 * a:15 * a + 15])
                for c in range(2):
                    Hk.index_add_(0, (f + a) * K + f + c, H30[:, 15 * a:15 * a + 15, 15 * c:15 * c + 15])
            A = Hk.view(K, K, 15, 15).permute(0, 2, 1, 3).reshape(15 * K, 15 * K)
            Jp = J[:, :, 6:]
            C = zk(N, 3, 3).index_add_(0, pt, Jp.mT @ Jp)
            bp = zk(N, 3).index_add_(0, pt, (Jp.mT @ r[:, :, None])[..., 0])
            B = zk(K * N, 15, 3).index_add_(0, kf * N + pt, Jk.mT @ Jp)
            B = B.view(K, N, 15, 3).permute(0, 2, 1, 3).reshape(15 * K, 3 * N)
        Al = A + lam * torch.diag(torch.diagonal(A).clamp(1e-6, 1e32))
        Ci = torch.linalg.inv(C + lam * torch.diag_embed(torch.diagonal(C, dim1=1, dim2=2).clamp(1e-6, 1e32)))
        BC = torch.einsum("rnk,nkc->rnc", B.view(-1, N, 3), Ci).reshape(15 * K, 3 * N)
        xk = torch.linalg.solve(Al - BC @ B.T, (-bk.reshape(-1) + BC @ bp.reshape(-1)))
        xp = -(Ci @ (bp + (B.T @ xk).view(N, 3))[:, :, None])[..., 0]
        Bx = B @ xp.reshape(-1)
        L = -float(bk.reshape(-1) @ xk + (bp * xp).sum() + 0.5 * (xk @ (A @ xk) + 2 * xk @ Bx + (xp * (C @ xp[:, :, None])[..., 0]).sum()))
        x = xk.view(K, 15)
        Rn, sn, Xn = R @ _t(_rotation(x[:, :3].cpu().numpy())), s + x[:, 3:], X + xp
        Fn = terms(Rn, sn, Xn)[0]
        fresh = L > 0 and Fn < F
        if fresh:
            R, s, X = Rn, sn, Xn
            lam *= max(1 / 3, 1 - (2 * (F - Fn) / L - 1) ** 3)
            F, nu = Fn, 2.0
        else:
            lam, nu = lam * nu, nu * 2
    return dict(states=np.concatenate([_rotvec(R.cpu().numpy()), s.cpu().numpy()], 1), pts=X, cost=F)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("solve", "step"):
        if kind == "solve" and case["n_cams"] > 222:
            return None     # thousands of plain conjugate-gradient iterations: over twenty seconds
        sc, fixed = _scene(case, seed)
        ba = _Ba(sc.cam_idx, sc.pt_idx, sc.obs, fixed, case["huber"], sc.n_cams, sc.n_pts)
        cams, pts = _t(sc.cams0), _t(sc.pts0)
        if kind == "solve":
            c, p, F = ba.solve(cams, pts, case["trials"])
            return dict(cams=c, pts=p, cost=F)
        ba.linearise(cams, pts)
        dc, dp = ba.step(case["lam"])
        return dict(dcam=dc, dpt=dp)
    if kind == "serve":
        got = []
        for q in _requests(case, seed):
            ba = _Ba(q["cam_idx"], q["pt_idx"], q["uv"], q["cam_fixed"], True, len(q["cams"]), len(q["pts"]))
            got.append(ba.solve(_t(q["cams"]), _t(q["pts"]), case["trials"]))
        return dict(cams=torch.cat([g[0] for g in got]), pts=torch.cat([g[1] for g in got]),
                    cost=np.array([g[2] for g in got]))
    if kind == "preint":
        return _exact_preint(*_imu_inputs(case, seed))
    # on a long trajectory the PCG stops at its iteration limit, far from the exact step
    return _exact_vi(case, seed) if case["n_kf"] <= 60 and case["solver"] == "schur" else None
