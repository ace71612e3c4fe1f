"""Points with more than 64 observations in the visual-inertial Schur solve
(they are split over wavefronts, and their observations ordered by sorts instead
of ranked): explicit keyframe blocks next to such points, repeated observations
of one, and the time their ordering takes."""
import numpy as np
import pytest

from oracle import imu, vi
from paper_2509_26581_amd import gba, synth_vi

pytestmark = pytest.mark.gpu

SIG_G, SIG_A, SIG_GW, SIG_AW = 1.7e-4, 2e-3, 2e-5, 3e-3


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    gba.load()


def _problem(n_kf, n_pts, n_long, short, twice=0):
    """A scene in which n_long points keep their tracks of more than 64
    observations and the others their first `short`; shuffled; `twice`
    observations of the long points repeated."""
    sc = synth_vi.make_vi_scene(seed=4, n_kf=n_kf, n_pts=n_pts, kf_dt=0.05)
    rng = np.random.default_rng(11)
    cnt = np.bincount(sc.st_pt, minlength=n_pts)
    longs = np.flatnonzero(cnt > 64)[:n_long]
    assert len(longs) == n_long
    seen = np.zeros(n_pts, int)
    keep = np.zeros(len(sc.st_kf), bool)
    for e, j in enumerate(sc.st_pt):
        keep[e] = j in longs or seen[j] < short
        seen[j] += 1
    kf, pt, obs = sc.st_kf[keep], sc.st_pt[keep], sc.st_obs[keep]
    order = rng.permutation(len(kf))
    again = order[np.isin(pt[order], longs)][:twice]
    order = np.concatenate([order, again])
    kf, pt, obs = kf[order], pt[order], obs[order] + 0.0
    obs[len(order) - len(again):] += 0.5
    R0 = np.stack([sc.R_true[k] @ imu.so3_exp(rng.normal(0, 0.01, 3) if k else np.zeros(3)) for k in range(n_kf)])
    dp, dv = rng.normal(0, 0.05, (2, n_kf, 3))
    dp[0] = dv[0] = 0.0
    X0 = sc.pts + rng.normal(0, 0.05, sc.pts.shape)
    x0 = vi.VIState(R0, sc.p_true + dp, sc.v_true + dv, sc.bg_true.copy(), sc.ba_true.copy(), X0)
    pre_o = [imu.preintegrate(sc.gyro[f], sc.acc[f], sc.imu_dt, sc.bg_true[f], sc.ba_true[f], SIG_G, SIG_A)
             for f in range(n_kf - 1)]
    prob = vi.VIProblem(kf, pt, obs, sc.intr, pre_o, sigma_px=1.0, delta2=7.815, sigma_gw=SIG_GW, sigma_aw=SIG_AW)
    off = np.arange(n_kf, dtype=np.int64) * sc.gyro.shape[1]
    pre_g = gba.gba_vi_preintegrate(0, off, sc.gyro.reshape(-1, 3), sc.acc.reshape(-1, 3), sc.imu_dt,
                                    np.concatenate([sc.bg_true[:-1], sc.ba_true[:-1]], axis=1), SIG_G, SIG_A)
    states = np.concatenate([np.array([imu.so3_log(R) for R in R0]), x0.p, x0.v, x0.bg, x0.ba], axis=1)

    def run(trials, **opt):
        return gba.gba_vi_solve(0, states, X0, kf, pt, obs, sc.intr, pre_g, trials, sigma_px=1.0,
                                huber_delta2=7.815, sigma_gw=SIG_GW, sigma_aw=SIG_AW,
                                options=gba.vi_options(solver=gba.GBA_SOLVER_SCHUR, **opt))
    return prob, x0, run, pt


@pytest.mark.parametrize("precision,bound", [(gba.GBA_FP64, 1e-8), (gba.GBA_MIXED_FP32, 1e-4)])
@pytest.mark.parametrize("k", [1, 6])
def test_explicit_blocks_with_long_tracks(k, precision, bound):
    # tolerances as for the other truncated steps: FP64 sums in another order;
    # the mixed mode's own for a first trial's step
    prob, x0, run, pt = _problem(70, 400, 5, 6)
    cnt = np.bincount(pt)
    pairs = int((cnt * (cnt - 1) // 2).sum())
    assert cnt.max() > 64 and pairs <= 16 * len(pt)   # explicit blocks
    _, _, rep, log = run(1, pcg_tol=0.0, pcg_max_iters=k, precision=precision)
    lin = prob.linearize(x0)
    dx, steps = prob.schur_pcg_step(lin, 1e-4, 1e-6, 1e32, 0.0, k)
    t = log[0]
    assert t["pcg_iters"] == steps == k
    F1, L = prob.cost(prob.step(x0, dx)), prob.model_decrease(lin, dx)
    assert abs(t["candidate_cost"] - F1) <= bound * F1, (t, F1)
    assert abs(t["model_decrease"] - L) <= bound * abs(L), (t, L)
    assert abs(t["step_norm"] - np.linalg.norm(dx)) <= bound * np.linalg.norm(dx)


def test_repeated_observations_of_long_tracks():
    # (implicit products, and not the exact diagonal blocks: converged)
    prob, x0, run, _ = _problem(70, 120, 5, 6, twice=40)
    _, _, _, log = run(1, pcg_tol=1e-12, pcg_max_iters=4000)
    lin = prob.linearize(x0)
    dx, _ = prob.schur_pcg_step(lin, 1e-4, 1e-6, 1e32, 1e-12, 4000)
    t = log[0]
    F1, L = prob.cost(prob.step(x0, dx)), prob.model_decrease(lin, dx)
    assert abs(t["candidate_cost"] - F1) <= 1e-8 * F1, (t, F1)
    assert abs(t["model_decrease"] - L) <= 1e-6 * abs(L), (t, L)
    assert abs(t["step_norm"] - np.linalg.norm(dx)) <= 1e-6 * np.linalg.norm(dx)


def test_ordering_time_is_near_linear():
    # 300,000 observations of one point: the set-up (uploads, orders) of a solve
    # takes some milliseconds; ranking each against the whole run took 72 ms
    sc = synth_vi.make_vi_scene(seed=4, n_kf=40, n_pts=60, kf_dt=0.05)
    cnt = np.bincount(sc.st_pt, minlength=60)
    j = int(np.argmax(cnt))
    mine = np.flatnonzero(sc.st_pt == j)
    e = np.concatenate([np.arange(len(sc.st_kf)), np.resize(mine, 300_000)])
    off = np.arange(40, dtype=np.int64) * sc.gyro.shape[1]
    pre = gba.gba_vi_preintegrate(0, off, sc.gyro.reshape(-1, 3), sc.acc.reshape(-1, 3), sc.imu_dt,
                                  np.concatenate([sc.bg_true[:-1], sc.ba_true[:-1]], axis=1), SIG_G, SIG_A)
    states = np.concatenate([np.array([imu.so3_log(R) for R in sc.R_true]), sc.p_true, sc.v_true, sc.bg_true,
                             sc.ba_true], axis=1)
    args = (0, states, sc.pts, sc.st_kf[e], sc.st_pt[e], sc.st_obs[e], sc.intr, pre, 1)
    rep = None
    for _ in range(2):
        _, _, rep, _ = gba.gba_vi_solve(*args, options=gba.vi_options(pcg_tol=0.0, pcg_max_iters=2))
    assert rep["ms_other"] < 50.0
