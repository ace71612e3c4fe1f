"""The explicit reduced camera system (small problems) against the implicit
products of the same library: the same truncated PCG iterates (FP64, through
gba_eval_step) and the same one-trial solves (mixed modes, where that entry
point keeps to the launched products) on the same scenes, at the edges of its layout (wavefront and column-group boundaries, the
largest size it takes and the first it does not), with fixed cameras, points
without observations and point counts around a bitmap word.

Both sides run the same recurrence on the same stored Jacobian; they differ in
the order of the sums.  A few steps amplify rounding by less than 1e6 in FP64
(1e-9 here); in the mixed modes the policy's own bound on solutions holds
(1e-3)."""
import numpy as np
import pytest

from paper_2509_26581_amd import gba, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    gba.load()


def _step(sc, precision, acc, steps, cam_fixed, extra=None, tol=0.0):
    ci, pi, obs = sc.cam_idx, sc.pt_idx, sc.obs
    if extra is not None:
        ci, pi, obs = (np.concatenate([a, b]) for a, b in zip((ci, pi, obs), extra))
    g = gba.Graph.from_arrays(sc.cams0, sc.pts0, ci, pi, obs, loss=gba.GBA_LOSS_HUBER, delta=1.0,
                              precision=precision, cam_fixed=cam_fixed,
                              options=gba.options(pcg_max_iters=steps, pcg_tol=tol, accumulation=acc))
    try:
        return gba.gba_eval_step(g.h, 1e-3, sc.n_cams, sc.n_pts)
    finally:
        g.close()


def _one_trial(sc, precision, acc, steps, cam_fixed):
    g = gba.Graph.from_arrays(sc.cams0, sc.pts0, sc.cam_idx, sc.pt_idx, sc.obs, loss=gba.GBA_LOSS_HUBER,
                              delta=1.0, precision=precision, cam_fixed=cam_fixed,
                              options=gba.options(pcg_max_iters=steps, pcg_tol=0.0, accumulation=acc,
                                                  initial_lambda=1e-3))
    try:
        rep = g.solve(1)
        assert rep.accepted == 1
        return g.cameras() - sc.cams0, g.points() - sc.pts0, rep.pcg_iters_total
    finally:
        g.close()


def _agree(a, b, bound):
    for x, y in zip(a[:2], b[:2]):
        assert np.linalg.norm(x - y) <= bound * np.linalg.norm(y)
    assert a[2] == b[2]


@pytest.mark.parametrize("precision", [gba.GBA_FP64, gba.GBA_MIXED_FP32, gba.GBA_MIXED_BF16])
@pytest.mark.parametrize("n_cams,n_pts", [(2, 40), (7, 63), (8, 64), (14, 65), (15, 400), (28, 1023),
                                          (29, 1500), (42, 2000), (43, 2048), (56, 3001), (57, 3001)])
def test_truncated_steps_equal_the_implicit_products(n_cams, n_pts, precision):
    sc = synth.make_scene("small", seed=n_cams, n_cams=n_cams, n_pts=n_pts, layout="sphere")
    fixed = np.zeros(n_cams, bool)
    fixed[0] = True
    # the last points lose their observations
    keep = sc.pt_idx < n_pts - 3
    sc.cam_idx, sc.pt_idx, sc.obs = sc.cam_idx[keep], sc.pt_idx[keep], sc.obs[keep]
    take = _step if precision == gba.GBA_FP64 else _one_trial
    got = take(sc, precision, gba.GBA_ACC_AUTO, 4, fixed)
    want = take(sc, precision, gba.GBA_ACC_LDS, 4, fixed)
    assert not got[0][0].any() and not got[1][n_pts - 3:].any()
    _agree(got, want, 1e-9 if precision == gba.GBA_FP64 else 1e-3)


def test_a_point_seen_twice_by_a_camera():
    sc = synth.make_scene("small", seed=3, n_cams=9, n_pts=200)
    extra = (sc.cam_idx[:5], sc.pt_idx[:5], sc.obs[:5] + 0.5)
    got = _step(sc, gba.GBA_FP64, gba.GBA_ACC_AUTO, 4, None, extra)
    want = _step(sc, gba.GBA_FP64, gba.GBA_ACC_LDS, 4, None, extra)
    _agree(got, want, 1e-9)


def test_requests_of_every_class_in_one_batch():
    # small, middle and large requests side by side: each as alone
    reqs = [synth.make_local_request(70 + k, k_range=(n, n), np_range=(300 + 40 * n, 300 + 40 * n))
            for k, n in enumerate((5, 14, 15, 29, 40))]
    alone, mixed = [], []
    for batch, out in ([[r] for r in reqs], alone), ([reqs], mixed):
        for rs in batch:
            s = gba.Server(precision=gba.GBA_FP64, budget_bytes=256 << 20, max_slots=8)
            try:
                out += [s.poll(t) for t in [s.submit(r) for r in rs]]
            finally:
                s.close()
    for a, b in zip(alone, mixed):
        assert abs(a["report"]["final_cost"] - b["report"]["final_cost"]) <= 1e-10 * a["report"]["final_cost"]
