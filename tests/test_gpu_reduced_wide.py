"""Launched PCG iterations on the explicit reduced system (one problem of 57
cameras and more) against the implicit products of the same library: the same
truncated iterates in FP64, the same one-trial solves in the mixed modes, over
the pair densities that change the forming kernel's lanes (most pairs with few
common points, about twenty, more than forty), the first size that takes it
and the first past its bounds.  The bounds are those of the small systems: a
few steps amplify rounding by less than 1e6 in FP64 (1e-9), 1e-3 in the mixed
modes."""
import numpy as np
import pytest

from paper_2509_26581_amd import gba, synth
from test_gpu_reduced import _agree, _one_trial, _step

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    gba.load()


@pytest.mark.parametrize("precision", [gba.GBA_FP64, gba.GBA_MIXED_FP32, gba.GBA_MIXED_BF16])
@pytest.mark.parametrize("n_cams,n_pts", [(57, 500), (57, 3001), (63, 12000), (113, 4001), (128, 1000),
                                          (200, 20000), (352, 3000)])
def test_truncated_steps_equal_the_implicit_products(n_cams, n_pts, precision):
    sc = synth.make_scene("small", seed=n_cams, n_cams=n_cams, n_pts=n_pts, layout="sphere")
    fixed = np.zeros(n_cams, bool)
    fixed[[0, n_cams - 1]] = True
    keep = sc.pt_idx < n_pts - 3   # the last points lose their observations
    sc.cam_idx, sc.pt_idx, sc.obs = sc.cam_idx[keep], sc.pt_idx[keep], sc.obs[keep]
    take = _step if precision == gba.GBA_FP64 else _one_trial
    got = take(sc, precision, gba.GBA_ACC_AUTO, 4, fixed)
    want = take(sc, precision, gba.GBA_ACC_LDS, 4, fixed)
    assert not got[0][0].any() and not got[1][n_pts - 3:].any()
    _agree(got, want, 1e-9 if precision == gba.GBA_FP64 else 1e-3)


def _graph(sc, precision, **opt):
    return gba.Graph.from_arrays(sc.cams0, sc.pts0, sc.cam_idx, sc.pt_idx, sc.obs, loss=gba.GBA_LOSS_HUBER,
                                 delta=1.0, precision=precision, options=gba.options(**opt))


def test_stop_rules_equal_the_implicit_products():
    sc = synth.make_scene("small", seed=5, n_cams=80, n_pts=4000, layout="sphere")
    for opt in (dict(pcg_tol=1e-3), dict(pcg_tol=0.0, pcg_max_iters=60, pcg_rejection_ratio=1.0)):
        out = []
        for acc in (gba.GBA_ACC_AUTO, gba.GBA_ACC_LDS):
            g = _graph(sc, gba.GBA_FP64, accumulation=acc, **opt)
            out.append(gba.gba_eval_step(g.h, 1e-3, sc.n_cams, sc.n_pts))
            g.close()
        _agree(out[0], out[1], 1e-6)


def test_solves_and_single_steps_alternate():
    # a mixed-mode handle multiplies by S in its solves and keeps to the point
    # passes in gba_eval_step: neither replays the other's recorded iterations
    sc = synth.make_scene("small", seed=6, n_cams=70, n_pts=3000, layout="sphere")
    opt = dict(pcg_max_iters=30, pcg_tol=1e-3)
    g = _graph(sc, gba.GBA_MIXED_FP32, **opt)
    one = _graph(sc, gba.GBA_MIXED_FP32, **opt)
    want_step = gba.gba_eval_step(one.h, 1e-3, sc.n_cams, sc.n_pts)
    one.close()
    costs = []
    for _ in range(3):
        gba.gba_reset(g.h)
        costs.append(g.solve(4).final_cost)
        gba.gba_reset(g.h)
        step = gba.gba_eval_step(g.h, 1e-3, sc.n_cams, sc.n_pts)
        np.testing.assert_array_equal(step[0], want_step[0])
    g.close()
    assert max(costs) - min(costs) <= 1e-6 * min(costs)
