"""The automatic split of the whole-system products into workgroups against a
split of 16 tiles: the same truncated FP64 steps (the sums' order differs; a
few steps amplify rounding by less than 1e6), from one tile to several
workgroups, with stored and recomputed Jacobians."""
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


@pytest.mark.parametrize("jacobian", [gba.GBA_JACOBIAN_ANALYTIC, gba.GBA_JACOBIAN_DYNAMIC])
@pytest.mark.parametrize("n_cams,n_pts", [(3, 8), (8, 45), (9, 60), (20, 800), (60, 5000)])
def test_full_steps_are_the_same_for_any_split(n_cams, n_pts, jacobian):
    sc = synth.make_scene("small", seed=n_cams, n_cams=n_cams, n_pts=n_pts)
    out = []
    for tiles in (0, 16):
        g = gba.Graph.from_arrays(sc.cams0, sc.pts0, sc.cam_idx, sc.pt_idx, sc.obs, loss=gba.GBA_LOSS_HUBER,
                                  delta=1.0, precision=gba.GBA_FP64,
                                  options=gba.options(pcg_max_iters=4, pcg_tol=0.0, solver=gba.GBA_SOLVER_FULL,
                                                      jacobian=jacobian, tiles_per_block=tiles))
        out.append(gba.gba_eval_step(g.h, 1e-3, sc.n_cams, sc.n_pts))
        g.close()
    for a, b in zip(out[0][:2], out[1][:2]):
        assert np.linalg.norm(a - b) <= 1e-9 * np.linalg.norm(b)
    assert out[0][2] == out[1][2]
