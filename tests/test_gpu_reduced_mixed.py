"""Mixed modes on the explicit reduced camera system: its sums, products and
vectors are FP64 (the launched products' camera sums are too), so a step's
error against the FP64 mode is that of the FP32 inputs (stored Jacobians,
point inverses, right-hand side)."""
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


def _cam_step(sc, precision, acc, steps):
    fixed = np.zeros(sc.n_cams, bool)
    fixed[0] = True
    g = gba.Graph.from_arrays(sc.cams0, sc.pts0, sc.cam_idx, sc.pt_idx, sc.obs, loss=gba.GBA_LOSS_HUBER,
                              delta=1.0, precision=precision, cam_fixed=fixed,
                              options=gba.options(pcg_max_iters=steps, pcg_tol=0.0, accumulation=acc,
                                                  initial_lambda=1e-3))
    try:
        rep = g.solve(1)
        assert rep.accepted == 1 and rep.pcg_iters_total == steps
        return g.cameras() - sc.cams0
    finally:
        g.close()


@pytest.mark.parametrize("n_cams,n_pts", [(5, 16000), (6, 16000)])
def test_sums_over_many_common_points(n_cams, n_pts):
    # Every block of S sums 16,000 terms of one sign.  The
    # launched products round each edge's term and every vector to FP32 in each
    # of 12 iterations; with FP64 sums and vectors only the inputs' roundings
    # are left, about a tenth of that: a fifth allowed.
    sc = synth.make_scene("small", seed=3, n_cams=n_cams, n_pts=n_pts, track=("uniform", n_cams, n_cams))
    want = _cam_step(sc, gba.GBA_FP64, gba.GBA_ACC_LDS, 12)
    err = [np.linalg.norm(_cam_step(sc, gba.GBA_MIXED_FP32, acc, 12) - want)
           for acc in (gba.GBA_ACC_AUTO, gba.GBA_ACC_LDS)]
    assert err[0] <= 0.2 * err[1], err
