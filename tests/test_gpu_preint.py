"""Preintegration of intervals of unequal lengths (none, one, and the edges of
the 16 samples a row of lanes prepares at once) side by side, in counts that do
not fill a workgroup, against the oracle."""
import numpy as np
import pytest

from oracle import imu
from paper_2509_26581_amd import gba

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    gba.load()


@pytest.mark.parametrize("lengths", [[1], [0, 3], [15, 16, 17], [33, 0, 1, 48, 5], [100, 2, 31, 32, 64, 0, 7, 16, 1]])
def test_unequal_intervals_match_the_oracle(lengths):
    rng = np.random.default_rng(sum(lengths))
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    gyro, acc = rng.normal(0, 0.5, (off[-1], 3)), rng.normal(0, 3.0, (off[-1], 3))
    gyro[::7] = 0.0   # the series of Exp and of the right Jacobian
    bias = rng.normal(0, 0.01, (len(lengths), 6))
    bias[0] = 0.0
    out = gba.gba_vi_preintegrate(0, off, gyro, acc, 0.005, bias, 1.7e-4, 2e-3)
    for f in range(len(lengths)):
        s = slice(off[f], off[f + 1])
        P = imu.preintegrate(gyro[s], acc[s], 0.005, bias[f, :3], bias[f, 3:], 1.7e-4, 2e-3)
        o = out[f]
        assert o[0] == pytest.approx(lengths[f] * 0.005, rel=1e-15)
        np.testing.assert_allclose(o[1:10].reshape(3, 3), P.dR, rtol=0, atol=1e-13)
        np.testing.assert_allclose(o[10:16], np.concatenate([P.dv, P.dp]), rtol=0,
                                   atol=1e-13 * max(1, np.abs(P.dv).max()))
        for k, J in enumerate((P.JRg, P.Jvg, P.Jva, P.Jpg, P.Jpa)):
            np.testing.assert_allclose(o[16 + 9 * k:25 + 9 * k].reshape(3, 3), J, rtol=0, atol=1e-13)
        np.testing.assert_array_equal(o[61:67], bias[f])
        np.testing.assert_allclose(o[67:148].reshape(9, 9), P.cov, rtol=1e-10, atol=1e-22)
