"""Visual-inertial solves that are refused before any device work (no GPU)."""
import numpy as np
import pytest

from paper_2509_26581_amd import gba


@pytest.mark.parametrize("kf,pt,status", [(0, 2, -2), (0, -1, -2), (2, 0, -2), (-1, 0, -2), (1, 1, -6)])
def test_unknown_ids_name_the_status_without_a_device(kf, pt, status):
    # no such device: ids that are not there are GBA_ERR_UNKNOWN_ID all the same
    with pytest.raises(gba.GbaError) as e:
        gba.gba_vi_solve(99, np.zeros((2, 15)), np.zeros((2, 3)), np.array([0, kf]), np.array([1, pt]),
                         np.zeros((2, 3)), (400.0, 400.0, 320.0, 240.0, 0.1), np.ones((1, 148)), 1)
    assert e.value.status == status
