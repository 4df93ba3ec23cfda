"""Inscribed-sphere maps of boxes short in x, whose distance passes give several rows to a wave, bit
for bit against the oracle."""
import numpy as np
import pytest

import paper_1410_1921_amd.workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx", [1, 2, 3, 4, 7, 8, 9, 16, 17, 31, 32, 33, 63, 64, 65])
def test_short_rows(nx):
    """Distance passes with several rows to a wave: powers of two and beside them, row counts that
    leave a wave and a workgroup partly filled."""
    import torch

    from paper_1410_1921_amd import lbm
    import oracle as orc
    for ny, nz, p in ((1, 1, 0.6), (5, 67, 0.7), (131, 9, 0.8)):
        m = W.random_mask((nz, ny, nx), p, nx + ny)
        m[0, 0, 0] = 0
        d = lbm.lbm_pore_diameter(torch.from_numpy(m).cuda(), lbm.LBM_PSD_MIS).cpu().numpy()
        assert np.array_equal(d, orc.mis(m)), (ny, nz)
