"""The flow sweep finds a node's sources through one record per neighbouring row: rows that
end inside a 32-voxel half segment, at its end and at a segment's end, rows shorter than a
half, and lanes that stand at both ends of a half at once (nx = 33), against the oracle."""
import numpy as np
import pytest
import torch

import paper_1410_1921_amd.workloads as W
from paper_1410_1921_amd import lbm

pytestmark = pytest.mark.gpu

W19 = np.array([1 / 3] + [1 / 18] * 6 + [1 / 36] * 12)


@pytest.mark.parametrize("pressure", [None, (1.0005, 0.9995)])
@pytest.mark.parametrize("nx", [1, 2, 31, 32, 33, 63, 64, 65, 96, 97, 130])
def test_row_ends(orc, nx, pressure):
    m = W.random_mask((4, 7, nx), 0.7, nx)
    m[0, 0, :] = 1  # one row open through both x faces
    g = torch.from_numpy(m).cuda()
    kw = dict(tau=0.8, force=(1e-5, 2e-6, -3e-6), fixed_steps=60, check_every=20)
    o = orc.flow_solve(m, pressure=pressure, **kw)
    vox = np.flatnonzero(m.reshape(-1))
    fo = o["f"].reshape(-1, 19)[vox] - W19
    # two steps past a check as well: the sweep that moves to new references
    for storage, bar in ((lbm.LBM_STORE_FP64, 1e-12), (lbm.LBM_STORE_FP32, 5e-5 * np.abs(fo).max())):
        r = lbm.lbm_flow_solve(g, pressure=pressure, storage=storage, want_u=True, **kw)
        f, flag = lbm.lbm_flow_sample(r.workspace, vox)
        assert flag.all()
        assert np.abs(f - fo).max() <= bar
        w = lbm.lbm_flow_solve(g, pressure=pressure, storage=storage, want_u=True,
                               variant=lbm.LBM_VARIANT_OFF64, **kw)
        assert torch.equal(w.field, r.field)
        u = r.field.cpu().numpy().astype(np.float64)
        assert np.abs(u - o["u"]).max() <= 1e-5 * np.abs(o["u"]).max()
    if pressure is None:
        _, _, us, _ = lbm.lbm_flow_solve_batch([g, g], want_u=True, group_bytes=-1, **kw)
        assert torch.equal(us[1], r.field)


@pytest.mark.parametrize("shape", [(1, 1, 5), (16, 33, 70), (530, 530, 3)])
def test_numbering(orc, shape):
    """The scan that numbers the nodes: one block, some, and more rows (34 x 34 columns of 256)
    than the largest grid has threads, so that a thread takes two."""
    m = W.random_mask(shape, 0.6, 5) if shape[0] > 1 else np.ones(shape, np.uint8)
    kw = dict(tau=0.8, force=(1e-5, 2e-6, -3e-6), fixed_steps=4, check_every=2)
    o = orc.flow_solve(m, **kw)
    nodes = np.flatnonzero(m.reshape(-1))
    vox = nodes[np.random.default_rng(1).integers(0, len(nodes), 20000)]
    fo = o["f"].reshape(-1, 19)[vox] - W19
    r = lbm.lbm_flow_solve(torch.from_numpy(m).cuda(), storage=lbm.LBM_STORE_FP64, **kw)
    f, flag = lbm.lbm_flow_sample(r.workspace, vox)
    assert flag.all()
    assert np.abs(f - fo).max() <= 1e-12


@pytest.mark.parametrize("nx", [2, 31, 32, 33, 63, 64, 65, 96, 97, 130])
def test_row_ends_diffusion(orc, nx):
    """The D3Q19 mass-transport sweep at the same row ends; the bar on the populations is the
    one of the ragged parity cases (binary32 deviations of a field of order 1)."""
    m = W.random_mask((4, 7, nx), 0.8, nx)
    diam = W.hash_field(m.shape, nx, 1.0, 40.0).astype(np.float64) * m
    tg = np.where(m == 1, orc.tau_g(diam, 20.0, 1.0), 1.0)
    kw = dict(d_ref_nm=30.0, voxel_nm=1.5, c_in=0.8, c_out=0.3, fixed_steps=100, check_every=50,
              want_c=True, lattice=lbm.LBM_LATTICE_D3Q19)
    g, d = torch.from_numpy(m).cuda(), torch.from_numpy(diam).cuda()
    r = lbm.lbm_knudsen_solve(g, d, **kw)
    o = orc.diffusion19_solve(m, tg, 0.8, 0.3, fixed_steps=100, check_every=50)
    vox = np.flatnonzero(m.reshape(-1))
    gs, _, flag = lbm.lbm_knudsen_sample(r.workspace, vox)
    assert flag.all()
    assert np.abs(gs - o["g"].reshape(-1, 19)[vox]).max() < 2e-6
    w = lbm.lbm_knudsen_solve(g, d, variant=lbm.LBM_VARIANT_OFF64, **kw)
    assert torch.equal(w.field, r.field)
