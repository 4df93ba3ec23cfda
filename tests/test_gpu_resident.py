"""Resident Knudsen sweeps (many steps in one launch, the lattice held on the chip) against one
launch per step: the same bits, for one to five nodes a thread, partly filled workgroups,
check intervals on both sides of the shortest resident run, and lattices whose workgroups
have more links than the resident sweep takes (it then leaves the steps to plain sweeps)."""
import numpy as np
import pytest
import torch

import paper_1410_1921_amd.workloads as W
from paper_1410_1921_amd import lbm

pytestmark = pytest.mark.gpu

PLAIN = lbm.LBM_VARIANT_EXPLICIT  # an explicit variant is one launch per step

# (nz, ny, nx), pore fraction, steps, check_every
CASES = [((1, 1, 3), 1.0, 60, 25), ((5, 6, 7), 0.7, 120, 50), ((2, 2, 130), 0.8, 55, 20),
         ((16, 17, 33), 0.6, 130, 50), ((40, 41, 42), 0.3, 100, 9), ((40, 41, 42), 0.5, 100, 10),
         ((64, 64, 64), 0.45, 110, 50),      # one node a thread
         ((90, 96, 100), 0.40, 110, 50),     # two
         ((120, 110, 120), 0.36, 110, 50),   # three
         ((128, 128, 128), 0.40, 110, 50),   # four
         ((130, 128, 128), 0.45, 110, 50),   # five
         ((130, 128, 128), 0.60, 60, 50),    # too many nodes
         ((16, 64, 1024), 0.80, 110, 50)]    # long rows: too many links


@pytest.mark.parametrize("shape,p,steps,every", CASES)
def test_resident_equals_plain(shape, p, steps, every):
    seed = sum(shape)
    m = W.blob_mask(shape, p, seed) if p < 1 else np.ones(shape, np.uint8)
    g = torch.from_numpy(m).cuda()
    rng = np.random.default_rng(seed)
    d = torch.from_numpy(3 + 20 * rng.random(shape)).cuda()
    c0 = torch.from_numpy((rng.random(shape) * m).astype(np.float32)).cuda()
    kw = dict(fixed_steps=steps, check_every=every, want_c=True, c_init=c0, voxel_nm=2.0)
    print(shape, p, int(m.sum()), flush=True)
    a = lbm.lbm_knudsen_solve(g, d, variant=PLAIN, **kw)
    b = lbm.lbm_knudsen_solve(g, d, **kw)
    assert torch.equal(a.field, b.field)
    for k in ("Deff_lattice", "residual", "sum_c", "phi_in", "flux_spread"):
        assert a[k] == b[k], k
    nodes = np.flatnonzero(m.reshape(-1))
    vox = nodes[rng.integers(0, len(nodes), 4000)]
    ga, ta, _ = lbm.lbm_knudsen_sample(a.workspace, vox)
    gb, tb, _ = lbm.lbm_knudsen_sample(b.workspace, vox)
    assert np.array_equal(ga, gb) and np.array_equal(ta, tb)
    # the state goes on from either as from the other
    lbm.lbm_knudsen_step(b.workspace, 3)
    kw.update(fixed_steps=every + 12, c_init=None)
    r = lbm.lbm_knudsen_solve(g, d, workspace=b.workspace, resume=True, **kw)
    lbm.lbm_knudsen_step(a.workspace, 3)
    q = lbm.lbm_knudsen_solve(g, d, workspace=a.workspace, resume=True, variant=PLAIN, **kw)
    assert torch.equal(r.field, q.field)
