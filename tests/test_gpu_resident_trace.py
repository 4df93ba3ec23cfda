"""What the resident Knudsen sweeps did, from the trace of the solve: they take the steps they
are meant to take, also where workgroups share no links (parts of the pore space that do not
meet) or are many links apart, so that nothing but the packets orders them.  Fields against one
launch per step, bit for bit."""
import ctypes as C

import numpy as np
import pytest
import torch

import paper_1410_1921_amd.workloads as W
from paper_1410_1921_amd import lbm

pytestmark = pytest.mark.gpu

PLAIN = lbm.LBM_VARIANT_EXPLICIT  # an explicit variant is one launch per step


class Trace(C.Structure):
    _fields_ = [("resident_steps", C.c_int64), ("launches", C.c_int32), ("gave_up", C.c_int32),
                ("refused", C.c_int32), ("pad", C.c_int32)]


class Traced:
    """The library with lbm_knudsen_solve filling a trace."""

    def __init__(self, lib, trace):
        fn, self._lib = lib.lbm_knudsen_solve_traced, lib
        fn.argtypes = lib.lbm_knudsen_solve.argtypes + [C.POINTER(Trace)]
        fn.restype = C.c_int32
        self.lbm_knudsen_solve = lambda *a: fn(*a, C.byref(trace))

    def __getattr__(self, name):
        return getattr(self._lib, name)


@pytest.fixture
def traced(monkeypatch):
    def solve(*a, **kw):
        t, lib = Trace(), lbm.load()
        with monkeypatch.context() as m:
            m.setattr(lbm, "load", lambda: Traced(lib, t))
            return lbm.lbm_knudsen_solve(*a, **kw), t
    return solve


def inputs(m, seed):
    rng = np.random.default_rng(seed)
    d = torch.from_numpy(3 + 20 * rng.random(m.shape)).cuda()
    c0 = torch.from_numpy((rng.random(m.shape) * m).astype(np.float32)).cuda()
    return torch.from_numpy(np.ascontiguousarray(m)).cuda(), d, c0


def resident(steps, every):
    """Steps of a solve from rest that resident sweeps take: all of an interval but the one that
    enters a frame and the one that checks, if they are at least 8."""
    n = [min(every, steps - t) - 2 for t in range(0, steps, every)]
    return sum(k for k in n if k >= 8), sum(k >= 8 for k in n)


def islands(shape):
    """The lower half of the planes pore space without a link (every other voxel of every other
    row of every other plane), a solid plane, then a porous part: workgroups without links that
    are done at once beside workgroups that wait for each other."""
    m = np.zeros(shape, np.uint8)
    h = shape[0] // 2
    m[0:h - 1:2, ::2, ::2] = 1
    m[h:-1] = W.blob_mask((shape[0] - h - 1, *shape[1:]), 0.5, 3)
    return m


CASES = [(islands((96, 128, 128)), 60, 12), (islands((97, 130, 65)), 110, 50),
         (np.ones((1, 1024, 40), np.uint8), 70, 20),   # a ring of workgroups
         (W.blob_mask((40, 41, 42), 0.5, 5), 100, 10), (W.blob_mask((40, 41, 42), 0.5, 5), 100, 9),
         (W.blob_mask((128, 128, 128), 0.40, 6), 130, 50)]


@pytest.mark.parametrize("k", range(len(CASES)))
def test_takes_its_steps(traced, k):
    m, steps, every = CASES[k]
    g, d, c0 = inputs(m, k)
    kw = dict(fixed_steps=steps, check_every=every, want_c=True, c_init=c0, voxel_nm=2.0)
    print(m.shape, int(m.sum()), steps, every, flush=True)
    a, ta = traced(g, d, variant=PLAIN, **kw)
    b, tb = traced(g, d, **kw)
    assert (ta.resident_steps, ta.launches) == (0, 0)
    assert (tb.resident_steps, tb.launches, tb.gave_up, tb.refused) == (*resident(steps, every), 0, 0)
    assert torch.equal(a.field, b.field)
    for n in ("Deff_lattice", "residual", "sum_c", "phi_in", "flux_spread"):
        assert a[n] == b[n] or (np.isnan(a[n]) and np.isnan(b[n])), n


@pytest.mark.parametrize("shape,p", [((130, 128, 128), 0.60), ((16, 64, 1024), 0.80)])
def test_leaves_what_does_not_fit(traced, shape, p):
    m = W.blob_mask(shape, p, sum(shape))  # too many nodes; too many links
    g, d, c0 = inputs(m, 1)
    _, t = traced(g, d, fixed_steps=60, check_every=50, c_init=c0, voxel_nm=2.0)
    assert (t.resident_steps, t.launches, t.gave_up, t.refused) == (0, 0, 0, 0)
