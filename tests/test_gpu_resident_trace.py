"""What the resident Knudsen sweeps did, from the trace of the solve: they take the steps they
are meant to take, also where workgroups share no links (parts of the pore space that do not
meet) or are many links apart, so that nothing but the packets orders them; and where one gives up a wait,
or the runtime refuses its launch, plain sweeps take its steps.  Fields against one launch per
step, bit for bit."""
import ctypes as C
import threading
import time

import numpy as np
import pytest
import torch

import paper_1410_1921_amd.workloads as W
from paper_1410_1921_amd import lbm

pytestmark = pytest.mark.gpu

PLAIN = lbm.LBM_VARIANT_EXPLICIT  # an explicit variant is one launch per step


class Trace(C.Structure):
    _fields_ = [("wait_ticks", C.c_int64), ("give_up_at", C.c_int32), ("refuse_at", C.c_int32),
                ("resident_steps", C.c_int64), ("launches", C.c_int32), ("gave_up", C.c_int32),
                ("refused", C.c_int32), ("lists", C.c_int32), ("min_steps", C.c_int32),
                ("pad", C.c_int32)]


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
    def solve(*a, wait=20_000_000, give_up_at=0, refuse_at=0, min_steps=8, **kw):
        t, lib = Trace(wait, give_up_at, refuse_at, min_steps=min_steps), lbm.load()
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


def same(a, b, m, seed):
    assert torch.equal(a.field, b.field)
    for n in ("steps", "converged", "Deff_lattice", "residual", "sum_c", "phi_in", "flux_spread"):
        assert a[n] == b[n], n
    nodes = np.flatnonzero(m.reshape(-1))
    vox = nodes[np.random.default_rng(seed).integers(0, len(nodes), 3000)]
    for x, y in zip(lbm.lbm_knudsen_sample(a.workspace, vox), lbm.lbm_knudsen_sample(b.workspace, vox)):
        assert np.array_equal(x, y)


# the launch that fails: the first of the solve (it follows the sweep that enters the first
# frame), a later one, and the last of a solve that ends inside an interval
@pytest.mark.parametrize("how", ["give_up_at", "refuse_at"])
@pytest.mark.parametrize("at", [1, 2, 4])
@pytest.mark.parametrize("shape,p", [((40, 41, 42), 0.5), ((96, 100, 90), 0.40)])
def test_plain_sweeps_take_over(traced, shape, p, at, how):
    m = W.blob_mask(shape, p, sum(shape))
    g, d, c0 = inputs(m, at)
    steps, every = 165, 50
    kw = dict(fixed_steps=steps, check_every=every, want_c=True, c_init=c0, voxel_nm=2.0)
    print(shape, p, how, at, flush=True)
    a = lbm.lbm_knudsen_solve(g, d, variant=PLAIN, **kw)
    b, t = traced(g, d, wait=100_000, **{how: at}, **kw)  # 1 ms: the packets never come
    assert (t.launches, t.gave_up, t.refused) == (at, int(how == "give_up_at"), int(how == "refuse_at"))
    assert t.resident_steps == (at - 1) * (every - 2)
    same(a, b, m, at)
    # on from either, now without a frame to enter before the first resident sweep
    kw.update(fixed_steps=every + 30, c_init=None, resume=True)
    q = lbm.lbm_knudsen_solve(g, d, variant=PLAIN, workspace=a.workspace, **kw)
    r, t = traced(g, d, workspace=b.workspace, wait=100_000, **{how: 1}, **kw)
    assert (t.launches, t.gave_up + t.refused, t.resident_steps) == (1, 1, 0)
    same(q, r, m, at)


def test_converges_at_the_same_step(traced):
    m = W.blob_mask((40, 41, 42), 0.7, 11)
    g, d, _ = inputs(m, 2)
    kw = dict(tol=3e-4, check_every=50, max_steps=20_000, want_c=True, voxel_nm=2.0)
    a = lbm.lbm_knudsen_solve(g, d, variant=PLAIN, **kw)
    assert a["converged"] and 300 < a["steps"]
    b, t = traced(g, d, **kw)
    assert (t.gave_up, t.refused) == (0, 0) and t.resident_steps == a["steps"] // 50 * 48
    same(a, b, m, 3)
    b, t = traced(g, d, wait=100_000, give_up_at=3, **kw)
    assert (t.gave_up, t.refused) == (1, 0) and t.resident_steps == 2 * 48
    same(a, b, m, 3)


def test_beside_other_streams():
    """Solves on streams of their own, from threads of their own, beside one another and beside a
    flow solve that keeps the chip busy: the results of the same solves alone."""
    m = W.blob_mask((96, 100, 90), 0.40, 5)
    cases = [inputs(m, k) for k in range(3)]
    kw = dict(fixed_steps=110, check_every=50, want_c=True, voxel_nm=2.0)

    def knudsen(g, d, c0):
        return [lbm.lbm_knudsen_solve(g, d, c_init=c0, **kw).field for _ in range(6)]

    def flow(g, _d, _c0):
        return [lbm.lbm_flow_solve(g, fixed_steps=300, want_u=True).field for _ in range(4)]

    jobs = [(knudsen, *cases[0]), (knudsen, *cases[1]), (flow, *cases[2])]
    alone = [f(*a) for f, *a in jobs]
    torch.cuda.synchronize()
    out, start = [None] * len(jobs), threading.Barrier(len(jobs))

    def work(k):
        f, *a = jobs[k]
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            start.wait()
            out[k] = f(*a)
            s.synchronize()

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(jobs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for a, b in zip(alone, out):
        for x, y in zip(a, b):
            assert torch.equal(x, y)


@pytest.mark.parametrize("every,first,then", [(8, (0, 0), (0, 0)), (9, (0, 0), (1, 1)), (10, (1, 3), (1, 3))])
def test_no_lists_for_short_intervals(traced, every, first, then):
    """(lists formed, launches) from rest and resumed: an interval from rest has two plain sweeps,
    the first one of a resumed solve only its check."""
    m = W.blob_mask((40, 41, 42), 0.5, 5)
    g, d, c0 = inputs(m, 4)
    kw = dict(fixed_steps=3 * every, check_every=every, voxel_nm=2.0)
    a, t = traced(g, d, c_init=c0, **kw)
    assert (t.lists, t.launches) == first
    _, t = traced(g, d, workspace=a.workspace, resume=True, **kw)
    assert (t.lists, t.launches) == then


@pytest.mark.parametrize("shape,p,every,launches", [((20, 20, 20), 0.5, 9, 0), ((20, 20, 20), 0.5, 50, 2),
                                                    ((128, 128, 128), 0.40, 14, 2),
                                                    ((40, 40, 300), 0.5, 14, 0), ((40, 40, 300), 0.5, 100, 2),
                                                    ((16, 64, 700), 0.6, 100, 0), ((24, 24, 1000), 0.5, 100, 0)])
def test_only_where_it_is_faster(traced, shape, p, every, launches):
    """The rule's clear cases: short intervals of a small lattice, and boxes whose workgroups have
    every neighbour row in another one, are left to plain sweeps."""
    m = W.blob_mask(shape, p, 3)
    g, d, c0 = inputs(m, 1)
    kw = dict(fixed_steps=2 * every, check_every=every, want_c=True, c_init=c0, voxel_nm=2.0)
    a = lbm.lbm_knudsen_solve(g, d, variant=PLAIN, **kw)
    b, t = traced(g, d, min_steps=0, **kw)
    assert (t.launches, t.gave_up) == (launches, 0)
    assert torch.equal(a.field, b.field)


def test_comes_back(traced):
    """After a launch that gave up 32 intervals are left to plain sweeps, after the next one 64; the
    packets and step numbers of the launches given up disturb no later one."""
    m = W.blob_mask((40, 41, 42), 0.5, 5)
    g, d, c0 = inputs(m, 6)
    kw = dict(fixed_steps=300 * 30, check_every=30, want_c=True, c_init=c0, voxel_nm=2.0)
    a = lbm.lbm_knudsen_solve(g, d, variant=PLAIN, **kw)
    b, t = traced(g, d, wait=100_000, give_up_at=2, **kw)
    # intervals 1 and 35 to 300 resident, 2 given up
    assert (t.launches, t.gave_up, t.resident_steps) == (268, 1, 267 * 28)
    same(a, b, m, 1)


def test_many_streams_still_overlap():
    """Eight solves on streams of their own against the same with plain sweeps, which overlap: about
    as long (a launch that kept the other streams' queues off the device took five times that)."""
    m = W.blob_mask((64, 64, 64), 0.40, 5)
    jobs = [inputs(m, k) for k in range(8)]
    kw = dict(fixed_steps=2000, check_every=100, voxel_nm=2.0, n_fluid=int(m.sum()))
    size = lbm.lbm_workspace_size(lbm.LBM_WS_KNUDSEN, m.shape, kw["n_fluid"])
    ws = [lbm.Workspace(size, jobs[0][0].device) for _ in jobs]
    streams = [torch.cuda.Stream() for _ in jobs]
    torch.cuda.synchronize()

    def together(variant):
        def work(k):
            with torch.cuda.stream(streams[k]):
                g, d, c0 = jobs[k]
                lbm.lbm_knudsen_solve(g, d, c_init=c0, workspace=ws[k], variant=variant, **kw)
        best = float("inf")
        for _ in range(4):
            threads = [threading.Thread(target=work, args=(k,)) for k in range(len(jobs))]
            t0 = time.perf_counter()
            for t in threads:
                t.start()
            for t in threads:
                t.join()
            best = min(best, time.perf_counter() - t0)
        return best

    plain = together(PLAIN | lbm.LBM_VARIANT_REMAP)
    auto = together(lbm.LBM_VARIANT_AUTO)
    print(f"plain {1e3 * plain:.1f} ms, auto {1e3 * auto:.1f} ms", flush=True)
    assert auto < 2.5 * plain
