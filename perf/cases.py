"""The work this library is timed on, case by case: the stages of the transport pipeline
(characterisation of a reconstruction, flow and Knudsen solves, batches) and the
warm-start network, called as a user's program calls them.

A case is a dict of plain values; `prepare` makes its inputs on the GPU from a seed,
`run` is one pass through the public entry points, `work` what a pass cannot do without,
`exact` the same outputs in 64 bits by plain torch.
"""
import math
import os

import numpy as np
import torch

import paper_1410_1921_amd
from paper_1410_1921_amd import lbm, warmstart
from paper_1410_1921_amd import workloads as W
from paper_1410_1921_amd.unet import C_IN, LEVELS, UNet

WEIGHTS = os.path.join(os.path.dirname(paper_1410_1921_amd.__file__), "weights",
                       "unet_warmstart.npz")
FORCE = 1e-6  # body force of every workload
PRESSURE = (1.0001, 0.9999)
COLLISION = {"bgk": lbm.LBM_COLLIDE_BGK, "mrt": lbm.LBM_COLLIDE_MRT, "trt": lbm.LBM_COLLIDE_TRT}
STORAGE = {"fp32": lbm.LBM_STORE_FP32, "fp64": lbm.LBM_STORE_FP64}
LATTICE = {"d3q7": lbm.LBM_LATTICE_D3Q7, "d3q19": lbm.LBM_LATTICE_D3Q19}
PSD = {"chord13": lbm.LBM_PSD_CHORD13, "mis": lbm.LBM_PSD_MIS}


def _geom(nx, ny, nz, porosity, d_mean, overlap):
    return dict(nx=nx, ny=ny, nz=nz, porosity=porosity, d_mean=d_mean, overlap=overlap)


def listed():
    return [
        # Characterisation (labelling, then the pore-size map), done once per geometry.
        # A small ragged sample with the 13-direction chords: launches and latency.
        dict(name="geometry_small", kind="geometry", psd="chord13",
             **_geom(45, 37, 32, 0.35, 8.0, 0.5)),
        # The 128^3 methane workload's geometry with the inscribed-sphere map.
        dict(name="geometry_128", kind="geometry", psd="mis",
             **_geom(128, 128, 128, 0.40, 12.0, 0.3)),
        # The 512^3 workload's geometry.
        dict(name="geometry_512", kind="geometry", psd="mis",
             **_geom(512, 512, 512, 0.25, 16.0, 0.7)),
        # Flow solves.  The 32^3 workload: a lattice far below the device's width.
        dict(name="flow_32", kind="flow", collision="bgk", storage="fp32", pressure=False,
             steps=1000, **_geom(32, 32, 32, 0.35, 8.0, 0.5)),
        # The 128^3 methane workload's flow: its state fits the Infinity Cache.
        dict(name="flow_128", kind="flow", collision="bgk", storage="fp32", pressure=False,
             steps=500, **_geom(128, 128, 128, 0.40, 12.0, 0.3)),
        # The benchmark's headline lattice: streams from HBM.
        dict(name="flow_512", kind="flow", collision="bgk", storage="fp32", pressure=False,
             steps=100, **_geom(512, 512, 512, 0.25, 16.0, 0.7)),
        # The paper's own setting, MRT between pressure boundaries, on a ragged box.
        dict(name="flow_pressure_mrt", kind="flow", collision="mrt", storage="fp32",
             pressure=True, steps=300, **_geom(150, 101, 86, 0.35, 10.0, 0.5)),
        # Knudsen solves: the 128^3 methane workload (most of the pipeline's time) ...
        dict(name="knudsen_128", kind="knudsen", lattice="d3q7", psd="mis", steps=1000,
             **_geom(128, 128, 128, 0.40, 12.0, 0.3)),
        # ... and the paper's D3Q19 mass-transport lattice on a ragged box.
        dict(name="knudsen19_ragged", kind="knudsen", lattice="d3q19", psd="chord13", steps=300,
             **_geom(100, 117, 84, 0.35, 10.0, 0.5)),
        # A batch of uneven reconstructions (edges 64 to 160), flow and Knudsen together.
        dict(name="batch_12", kind="batch", count=12, steps=300),
        # The warm-start network: inference before a solve, and a training step's
        # forward and backward.
        dict(name="unet_predict_96", kind="predict", **_geom(96, 96, 96, 0.35, 12.0, 0.5)),
        dict(name="unet_train_96", kind="train", **_geom(96, 96, 96, 0.35, 12.0, 0.5)),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["geometry", "flow", "flow", "knudsen", "knudsen", "batch", "predict",
                       "train"])
    if kind == "batch":
        return dict(kind=kind, count=rng.randint(4, 12), steps=rng.choice([100, 200, 300]))
    d_mean = round(rng.uniform(7.0, 16.0), 2)
    mix = (round(rng.uniform(0.25, 0.42), 3), d_mean, round(rng.uniform(0.3, 0.7), 2))
    if kind in ("predict", "train"):
        top = 112 if kind == "predict" else 96  # sizes are multiples of 8 (three poolings)
        nx, ny, nz = (8 * rng.randint(4, top // 8) for _ in range(3))
        while (nx // 8) * (ny // 8) * (nz // 8) % 16:
            nx, ny, nz = (8 * rng.randint(4, top // 8) for _ in range(3))
        return dict(kind=kind, **_geom(nx, ny, nz, *mix))
    if kind == "geometry":
        n = [_log_int(rng, 30, 400) for _ in range(3)]
        return dict(kind=kind, psd=rng.choice(["mis", "chord13"]), **_geom(*n, *mix))
    n = [_log_int(rng, 32, 250) for _ in range(3)]
    steps = rng.choice([100, 200, 300])
    if kind == "flow":
        return dict(kind=kind, collision=rng.choice(["bgk", "bgk", "mrt", "trt"]),
                    storage=rng.choice(["fp32", "fp32", "fp64"]),
                    pressure=rng.random() < 0.3, steps=steps, **_geom(*n, *mix))
    return dict(kind=kind, lattice=rng.choice(["d3q7", "d3q7", "d3q19"]),
                psd=rng.choice(["mis", "chord13"]), steps=steps, **_geom(*n, *mix))


# ------------------------------------------------------------------ inputs
def _pore(c, seed):
    d = c["d_mean"]
    return lbm.lbm_reconstruct((c["nx"], c["ny"], c["nz"]), c["porosity"], d, d / 4.0, 1.0,
                               c["overlap"], 0.5, seed % (1 << 31))[0]


def _noise(shape, seed, scale):
    g = torch.Generator(device="cuda").manual_seed(seed % (1 << 31))
    return scale * (2.0 * torch.rand(shape, generator=g, device="cuda") - 1.0)


def _c_init(pore, seed):
    """A concentration near its final profile, as a warm start gives: the linear ramp
    between the ghost planes, with a perturbation."""
    nx = pore.shape[2]
    ramp = 1.0 - (torch.arange(nx, device="cuda", dtype=torch.float32) + 1.0) / (nx + 1.0)
    c = ramp.expand(pore.shape) + _noise(pore.shape, seed, 0.02)
    return (c * pore).float().contiguous()


def _knudsen_diam(c, pore):
    return lbm.lbm_pore_diameter(pore, PSD[c["psd"]])


def _batch_shapes(c, seed):
    """Lattices with the laws of the batch workload: every edge in turn, drawn otherwise."""
    rng = np.random.default_rng(seed)
    out = []
    for i in range(c["count"]):
        e = (64, 96, 128, 160)[i % 4]
        out.append(_geom(e, e, e, float(rng.uniform(0.2, 0.42)), float(rng.uniform(6.0, 20.0)),
                         float(rng.uniform(0.3, 0.9))))
    return out


def prepare(case, seed):
    c, s = dict(case), {"case": dict(case)}
    kind = c["kind"]
    if kind == "batch":
        geoms = _batch_shapes(c, seed)
        s["pores"] = [_pore(g, seed + i) for i, g in enumerate(geoms)]
        s["diams"] = [lbm.lbm_pore_diameter(p, lbm.LBM_PSD_CHORD13) for p in s["pores"]]
        s["c_inits"] = [_c_init(p, seed + i) for i, p in enumerate(s["pores"])]
        s["n_fluids"] = [lbm.lbm_count(p) for p in s["pores"]]
        shapes = [p.shape for p in s["pores"]]
        dev = s["pores"][0].device
        s["ws_flow"] = lbm.Workspace(lbm.lbm_flow_batch_workspace(shapes, s["n_fluids"]), dev)
        s["ws_kn"] = lbm.Workspace(lbm.lbm_knudsen_batch_workspace(shapes, s["n_fluids"]), dev)
        return s
    s["pore"] = pore = _pore(c, seed)
    if kind == "geometry":
        return s
    if kind in ("flow", "knudsen"):
        s["n_fluid"] = lbm.lbm_count(pore)
        if kind == "flow":
            ws = lbm.LBM_WS_FLOW_FP64 if c["storage"] == "fp64" else lbm.LBM_WS_FLOW
        else:
            ws = lbm.LBM_WS_KNUDSEN_D3Q19 if c["lattice"] == "d3q19" else lbm.LBM_WS_KNUDSEN
            s["diam"] = _knudsen_diam(c, pore)
            s["c_init"] = _c_init(pore, seed)
        s["ws"] = lbm.Workspace(lbm.lbm_workspace_size(ws, pore.shape, s["n_fluid"]), pore.device)
        return s
    s["diam"] = lbm.lbm_pore_diameter(pore, lbm.LBM_PSD_MIS)
    s["net"] = UNet.load(WEIGHTS)
    if kind == "train":
        nv = pore.numel()
        s["x0"] = warmstart.network_input(pore, s["diam"])
        fields = _noise((5, nv), seed, 1.0)
        fields[4] = _c_init(pore, seed).reshape(-1)
        s["target"] = (fields * pore.reshape(1, -1)).contiguous()
        s["wt"] = torch.ones(5, dtype=torch.float32, device="cuda")
        s["mask"] = pore.reshape(-1)
        s["n_mask"] = float(lbm.lbm_count(pore))
    return s


# ------------------------------------------------------------------ one pass
_KN = dict(tau_ref=1.0, d_ref_nm=60.0, voxel_nm=2.0, c_in=1.0, c_out=0.0, T=400.0,
           check_every=100)
_FLOW = dict(tau=0.8, check_every=100, voxel_nm=2.0)


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "geometry":
        label, transport, st = lbm.lbm_label(s["pore"])
        diam = lbm.lbm_pore_diameter(s["pore"], PSD[c["psd"]])
        return {"label": label, "transport": transport, "diam": diam, "n_pore": st["n_pore"],
                "n_transport": st["n_transport"], "n_components": st["n_components"]}
    if kind == "flow":
        r = lbm.lbm_flow_solve(s["pore"], force=(0.0 if c["pressure"] else FORCE, 0.0, 0.0),
                               pressure=PRESSURE if c["pressure"] else None,
                               collision=COLLISION[c["collision"]], storage=STORAGE[c["storage"]],
                               fixed_steps=c["steps"], want_u=True, n_fluid=s["n_fluid"],
                               workspace=s["ws"], **_FLOW)
        return {"u": r.field, "k": r["k_lattice"], "residual": r["residual"]}
    if kind == "knudsen":
        r = lbm.lbm_knudsen_solve(s["pore"], s["diam"], fixed_steps=c["steps"], want_c=True,
                                  c_init=s["c_init"], n_fluid=s["n_fluid"], workspace=s["ws"],
                                  lattice=LATTICE[c["lattice"]], **_KN)
        return {"c": r.field, "deff": r["Deff_lattice"], "residual": r["residual"]}
    if kind == "batch":
        # group budgets as the autotuner ends up with on long solves
        _, fr, us, _ = lbm.lbm_flow_solve_batch(
            s["pores"], force=(FORCE, 0.0, 0.0), fixed_steps=c["steps"], want_u=True,
            n_fluids=s["n_fluids"], workspace=s["ws_flow"], group_bytes=256_000_000, **_FLOW)
        _, kr, cs, _ = lbm.lbm_knudsen_solve_batch(
            s["pores"], s["diams"], fixed_steps=c["steps"], want_c=True, c_inits=s["c_inits"],
            n_fluids=s["n_fluids"], workspace=s["ws_kn"], group_bytes=256_000_000, **_KN)
        return {"u": us, "c": cs, "k": np.array([r["k_lattice"] for r in fr], np.float32),
                "deff": np.array([r["Deff_lattice"] for r in kr], np.float32)}
    if kind == "predict":
        u, conc = warmstart.predict(s["net"], s["pore"], s["diam"])
        return {"u": u, "c": conc}
    loss = s["net"].loss_and_grad(tuple(s["pore"].shape), s["x0"], s["target"], s["mask"], s["wt"],
                                  s["n_mask"])
    return {"loss": loss, "grad": s["net"].g}


# ------------------------------------------------------------------ what a pass needs
def _conv_flops(nv):
    net, f = [("enc0a", C_IN, LEVELS[0]), ("enc0b", LEVELS[0], LEVELS[0])], 0.0
    for i in range(1, len(LEVELS)):
        net += [(f"enc{i}a", LEVELS[i - 1], LEVELS[i]), (f"enc{i}b", LEVELS[i], LEVELS[i])]
    for i in range(len(LEVELS) - 2, -1, -1):
        net += [(f"dec{i}a", LEVELS[i] + LEVELS[i + 1], LEVELS[i]),
                (f"dec{i}b", LEVELS[i], LEVELS[i])]
    for name, ci, co in net:
        f += 2.0 * 27 * ci * co * (nv / 8 ** int(name[3]))
    return f


def work(case):
    c = case
    if c["kind"] == "batch":
        nv = [(64, 96, 128, 160)[i % 4] ** 3 for i in range(c["count"])]
        nf = 0.31 * sum(nv)
        return {"bytes": nf * c["steps"] * (152.0 + 60.0) + sum(nv) * (2.0 + 12.0 + 12.0),
                "flops": nf * c["steps"] * (300.0 + 40.0)}
    nv = float(c["nx"] * c["ny"] * c["nz"])
    nf = c["porosity"] * nv
    if c["kind"] == "geometry":
        return {"bytes": nv * (1 + 4 + 1 + 1 + 8), "flops": 0.0}
    if c["kind"] == "flow":
        return {"bytes": nf * c["steps"] * 38 * (8 if c["storage"] == "fp64" else 4) + 13 * nv,
                "flops": nf * c["steps"] * 300.0}
    if c["kind"] == "knudsen":
        q = 7 if c["lattice"] == "d3q7" else 19
        return {"bytes": nf * c["steps"] * (8.0 * q + 4.0) + nv * 17.0,
                "flops": nf * c["steps"] * 6.0 * q}
    params = 4.0 * 1_460_000
    if c["kind"] == "predict":
        return {"bytes": nv * (1 + 8 + 20) + params / 2, "flops": _conv_flops(nv)}
    return {"bytes": nv * (2.0 * C_IN + 20 + 1) + 1.5 * params, "flops": 3.0 * _conv_flops(nv)}


# ------------------------------------------------------------------ the same in 64 bits
_E19 = [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1),
        (1, 1, 0), (-1, 1, 0), (1, -1, 0), (-1, -1, 0), (1, 0, 1), (-1, 0, 1), (1, 0, -1),
        (-1, 0, -1), (0, 1, 1), (0, -1, 1), (0, 1, -1), (0, -1, -1)]
_W19 = [1 / 3] + [1 / 18] * 6 + [1 / 36] * 12


class _Sparse:
    """Fluid nodes of a mask and, per velocity, the node a population is pulled from: its
    index, -1 beyond a solid link; beyond an x face, `face` marks the row's node there."""

    def __init__(self, pore, vel, open_x):
        nz, ny, nx = pore.shape
        ids = torch.full(pore.shape, -1, dtype=torch.int64, device=pore.device)
        z, y, x = torch.nonzero(pore, as_tuple=True)
        self.x, self.n = x, x.numel()
        ids[z, y, x] = torch.arange(self.n, device=pore.device)
        self.vox = (z * ny + y) * nx + x
        self.src, self.face = [], []
        for ex, ey, ez in vel:
            xs = x - ex
            out = (xs < 0) | (xs >= nx)
            xs = torch.where(out, x, xs) if open_x else xs % nx
            j = ids[(z - ez) % nz, (y - ey) % ny, xs]
            self.src.append(j)
            self.face.append(out if open_x else None)

    def dense(self, vals, shape):
        out = torch.zeros((len(vals), shape[0] * shape[1] * shape[2]), dtype=torch.float64,
                          device=self.vox.device)
        for k, v in enumerate(vals):
            out[k][self.vox] = v
        return out


def _opp(vel):
    return [vel.index((-a, -b, -c)) for a, b, c in vel]


def _exact_flow(pore, steps, tau, force, pressure, collision, nc=100):
    """BGK (compressible equilibrium, Guo force) or, for MRT and TRT alike, two relaxation
    rates towards the incompressible equilibrium, in offsets f - w."""
    sp = _Sparse(pore, _E19, pressure is not None)
    opp, q = _opp(_E19), 19
    F = force
    f = [torch.zeros(sp.n, dtype=torch.float64, device=pore.device) for _ in range(q)]
    s_nu = 1.0 / tau
    s_q = s_nu if collision == "bgk" else 8.0 * (2.0 * tau - 1.0) / (8.0 * tau - 1.0)
    nx = pore.shape[2]
    u = [torch.zeros_like(f[0]) for _ in range(3)]
    snap, resid = u, math.inf
    for t in range(1, steps + 1):
        if pressure is not None:
            # ghost populations of the face nodes (non-equilibrium extrapolation)
            dr = sum(f)
            ub = [sum(e[a] * f[i] for i, e in enumerate(_E19) if e[a]) / (1.0 + dr)
                  for a in range(3)]
            uu = 1.5 * sum(v * v for v in ub)
        g = []
        for i, e in enumerate(_E19):
            if i == 0:
                g.append(f[0])
                continue
            j = sp.src[i]
            jj = j.clamp(min=0)
            v = f[i][jj]
            if pressure is not None and e[0]:
                eu = sum(e[a] * ub[a] for a in range(3) if e[a])
                jump = (pressure[0] if e[0] == 1 else pressure[1]) - 1.0 - dr
                gh = f[i] + _W19[i] * jump * (1.0 + 3.0 * eu + 4.5 * eu * eu - uu)
                v = torch.where(sp.face[i], gh[jj], v)
            g.append(torch.where(j >= 0, v, f[opp[i]]))
        dr = sum(g)
        rho = 1.0 + dr
        m = [sum(e[a] * g[i] for i, e in enumerate(_E19) if e[a]) + 0.5 * F[a] for a in range(3)]
        u = [v / rho for v in m]
        uF = sum(u[a] * F[a] for a in range(3))
        f = [None] * q
        if collision == "bgk":
            uu = 1.5 * sum(v * v for v in u)
            for i, e in enumerate(_E19):
                eu = sum(e[a] * u[a] for a in range(3) if e[a]) if i else 0.0 * dr
                eF = sum(e[a] * F[a] for a in range(3))
                feq = _W19[i] * (dr + rho * (3.0 * eu + 4.5 * eu * eu - uu))
                src = (1.0 - 0.5 * s_nu) * _W19[i] * (3.0 * (eF - uF) + 9.0 * eu * eF)
                f[i] = g[i] - s_nu * (g[i] - feq) + src
        else:
            jj = 1.5 * sum(v * v for v in m)
            f[0] = g[0] - s_nu * (g[0] - _W19[0] * (dr - jj)) \
                - (1.0 - 0.5 * s_nu) * _W19[0] * 3.0 * uF
            for i in range(1, q):
                k, e, w = opp[i], _E19[i], _W19[i]
                if k < i:
                    continue
                ej = sum(e[a] * m[a] for a in range(3) if e[a])
                eu = sum(e[a] * u[a] for a in range(3) if e[a])
                eF = sum(e[a] * F[a] for a in range(3))
                even = 0.5 * (g[i] + g[k]) - w * (dr + 4.5 * ej * ej - jj)
                odd = 0.5 * (g[i] - g[k]) - 3.0 * w * ej
                de = (1.0 - 0.5 * s_nu) * w * (9.0 * eu * eF - 3.0 * uF) - s_nu * even
                dd = (1.0 - 0.5 * s_q) * 3.0 * w * eF - s_q * odd
                f[i], f[k] = g[i] + de + dd, g[k] + de - dd
        if t % nc == 0 or t == steps:
            d2 = float(sum(((a - b) ** 2).sum() for a, b in zip(u, snap)))
            u2 = float(sum((a * a).sum() for a in u))
            if t % nc == 0:
                resid = math.sqrt(d2) / (nc * math.sqrt(u2))
            snap = [a.float().double() for a in u]
    drive = F[0] + (0.0 if pressure is None else (pressure[0] - pressure[1]) / (3.0 * (nx + 1)))
    k = (tau - 0.5) / 3.0 * float(m[0].sum()) / pore.numel() / drive
    return sp.dense(u, pore.shape).reshape((3,) + tuple(pore.shape)), k, resid


def _exact_knudsen(pore, diam, c_init, steps, lattice, nc=100):
    d3q7 = lattice == "d3q7"
    vel = _E19[:7] if d3q7 else _E19
    w = [0.25] + [0.125] * 6 if d3q7 else _W19
    sp, opp = _Sparse(pore, vel, True), _opp(vel)
    nz, ny, nx = pore.shape
    d_ref = _KN["d_ref_nm"] / _KN["voxel_nm"]
    om = 1.0 / (diam.reshape(-1)[sp.vox] / d_ref * (_KN["tau_ref"] - 0.5) + 0.5)
    conc = c_init.reshape(-1)[sp.vox].double()
    g = [wi * conc for wi in w]
    snap, resid = conc, math.inf
    for t in range(1, steps + 1):
        p = [g[0]]
        for i in range(1, len(vel)):
            j = sp.src[i]
            v = g[i][j.clamp(min=0)]
            if vel[i][0]:  # ghost planes at the faces (the row's own voxel stands in: any)
                cg = _KN["c_in"] if vel[i][0] == 1 else _KN["c_out"]
                v = torch.where(j >= 0, v, g[opp[i]])
                v = torch.where(sp.face[i], torch.full_like(v, w[i] * cg), v)
            else:
                v = torch.where(j >= 0, v, g[opp[i]])
            p.append(v)
        conc = sum(p)
        g = [a - om * (a - wi * conc) for a, wi in zip(p, w)]
        if t % nc == 0:
            resid = math.sqrt(float(((conc - snap) ** 2).sum())) / \
                (nc * math.sqrt(float((conc * conc).sum())))
            snap = conc.float().double()
    last = sp.x == nx - 1
    phi = sum(float((g[i][last] - w[i] * _KN["c_out"]).sum())
              for i in range(len(vel)) if vel[i][0] == 1)
    deff = phi / (ny * nz) * (nx + 1) / (_KN["c_in"] - _KN["c_out"])
    return sp.dense([conc], pore.shape).reshape(pore.shape), deff, resid


def _exact_mis(pore):
    """2 sqrt(max squared distance of a covering ball) - 1, by brute force."""
    inf = 1 << 28
    d = torch.where(pore > 0, inf, 0).to(torch.int32)
    for axis in range(3):
        n = d.shape[axis]
        out = d.clone()
        for r in range(1, n):
            if axis and r * r >= int(out[out < inf].max() if (out < inf).any() else inf):
                break
            a, b = out.narrow(axis, r, n - r), d.narrow(axis, 0, n - r)
            torch.minimum(a, b + r * r, out=a)
            a, b = out.narrow(axis, 0, n - r), d.narrow(axis, r, n - r)
            torch.minimum(a, b + r * r, out=a)
        d = out
    best = torch.zeros_like(d)
    rmax = int(math.isqrt(int(d.max())))
    nz, ny, nx = d.shape
    for dz in range(-rmax, rmax + 1):
        for dy in range(-rmax, rmax + 1):
            for dx in range(-rmax, rmax + 1):
                d2 = dz * dz + dy * dy + dx * dx
                if d2 >= int(rmax + 1) ** 2 or abs(dz) >= nz or abs(dy) >= ny or abs(dx) >= nx:
                    continue
                dst, src = [], []
                for o, n in ((dz, nz), (dy, ny), (dx, nx)):
                    dst.append(slice(max(0, -o), n - max(0, o)))
                    src.append(slice(max(0, o), n - max(0, -o)))
                e = d[tuple(src)]
                b = best[tuple(dst)]
                torch.maximum(b, torch.where(e > d2, e, 0), out=b)
    return torch.where(pore > 0, 2.0 * best.double().sqrt() - 1.0, 0.0)


def _exact_chord(pore):
    p = torch.nn.functional.pad(pore.double(), (1, 1, 1, 1, 1, 1))
    sums = [torch.zeros_like(p) for _ in range(3)]
    for dz in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                m = abs(dx) + abs(dy) + abs(dz)
                if (dz, dy, dx) <= (0, 0, 0) or m == 0:
                    continue
                run = p.clone()
                for sgn in (1, -1):  # pore voxels in a row beyond p on either side
                    ahead = p.clone()
                    while True:
                        ahead = torch.roll(ahead, (sgn * dz, sgn * dy, sgn * dx), (0, 1, 2)) * p
                        if not bool(ahead.any()):
                            break
                        run += ahead
                sums[m - 1] += run
    d = (sums[0] + math.sqrt(2.0) * sums[1] + math.sqrt(3.0) * sums[2]) / 13.0
    return (d * p)[1:-1, 1:-1, 1:-1].contiguous()


def _net64(s):
    """The network's parameters (the bf16 weights the layers use) as 64-bit leaves."""
    net = s["net"]
    P = {}
    for key, (o, k) in net.off.items():
        src = net.pb if key.endswith(".w") and not key.startswith("head") else net.p
        P[key] = src[o:o + k].double().clone().requires_grad_(True)
    return P


def _forward64(P, x, shape):
    """x: [nz, ny, nx, c]."""
    def conv(name, h, ci, co):
        w = P[name + ".w"].reshape(27, co, ci)
        nz, ny, nx = h.shape[:3]
        hp = torch.nn.functional.pad(h, (0, 0, 1, 1, 1, 1, 1, 1))
        y = P[name + ".b"].expand(nz * ny * nx, co)
        for t in range(27):
            z0, y0, x0 = t // 9, (t // 3) % 3, t % 3
            y = y + hp[z0:z0 + nz, y0:y0 + ny, x0:x0 + nx].reshape(-1, ci) @ w[t].t()
        return torch.relu(y).reshape(nz, ny, nx, co)

    def pool(h):
        nz, ny, nx, ch = h.shape
        return h.reshape(nz // 2, 2, ny // 2, 2, nx // 2, 2, ch).mean((1, 3, 5))

    def up(h):
        for a in range(3):
            h = h.repeat_interleave(2, a)
        return h

    L, skips, h = LEVELS, [], x
    for i in range(len(L)):
        h = conv(f"enc{i}a", h, C_IN if i == 0 else L[i - 1], L[i])
        h = conv(f"enc{i}b", h, L[i], L[i])
        if i < len(L) - 1:
            skips.append(h)
            h = pool(h)
    for i in range(len(L) - 2, -1, -1):
        h = torch.cat([skips[i], up(h)], 3)
        h = conv(f"dec{i}a", h, L[i] + L[i + 1], L[i])
        h = conv(f"dec{i}b", h, L[i], L[i])
    wh = P["head.w"].reshape(-1, L[0])
    return (h.reshape(-1, L[0]) @ wh.t() + P["head.b"]).t()


def exact(case, seed):
    c = dict(case)
    kind = c["kind"]
    nv = 0 if kind == "batch" else c["nx"] * c["ny"] * c["nz"]
    if kind == "geometry":
        if nv > (3_000_000 if c["psd"] == "mis" else 20_000_000):
            return None
        pore = _pore(c, seed)
        return {"diam": _exact_mis(pore) if c["psd"] == "mis" else _exact_chord(pore)}
    s = prepare(case, seed)
    if kind == "flow":
        u, k, resid = _exact_flow(s["pore"], c["steps"], _FLOW["tau"],
                                  (0.0 if c["pressure"] else FORCE, 0.0, 0.0),
                                  PRESSURE if c["pressure"] else None, c["collision"])
        return {"u": u, "k": k, "residual": resid}
    if kind == "knudsen":
        conc, deff, resid = _exact_knudsen(s["pore"], s["diam"], s["c_init"], c["steps"],
                                           c["lattice"])
        return {"c": conc, "deff": deff, "residual": resid}
    if kind == "batch":
        us, cs, ks, ds = [], [], [], []
        for p, d, ci in zip(s["pores"], s["diams"], s["c_inits"]):
            u, k, _ = _exact_flow(p, c["steps"], _FLOW["tau"], (FORCE, 0.0, 0.0), None, "bgk")
            conc, deff, _ = _exact_knudsen(p, d, ci, c["steps"], "d3q7")
            us, cs, ks, ds = us + [u], cs + [conc], ks + [k], ds + [deff]
        return {"u": us, "c": cs, "k": np.array(ks), "deff": np.array(ds)}
    shape = tuple(s["pore"].shape)
    P = _net64(s)
    if kind == "predict":
        with torch.no_grad():
            x = torch.zeros(shape + (C_IN,), dtype=torch.float64, device="cuda")
            x[..., 0] = s["pore"]
            x[..., 1] = s["diam"] / warmstart.D_SCALE
            out = _forward64(P, x, shape)
            scale = torch.tensor([warmstart.U_SCALE] * 3 + [warmstart.R_SCALE, 1.0],
                                 dtype=torch.float64, device="cuda")
            out = out * scale[:, None] * s["pore"].reshape(1, -1)
        return {"u": out[:4].reshape((4,) + shape), "c": out[4].reshape(shape)}
    out = _forward64(P, s["x0"].double().reshape(shape + (C_IN,)), shape)
    err = (out - s["target"].double()) ** 2 * s["mask"].double()
    loss = (err.sum(1) * s["wt"].double()).sum() / s["n_mask"]
    loss.backward()
    net = s["net"]
    grad = torch.zeros(net.n_params, dtype=torch.float64, device="cuda")
    for key, (o, k) in net.off.items():
        grad[o:o + k] = P[key].grad.reshape(-1)
    return {"loss": float(loss), "grad": grad}
