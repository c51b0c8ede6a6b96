"""Timing cases of the framework's public entry points.

Each case is one call (or the short sequence of calls) a user's program makes on a
prepared simulation: a run of time steps from an initial field to the field read back, a
run with FP64 balances or region masses sampled along it, a steady-state solve, a batch of
tortuosities, a gradient, a signed distance.  Geometries are synthetic porous media drawn
from the seed: "soil" (a smooth random field thresholded at porosity 0.3), "packing" (the
pores between overlapping spheres of radius 4 to 8) and "foam" (the solid around
overlapping pores of radius 10 to 30).

  listed()             the standing cases
  draw(rng)            one more case of the same ranges
  prepare(case, seed)  geometry, bound simulation and input fields on the GPU
  run(state)           one pass; returns its outputs
  work(case)           bytes and operations a pass cannot do without
  exact(case, seed)    the outputs in FP64 from plain torch (None where not available)
"""
import math

import numpy as np
import torch

from paper_2304_11165_amd import rd

# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------

# species set-ups: diffusion coefficients, reactions (from, to, rate), Robin uptake per
# species, Dirichlet values (species, face) -> value, time step
MODELS = {
    # one species entering from the x = 0 face
    "inlet": dict(D=[1.0], reactions=[], robin={}, dirichlet={(0, 0): 1.0}, dt=0.1),
    # two species, A -> B, uptake of B at the walls, A held on x = 0
    "soil": dict(D=[1.0, 0.4], reactions=[(0, 1, 0.01)], robin={1: 0.05}, dirichlet={(0, 0): 1.0}, dt=0.1),
    # diffusion with first-order decay
    "decay": dict(D=[0.8], reactions=[(0, -1, 0.02)], robin={}, dirichlet={(0, 0): 1.0}, dt=0.1),
    # closed box (bleaching and recovery)
    "closed": dict(D=[1.0], reactions=[], robin={}, dirichlet={}, dt=0.1),
}
POROSITY = {"soil": 0.3, "packing": 0.5, "foam": 0.85}
ELEM = {"fp32": 4, "bf16": 2, "fp16": 2}


def listed():
    return [
        # a small packing, one species: the shortest run, a few microseconds per step
        dict(name="step_packing64_fp32", kind="step", medium="packing", nz=64, ny=64, nx=64, model="inlet",
             storage="fp32", layout="blocks", kernel="column", edge=8, sround=False, steps=128),
        # the soil volume at full size, FP32 with unbiased rounding: the production run
        dict(name="step_soil512_fp32", kind="step", medium="soil", nz=512, ny=512, nx=512, model="soil",
             storage="fp32", layout="compact", kernel="column", edge=8, sround=True, steps=64),
        # a ragged crop in BF16 storage (half the field bytes)
        dict(name="step_soil_ragged_bf16", kind="step", medium="soil", nz=283, ny=311, nx=257, model="soil",
             storage="bf16", layout="blocks", kernel="column", edge=8, sround=True, steps=64),
        # diffusion with decay in FP16 storage, round to nearest
        dict(name="step_packing_fp16", kind="step", medium="packing", nz=192, ny=192, nx=192, model="decay",
             storage="fp16", layout="blocks", kernel="column_xch", edge=8, sround=False, steps=64),
        # diffusion coefficient varying in space
        dict(name="dphi_soil320_fp32", kind="dphi", medium="soil", nz=320, ny=320, nx=320, model="soil",
             storage="fp32", layout="blocks", kernel="column_xch", edge=8, sround=False, steps=64),
        # mass balance of both species sampled during a run
        dict(name="monitor_soil256_fp32", kind="monitor", medium="soil", nz=256, ny=256, nx=256, model="soil",
             storage="fp32", layout="blocks", kernel="column", edge=8, sround=False, steps=10, samples=6),
        # simulated bleaching: mass in a box sampled during the recovery
        dict(name="frap_packing160_fp32", kind="frap", medium="packing", nz=160, ny=160, nx=160, model="closed",
             storage="fp32", layout="blocks", kernel="column", edge=8, sround=False, steps=10, samples=16),
        # tortuosity of one ceramic-foam volume
        dict(name="steady_foam208_fp32", kind="steady", medium="foam", nz=208, ny=208, nx=208, storage="fp32",
             edge=8, axis=0),
        # tortuosities of a set of packings in one batch
        dict(name="batch_tau16_fp32", kind="batch", medium="packing", count=16, nmin=48, nmax=144, storage="fp32",
             edge=8, axis=0),
        # forward run and gradient in D and k through autograd
        dict(name="adjoint_decay128_fp32", kind="adjoint", medium="packing", nz=128, ny=128, nx=128, model="decay",
             storage="fp32", edge=8, steps=100, every=20),
        # gradient with respect to the diffusivity of every voxel
        dict(name="adjoint_factor160_fp32", kind="factor", medium="packing", nz=160, ny=160, nx=160, model="decay",
             storage="fp32", edge=8, steps=60, every=15),
        # signed distance of a segmented image
        dict(name="sdf_soil_ragged", kind="sdf", medium="soil", nz=365, ny=411, nx=320),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _shape(rng, lo, hi):
    n = _log_int(rng, lo, hi)
    return {k: max(lo, min(hi, int(round(n * rng.uniform(0.75, 1.25))))) for k in ("nz", "ny", "nx")}


def _box(case):
    return [case["nz"], case["ny"], case["nx"]]


def draw(rng):
    kind = rng.choice(["step", "step", "step", "dphi", "monitor", "frap", "steady", "batch", "adjoint", "factor",
                       "sdf", "sdf"])
    storage = rng.choice(["fp32", "fp32", "bf16", "fp16"])
    edge = rng.choice([8, 8, 8, 4])
    layout, kernel = "blocks", rng.choice(["column", "column_xch"])
    if kind == "step" and edge == 8 and rng.random() < 0.4:
        layout = "compact"
    c = dict(kind=kind, storage=storage, edge=edge, layout=layout, kernel=kernel)
    if kind == "step":
        c.update(medium=rng.choice(["soil", "packing"]), **_shape(rng, 24, 400),
                 model=rng.choice(["inlet", "soil", "decay"]), sround=storage == "bf16" or rng.random() < 0.5,
                 steps=rng.randint(20, 64))
    elif kind == "dphi":
        c.update(medium=rng.choice(["soil", "packing"]), **_shape(rng, 32, 320),
                 model=rng.choice(["inlet", "soil", "decay"]), sround=storage == "bf16", steps=rng.randint(10, 48))
        c.update(edge=8)
    elif kind == "monitor":
        c.update(medium="soil", **_shape(rng, 32, 256), model=rng.choice(["inlet", "soil"]), sround=storage == "bf16",
                 steps=rng.randint(2, 12), samples=rng.randint(2, 6))
    elif kind == "frap":
        c.update(medium="packing", **_shape(rng, 32, 224), model="closed", sround=storage == "bf16",
                 steps=rng.randint(4, 16), samples=rng.randint(4, 16))
    elif kind == "steady":
        c = dict(kind=kind, medium=rng.choice(["foam", "packing"]), **_shape(rng, 32, 208), storage="fp32",
                 edge=8, axis=rng.randrange(3))
    elif kind == "batch":
        lo = rng.randint(24, 64)
        c = dict(kind=kind, medium="packing", count=rng.randint(2, 16), nmin=lo, nmax=rng.randint(lo, 144),
                 storage="fp32", edge=8, axis=rng.randrange(3))
    elif kind in ("adjoint", "factor"):
        c = dict(kind=kind, medium="packing", **_shape(rng, 24, 144), model="decay", storage="fp32",
                 edge=edge if kind == "adjoint" else 8, steps=rng.randint(10, 80), every=rng.randint(4, 20))
    else:
        c = dict(kind="sdf", medium=rng.choice(["soil", "packing", "foam"]), **_shape(rng, 24, 360))
    return c


# ---------------------------------------------------------------------------
# synthetic media (seeded, on the GPU; integer or elementwise arithmetic only, so the same
# seed gives the same voxels everywhere)
# ---------------------------------------------------------------------------

def _gen(seed, k=0):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + k) % (1 << 62))
    return g


def _smooth_noise(shape, seed):
    # white noise of small integers under three box filters of width 17 per axis (close to a
    # Gaussian of standard deviation 8.5); exact in float64
    f = torch.randint(0, 256, shape, generator=_gen(seed), device="cuda", dtype=torch.int32).to(torch.float64)
    for d in range(3):
        for _ in range(3):
            s = f
            for sh in (1, 2, 4, 8):
                s = s + torch.roll(s, sh, d)
            f = s + torch.roll(f, 16, d)
    return f


def _threshold(f, q):
    v = f.reshape(-1)
    v = v[:: max(1, v.numel() // (1 << 20))].sort().values
    return v[min(v.numel() - 1, int(q * v.numel()))]


def _balls(shape, fraction, rmin, rmax, seed):
    # union of balls with Poisson centres covering `fraction` of the volume on average
    nz, ny, nx = shape
    rng = np.random.default_rng(int(seed))
    er3 = (rmax ** 4 - rmin ** 4) / (4.0 * (rmax - rmin))
    lam = -math.log(1.0 - fraction) / (4.0 / 3.0 * math.pi * er3)
    ext = np.array([nz, ny, nx], dtype=np.float64) + 2 * rmax
    n = int(rng.poisson(lam * float(np.prod(ext))))
    cen = torch.as_tensor(rng.uniform(0.0, 1.0, size=(n, 3)) * ext - rmax, device="cuda")
    rad = torch.as_tensor(rng.uniform(rmin, rmax, size=n), device="cuda")
    out = torch.zeros(nz * ny * nx, dtype=torch.bool, device="cuda")
    w = 2 * int(math.ceil(rmax)) + 2
    o = torch.arange(w, device="cuda")
    off = torch.stack(torch.meshgrid(o, o, o, indexing="ij"), -1).reshape(-1, 3)
    lim = torch.tensor([nz, ny, nx], device="cuda")
    chunk = max(1, (1 << 24) // off.shape[0])
    for i in range(0, n, chunk):
        c, r = cen[i:i + chunk], rad[i:i + chunk]
        p = torch.floor(c - r[:, None]).to(torch.int64)[:, None, :] + off[None]
        ok = ((p >= 0) & (p < lim)).all(-1) & (((p - c[:, None, :]) ** 2).sum(-1) <= (r * r)[:, None])
        p = p[ok]
        out[(p[:, 0] * ny + p[:, 1]) * nx + p[:, 2]] = True
    return out.reshape(nz, ny, nx)


def _image(medium, shape, seed, porosity=None):
    if medium == "soil":
        f = _smooth_noise(tuple(shape), seed)
        return (f < _threshold(f, POROSITY["soil"])).to(torch.uint8)
    if medium == "packing":
        return (~_balls(shape, 1.0 - (porosity or POROSITY["packing"]), 4.0, 8.0, seed)).to(torch.uint8)
    return (~_balls(shape, 1.0 - POROSITY["foam"], 10.0, 30.0, seed)).to(torch.uint8)


def _fields(case, img, seed):
    # concentration falling off from the inlet with some scatter; later species start lower
    nz, ny, nx = img.shape
    x = torch.arange(nx, device="cuda", dtype=torch.float32) / nx
    out = []
    for s in range(len(MODELS[case["model"]]["D"])):
        u = torch.rand((nz, ny, nx), generator=_gen(seed, 10 + s), device="cuda")
        out.append((1.0 - x) * (0.9 + 0.1 * u) * (0.3 ** s) * img)
    return out


def _factor(shape, seed):
    # smooth diffusivity factor between 0.1 and 1
    f = _smooth_noise(tuple(shape), seed + 77)
    lo, hi = _threshold(f, 0.02), _threshold(f, 0.98)
    return (0.1 + 0.9 * torch.sigmoid(8.0 * (f - lo) / (hi - lo + 1.0) - 4.0)).to(torch.float32)


def _region(shape):
    nz, ny, nx = shape
    return [nx // 2 - nx // 8, nx // 2 + nx // 8, ny // 2 - ny // 8, ny // 2 + ny // 8,
            nz // 2 - nz // 8, nz // 2 + nz // 8]


def _bleached(img):
    c = img.to(torch.float32)
    x0, x1, y0, y1, z0, z1 = _region(img.shape)
    c[z0:z1, y0:y1, x0:x1] = 0.0
    return c


def _batch_members(case):
    n = case["count"]
    return [(case["nmin"] + (case["nmax"] - case["nmin"]) * i // max(1, n - 1), 0.35 + 0.05 * (i % 7))
            for i in range(n)]


# ---------------------------------------------------------------------------
# prepare / run
# ---------------------------------------------------------------------------

def _model(sim, m):
    for d in m["D"]:
        sim.add_species(d)
    for r in m["reactions"]:
        sim.add_reaction(*r)
    for s, k in m["robin"].items():
        sim.set_robin(s, k)
    for (s, f), v in m["dirichlet"].items():
        sim.set_dirichlet(s, f, v)


def prepare(case, seed):
    kind = case["kind"]
    st = dict(case=case)
    if kind == "sdf":
        st["image"] = _image(case["medium"], _box(case), seed)
        return st
    if kind == "batch":
        geoms = []
        for i, (n, p) in enumerate(_batch_members(case)):
            img = _image(case["medium"], [n, n, n], seed * 97 + i, p)
            geoms.append(rd.Geometry(img.cpu().numpy(), None, 1.0, case["edge"]))
        st["geoms"] = geoms
        st["batch"] = rd.Batch(geoms, case["storage"]).bind()
        return st
    img = _image(case["medium"], _box(case), seed)
    geo = rd.Geometry(img.cpu().numpy(), None, 1.0, case["edge"])
    sim = rd.Sim(geo, case["storage"])
    st.update(geometry=geo, sim=sim)
    if kind == "steady":
        sim.add_species(1.0)
        sim.bind(features=rd.RD_WS_SOLVER)
        return st
    m = MODELS[case["model"]]
    _model(sim, m)
    if kind in ("adjoint", "factor"):
        slots = -(-case["steps"] // case["every"]) + case["every"] - 1
        feats = rd.RD_WS_ADJOINT | (rd.RD_WS_DIFFUSIVITY if kind == "factor" else 0)
        sim.bind(features=feats, checkpoint_slots=slots)
        if kind == "factor":
            sim.set_diffusivity(_factor(_box(case), seed))
        st["c0"] = _fields(case, img, seed)[0]
        st["target"] = 0.8 * st["c0"]
        return st
    if case["edge"] == 8:
        if case["layout"] == "compact":
            sim.set_layout("compact")
        sim.set_kernel(case["kernel"])
    sim.set_launch(graph_steps=16, use_graph=True, xcd_map=False)
    if case["sround"]:
        sim.set_rounding(True, seed)
    sim.bind(features=rd.RD_WS_DIFFUSIVITY if kind == "dphi" else 0)
    if kind == "dphi":
        sim.set_diffusivity(_factor(_box(case), seed))
    st["dt"] = m["dt"]
    st["c0"] = [_bleached(img)] if kind == "frap" else _fields(case, img, seed)
    return st


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "sdf":
        return rd.sdf_from_image(state["image"])
    if kind == "batch":
        tau, _, _ = state["batch"].tortuosity(axis=case["axis"])
        return tau
    sim = state["sim"]
    if kind == "steady":
        r = sim.steady_state(case["axis"])
        return [r["tau"], sim.get_field(0)]
    if kind == "adjoint":
        m = MODELS[case["model"]]
        D = torch.tensor(m["D"][0], dtype=torch.float64, device="cuda", requires_grad=True)
        k = torch.tensor(m["reactions"][0][2], dtype=torch.float64, device="cuda", requires_grad=True)
        c = rd.DiffusionDecay.apply(D, k, sim, state["c0"], case["steps"], m["dt"], case["every"])
        loss = 0.5 * ((c - state["target"]) ** 2).sum()
        loss.backward()
        return [c.detach(), D.grad, k.grad]
    if kind == "factor":
        sim.set_field(0, state["c0"])
        loss, gD, gk, ge = sim.adjoint_factor(state["target"], case["steps"], MODELS[case["model"]]["dt"],
                                              case["every"])
        return [loss, gD, gk, ge]
    for s, c in enumerate(state["c0"]):
        sim.set_field(s, c)
    if kind == "frap":
        return sim.frap_curve(0, _region(_box(case)), state["dt"], case["steps"], case["samples"])
    if kind == "monitor":
        out = []
        for _ in range(case["samples"]):
            sim.step(state["dt"], case["steps"])
            out += [sim.balance(s) for s in range(len(state["c0"]))]
        return out + [sim.get_field(s) for s in range(len(state["c0"]))]
    sim.step(state["dt"], case["steps"])
    return [sim.get_field(s) for s in range(len(state["c0"]))]


# ---------------------------------------------------------------------------
# the work a pass cannot do without
# ---------------------------------------------------------------------------

def work(case):
    kind = case["kind"]
    if kind == "batch":
        by = fl = 0.0
        for n, p in _batch_members(case):
            its = 3.3 * n  # iterations to 1e-8
            by += its * 36 * p * n ** 3
            fl += its * 80 * p * n ** 3
        return {"bytes": by, "flops": fl}
    nz, ny, nx = _box(case)
    vox = float(nz * ny * nx)
    act = POROSITY[case["medium"]] * vox
    if kind == "sdf":  # the image in, the distance out
        return {"bytes": 5 * vox, "flops": 20 * vox}
    e = ELEM[case["storage"]]
    if kind == "steady":  # p, x, r, z read and written per iteration, the field out
        its = 2.6 * _box(case)[2 - case["axis"]]
        return {"bytes": its * 36 * act + 4 * vox, "flops": its * 80 * act}
    S = len(MODELS[case["model"]]["D"])
    if kind in ("adjoint", "factor"):
        # a forward, a recomputing and an adjoint sweep; the start field and target in, the
        # final field (or the gradient per voxel) out
        n, f = case["steps"], 4 if kind == "factor" else 0
        by = n * act * (2 * (2 * e + f) + 8 + e + f) + (8 + (8 if f else 4)) * vox
        return {"bytes": by, "flops": n * act * (60 if f else 45)}
    steps = case["steps"] * case.get("samples", 1)
    per = 2 * e * S + (4 if kind == "dphi" else 0)  # each step reads and writes every value once
    by = steps * per * act + 4 * vox * S  # and the start fields in
    if kind != "frap":  # the fields out
        by += 4 * vox * S
    if kind == "monitor":
        by += case["samples"] * e * act * (S + 1)
    elif kind == "frap":
        by += (case["samples"] + 1) * e * act / 64
    return {"bytes": by, "flops": steps * S * act * (25 if kind == "dphi" else 17)}


# ---------------------------------------------------------------------------
# the outputs in FP64 (plain torch, dense arrays)
# ---------------------------------------------------------------------------

def _pairs(m):
    # per axis: the faces between two active voxels
    out = []
    for d in range(3):
        n = m.shape[d]
        out.append((m.narrow(d, 1, n - 1) & m.narrow(d, 0, n - 1)).to(torch.float64))
    return out


def _div(c, w):
    # sum over the active neighbours q of w_pq (c_q - c_p)
    out = torch.zeros_like(c)
    for d in range(3):
        n = c.shape[d]
        f = (c.narrow(d, 1, n - 1) - c.narrow(d, 0, n - 1)) * w[d]
        out.narrow(d, 0, n - 1).add_(f)
        out.narrow(d, 1, n - 1).sub_(f)
    return out


def _plane(shape, face):
    p = torch.zeros(tuple(shape), dtype=torch.bool, device="cuda")
    d = 2 - face // 2
    p.select(d, -1 if face % 2 else 0).fill_(True)
    return p


def _walls(m):
    # in-box inactive neighbours of every voxel
    out = torch.zeros(m.shape, dtype=torch.float64, device="cuda")
    for d in range(3):
        n = m.shape[d]
        out.narrow(d, 0, n - 1).add_((~m.narrow(d, 1, n - 1)).to(torch.float64))
        out.narrow(d, 1, n - 1).add_((~m.narrow(d, 0, n - 1)).to(torch.float64))
    return out


class _Ref:
    """Explicit steps in FP64."""

    def __init__(self, case, img, e=None):
        self.md = MODELS[case["model"]]
        self.m = img != 0
        self.w = _pairs(self.m)
        if e is not None:
            e = e.to(torch.float64)
            for d in range(3):
                n = e.shape[d]
                self.w[d] *= 0.5 * (e.narrow(d, 1, n - 1) + e.narrow(d, 0, n - 1))
        self.free = []
        for s in range(len(self.md["D"])):
            f = self.m.clone()
            for (sp, face), _ in self.md["dirichlet"].items():
                if sp == s:
                    f &= ~_plane(img.shape, face)
            self.free.append(f.to(torch.float64))
        self.walls = _walls(self.m) if self.md["robin"] else None

    def start(self, c0):
        c = [a.to(torch.float64) * self.m for a in c0]
        for (sp, face), v in self.md["dirichlet"].items():
            c[sp][_plane(c[sp].shape, face) & self.m] = v
        return c

    def step(self, c):
        dt = self.md["dt"]
        inc = []
        for s, D in enumerate(self.md["D"]):
            i = _div(c[s], self.w).mul_(D)
            if s in self.md["robin"]:
                i -= self.md["robin"][s] * self.walls * c[s]
            for a, b, k in self.md["reactions"]:
                if a == s:
                    i -= k * c[s]
                if b == s:
                    i += k * c[a]
            inc.append(i.mul_(dt).mul_(self.free[s]))
        return [a + b for a, b in zip(c, inc)]

    def balance(self, c, s):
        md, u = self.md, c[s] * self.free[s]
        inflow = np.zeros(6)
        for (sp, face), _ in md["dirichlet"].items():
            if sp != s:
                continue
            # the flux from the held voxels into their free neighbours
            hold = (_plane(u.shape, face) & self.m).to(torch.float64)
            q = 0.0
            for d in range(3):
                n = u.shape[d]
                lo, hi = [a.narrow(d, 0, n - 1) for a in (c[s], hold, self.free[s])], \
                         [a.narrow(d, 1, n - 1) for a in (c[s], hold, self.free[s])]
                df = (lo[0] - hi[0]) * self.w[d]
                q += float((df * (lo[1] * hi[2] - hi[1] * lo[2])).sum())
            inflow[face] = md["D"][s] * q
        react = 0.0
        for a, b, k in md["reactions"]:
            if a == s:
                react -= k * float(u.sum())
            if b == s:
                react += k * float((c[a] * self.free[s]).sum())
        up = md["robin"].get(s, 0.0)
        return {"mass": float(u.sum()), "inflow": inflow,
                "uptake": up * float((self.walls * u).sum()) if up else 0.0, "react": react}


def _exact_steady(img, axis, tol=1e-13):
    m = img != 0
    shape = m.shape
    inlet, outlet = _plane(shape, 2 * axis) & m, _plane(shape, 2 * axis + 1) & m
    free = m & ~inlet & ~outlet
    w = _pairs(m)
    ff = free.to(torch.float64)
    x0 = inlet.to(torch.float64)
    diag = torch.zeros(shape, dtype=torch.float64, device="cuda")
    for d in range(3):
        n = shape[d]
        diag.narrow(d, 0, n - 1).add_(w[d])
        diag.narrow(d, 1, n - 1).add_(w[d])
    inv = torch.where(diag > 0, 1.0 / diag.clamp(min=1.0), torch.zeros_like(diag)) * ff
    r = _div(x0, w) * ff
    x = torch.zeros_like(x0)
    z = inv * r
    p = z.clone()
    rz = (r * z).sum()
    b2 = float((r * r).sum())
    if b2 > 0:
        for it in range(20000):
            ap = -_div(p, w) * ff
            al = rz / (p * ap).sum()
            x += al * p
            r -= al * ap
            if it % 25 == 24 and float((r * r).sum()) <= tol * tol * b2:
                break
            z = inv * r
            rn = (r * z).sum()
            p = z + (rn / rz) * p
            rz = rn
    x = x + x0
    q = [0.0, 0.0]
    for d in range(3):
        n = shape[d]
        df = (x.narrow(d, 0, n - 1) - x.narrow(d, 1, n - 1)) * w[d]
        fl, fh = ff.narrow(d, 0, n - 1), ff.narrow(d, 1, n - 1)
        for k, h in enumerate((inlet, outlet)):
            hl, hh = h.narrow(d, 0, n - 1).to(torch.float64), h.narrow(d, 1, n - 1).to(torch.float64)
            q[k] += float((df * (hl * fh - hh * fl)).sum())
    flux = 0.5 * (q[0] - q[1])
    n = shape[2 - axis]
    area = float(np.prod(shape)) / n
    psi = float(m.sum()) / float(np.prod(shape))
    tau = psi * area / (flux * (n - 1)) if flux > 1e-9 else float("inf")
    return tau, x


def _dist2(feature):
    # squared distance to the nearest set voxel; one axis after the other, every offset
    big = float(4 * sum(n * n for n in feature.shape))
    g = torch.where(feature, 0.0, big).to(torch.float32)  # exact: integers below 2^24
    for d in range(3):
        n = g.shape[d]
        out = g.clone()
        for k in range(1, n):
            if k * k > float(out.max()):
                break
            torch.minimum(out.narrow(d, k, n - k), g.narrow(d, 0, n - k) + float(k * k),
                          out=out.narrow(d, k, n - k))
            torch.minimum(out.narrow(d, 0, n - k), g.narrow(d, k, n - k) + float(k * k),
                          out=out.narrow(d, 0, n - k))
        g = out
    return g


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        return np.array([_exact_steady(_image(case["medium"], [n, n, n], seed * 97 + i, p), case["axis"])[0]
                         for i, (n, p) in enumerate(_batch_members(case))])
    img = _image(case["medium"], _box(case), seed)
    if kind == "sdf":
        m = img != 0
        if not bool(m.any()) or bool(m.all()):
            return None
        d2 = torch.where(m, _dist2(~m), _dist2(m)).to(torch.float64)
        d = torch.sqrt(d2) - 0.5
        return torch.where(m, d, -d)
    if kind == "steady":
        return list(_exact_steady(img, case["axis"]))
    if kind == "frap":
        ref = _Ref(case, img)
        c = ref.start([_bleached(img)])
        x0, x1, y0, y1, z0, z1 = _region(_box(case))
        out = [float(c[0][z0:z1, y0:y1, x0:x1].sum())]
        for _ in range(case["samples"]):
            for _ in range(case["steps"]):
                c = ref.step(c)
            out.append(float(c[0][z0:z1, y0:y1, x0:x1].sum()))
        return np.array(out)
    c0 = _fields(case, img, seed)
    e = _factor(_box(case), seed) if kind in ("dphi", "factor") else None
    ref = _Ref(case, img, e)
    c = ref.start(c0)
    if kind == "monitor":
        out = []
        for _ in range(case["samples"]):
            for _ in range(case["steps"]):
                c = ref.step(c)
            out += [ref.balance(c, s) for s in range(len(c))]
        return out + c
    if kind in ("step", "dphi"):
        for _ in range(case["steps"]):
            c = ref.step(c)
        return c
    # gradients: the transposed step backwards over the stored states
    md = ref.md
    D, k, dt = md["D"][0], md["reactions"][0][2], md["dt"]
    states = [c[0]]
    for _ in range(case["steps"]):
        c = ref.step(c)
        states.append(c[0])
    free = ref.free[0]
    target = (0.8 * c0[0]).to(torch.float64)
    lam = (states[-1] - target) * free
    loss = 0.5 * float((lam * lam).sum())
    gD = gk = 0.0
    ge = torch.zeros_like(lam) if kind == "factor" else None
    if ge is not None:
        wp = _pairs(ref.m)
    for n in range(case["steps"] - 1, -1, -1):
        cn = states[n]
        gD += dt * float((lam * _div(cn, ref.w)).sum())
        gk -= dt * float((lam * cn * free).sum())
        if ge is not None:
            for d in range(3):
                L = cn.shape[d]
                t = (cn.narrow(d, 1, L - 1) - cn.narrow(d, 0, L - 1)) * \
                    (lam.narrow(d, 0, L - 1) - lam.narrow(d, 1, L - 1)) * wp[d] * (0.5 * D * dt)
                ge.narrow(d, 0, L - 1).add_(t)
                ge.narrow(d, 1, L - 1).add_(t)
        lam = lam + dt * (D * _div(lam, ref.w) - k * lam) * free
    if kind == "factor":
        return [loss, gD, gk, ge]
    return [states[-1], torch.tensor(gD, dtype=torch.float64), torch.tensor(gk, dtype=torch.float64)]
