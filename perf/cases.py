"""Timing cases of the framework: what a program that coarse grains particles has it do.

Each case is one call (or the few calls that belong together) through the
public entry points of paper_1409_0001_amd, with the inputs, the mesh and the
output buffers such a program keeps between time steps already on the GPU.
Sizes come from the repository's own workloads (inputs.py, bench.py) and
tests; the drawn cases spread over the same ranges.  `exact` computes the same
result in float64 with plain torch on the same device.
"""
import math

import numpy as np
import torch

import paper_1409_0001_amd as cgd
from paper_1409_0001_amd import inputs

DEV = "cuda"


def listed():
    return [
        # the paper's own order of size: 24^3 cells, 20,000 spheres; launches and read-backs decide
        {"name": "hex_small", "kind": "hex", "nx": 24, "ny": 24, "nz": 24, "n": 20_000, "F": 1, "depth": 1.0,
         "bcells": 1.2, "steps": 4, "scheme": "be", "stats": False},
        # one time step of a coupled run on a 128^3 mesh: solid volume and three momentum components
        {"name": "hex_momentum", "kind": "hex", "nx": 128, "ny": 128, "nz": 128, "n": 2_000_000, "F": 4,
         "depth": 1.0, "bcells": 4.0, "steps": 4, "scheme": "be", "stats": False},
        # a mesh whose sizes are whatever the geometry gave (odd, wider than a wave covers), the paper's integrator
        {"name": "hex_odd_cn", "kind": "hex", "nx": 275, "ny": 147, "nz": 93, "n": 1_000_000, "F": 2, "depth": 0.6,
         "bcells": 4.0, "steps": 3, "scheme": "cn", "stats": False},
        # the dense bed at full size
        {"name": "hex_dense_bed", "kind": "hex", "nx": 256, "ny": 256, "nz": 512, "n": 20_000_000, "F": 1,
         "depth": 2.0, "bcells": 4.0, "steps": 4, "scheme": "be", "stats": False},
        # the same recipe with the solver's statistics asked for (iterations, residuals, mass; the iterations come back)
        {"name": "hex_stats", "kind": "hex", "nx": 128, "ny": 128, "nz": 256, "n": 2_500_000, "F": 1, "depth": 2.0,
         "bcells": 4.0, "steps": 4, "scheme": "be", "stats": True},
        # stretched across the bed, diffusivity 0 in the outer layers (deposited values kept there)
        {"name": "rect_stretched", "kind": "rect", "nx": 128, "ny": 128, "nz": 256, "n": 2_500_000, "F": 1,
         "depth": 2.0, "ratio": 1.02, "axis": 0, "cut": 0.45, "periodic": 0, "bcells": 4.0, "steps": 4,
         "scheme": "be"},
        # a channel: periodic along x and y, cells refined towards the walls in z
        {"name": "rect_channel", "kind": "rect", "nx": 96, "ny": 64, "nz": 80, "n": 400_000, "F": 2, "depth": 1.0,
         "ratio": 1.03, "axis": 2, "cut": 1.0, "periodic": 3, "bcells": 3.0, "steps": 3, "scheme": "be"},
        # an unstructured mesh: 40^3 x 6 jittered tets, location and solve
        {"name": "tet", "kind": "tet", "hexes": 40, "n": 320_000, "F": 1, "bcells": 4.0, "steps": 4,
         "scheme": "be"},
        # many snapshots at once, uneven particle counts, volume and three drag components
        {"name": "batched", "kind": "batched", "nx": 128, "ny": 128, "nz": 128, "snaps": 16, "n": 20_000_000,
         "F": 4, "bcells": 4.0, "steps": 4, "scheme": "be"},
        # the centroid method alone: four fields, whole-number sums asked for
        {"name": "deposit", "kind": "deposit", "nx": 128, "ny": 128, "nz": 256, "n": 8_000_000, "F": 4, "depth": 2.0},
        # the learned guess: one prediction on the trained grid
        {"name": "unet_forward", "kind": "unet", "nx": 128, "ny": 128, "nz": 128, "grad": False},
        # the learned guess: loss and gradients of one training pair
        {"name": "unet_grad", "kind": "unet", "nx": 64, "ny": 64, "nz": 64, "grad": True},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["hex"] * 6 + ["rect"] * 3 + ["batched"] * 2 + ["deposit"] * 2 + ["tet", "unet"])
    nx, ny, nz = (_log(rng, 16, 300) for _ in range(3))
    if rng.random() < 0.4:  # grids of powers of two are as common as odd ones
        nx, ny, nz = (1 << rng.randint(4, 8) for _ in range(3))
    cells = nx * ny * nz
    F = rng.choice([1, 1, 2, 4]) if cells < 8_000_000 else 1
    n = min(int(cells * math.exp(rng.uniform(math.log(0.1), math.log(2.0)))), 16_000_000 // F) + rng.randint(0, 99)
    steps = rng.choice([1, 2, 3, 4, 4, 6])
    bcells = round(rng.uniform(2.0, 6.0), 2)
    scheme = rng.choice(["be", "be", "be", "cn"])
    depth = round(rng.uniform(0.5, 2.0), 2)
    if kind == "hex":
        return {"kind": kind, "nx": nx, "ny": ny, "nz": nz, "n": n, "F": F, "depth": depth, "bcells": bcells,
                "steps": steps, "scheme": scheme, "stats": rng.random() < 0.2}
    if kind == "deposit":
        return {"kind": kind, "nx": nx, "ny": ny, "nz": nz, "n": n, "F": F, "depth": depth}
    if kind == "rect":
        nx, ny, nz = (max(8, v // 2) for v in (nx, ny, nz))
        periodic = rng.choice([0, 0, 3])
        return {"kind": kind, "nx": nx, "ny": ny, "nz": nz, "n": n // 8 + 1000, "F": min(F, 2), "depth": depth,
                "ratio": round(1.0 + rng.uniform(0.0, 2.0) / max(nx, ny, nz), 4), "axis": 2 if periodic else 0,
                "cut": rng.choice([0.45, 1.0]), "periodic": periodic, "bcells": bcells, "steps": steps,
                "scheme": scheme}
    if kind == "batched":
        nx, ny, nz = (max(16, v // 2) for v in (nx, ny, nz))
        snaps = rng.randint(2, 12)
        return {"kind": kind, "nx": nx, "ny": ny, "nz": nz, "snaps": snaps, "n": snaps * (n // 8 + 1000), "F": F,
                "bcells": bcells, "steps": steps, "scheme": scheme}
    if kind == "tet":
        hexes = _log(rng, 8, 44)
        return {"kind": kind, "hexes": hexes, "n": 5 * hexes ** 3 + rng.randint(0, 99), "F": min(F, 2),
                "bcells": round(rng.uniform(2.0, 4.0), 2), "steps": steps, "scheme": scheme}
    return {"kind": "unet", "nx": 4 * rng.randint(4, 32), "ny": 4 * rng.randint(4, 24), "nz": 4 * rng.randint(4, 16),
            "grad": rng.random() < 0.5}


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * int(seed) + 17)
    return g


def _bed(n, F, depth, g, lo=(0.0, 0.0, 0.0), hi=None):
    """Dense bed: 70 % of the spheres uniform in the bottom quarter, 30 % in
    50 Gaussian clumps; lognormal diameters.  Field 0 is the sphere volume,
    the others the volume times N(0, 1) components."""
    n_bed = int(0.7 * n)
    pos = torch.rand((n, 3), generator=g, device=DEV, dtype=torch.float32)
    pos[:n_bed, 2] *= 0.25
    centres = torch.rand((50, 3), generator=g, device=DEV)
    which = torch.randint(0, 50, (n - n_bed,), generator=g, device=DEV)
    clump = centres[which] + 0.05 * torch.randn((n - n_bed, 3), generator=g, device=DEV)
    clump = torch.where(clump < 0, -clump, clump)
    clump = torch.where(clump > 1, 2 - clump, clump)
    pos[n_bed:] = clump.clamp_(0.0, 1.0)
    pos[:, 2] *= depth
    pos = pos[torch.randperm(n, generator=g, device=DEV)].contiguous()
    return pos, _values(n, F, g)


def _values(n, F, g):
    d = torch.exp(math.log(0.003) + 0.3 * torch.randn(n, generator=g, device=DEV))
    vals = torch.empty((F, n), device=DEV)
    vals[0] = math.pi / 6.0 * d ** 3
    for f in range(1, F):
        vals[f] = vals[0] * torch.randn(n, generator=g, device=DEV)
    return vals


def _box(case):
    return (0.0, 0.0, 0.0), (1.0, 1.0, float(case.get("depth", 1.0)))


def _b(case):
    """Bandwidth: bcells widths of the mean cell."""
    lo, hi = _box(case)
    vol = math.prod((hi[a] - lo[a]) / case["n" + "xyz"[a]] for a in range(3))
    return case["bcells"] * vol ** (1.0 / 3.0)


def _edges(case):
    lo, hi = _box(case)
    out = []
    for a, n in enumerate((case["nx"], case["ny"], case["nz"])):
        w = np.ones(n)
        if a == case["axis"]:
            mid = np.abs(np.arange(n) - (n - 1) / 2.0)
            # x: wider away from the centre plane; z: finer towards both walls
            w = case["ratio"] ** (mid if a == 0 else -mid)
        e = np.concatenate([[0.0], np.cumsum(w)])
        e *= (hi[a] - lo[a]) / e[-1]
        e[-1] = hi[a]
        out.append(e)
    return out


def _diffusivity(case, edges):
    """None, or 0 in the cells further than `cut` from the centre plane of axis 0 and 1 elsewhere."""
    if case["cut"] >= 1.0:
        return None
    xc = 0.5 * (edges[0][1:] + edges[0][:-1])
    d = (np.abs(xc - 0.5) <= case["cut"]).astype(np.float32)
    return np.ascontiguousarray(np.broadcast_to(d, (case["nz"], case["ny"], case["nx"])).ravel())


def _offsets(case, seed):
    r = np.random.default_rng(seed + 5)
    share = r.uniform(0.5, 4.0, case["snaps"])
    cut = np.floor(np.cumsum(share) / share.sum() * case["n"]).astype(np.int64)
    cut[-1] = case["n"]
    return np.concatenate([[0], cut]).astype(np.int64)


_LAYERS = [("e1a", 1, 16), ("e1b", 16, 16), ("e2a", 16, 32), ("e2b", 32, 32), ("e3a", 32, 64), ("e3b", 64, 64),
           ("u2", 64, 32), ("d2a", 64, 32), ("d2b", 32, 32), ("u1", 32, 16), ("d1a", 32, 16), ("d1b", 16, 16)]


def _unet_params(seed):
    r = np.random.default_rng(seed + 9)
    v = []
    for _, ci, co in _LAYERS:
        v.append(r.standard_normal(co * 27 * ci) * math.sqrt(2.0 / (27 * ci)))
        v.append(0.02 * r.standard_normal(co))
    v.append(0.1 * r.standard_normal(17))
    return np.concatenate(v).astype(np.float32)


def _smooth(e, times):
    for _ in range(times):
        for a in range(3):
            p = torch.cat([e.narrow(a, 0, 1), e, e.narrow(a, e.shape[a] - 1, 1)], dim=a)
            n = e.shape[a]
            e = 0.25 * p.narrow(a, 0, n) + 0.5 * e + 0.25 * p.narrow(a, 2, n)
    return e


def _pair(case, seed):
    """A deposited-looking field and the same field one diffusion step on."""
    g = _gen(seed)
    shape = (case["nz"], case["ny"], case["nx"])
    density = _smooth(torch.rand(shape, generator=g, device=DEV) ** 4, 4)
    density[: shape[0] // 2] *= 3.0
    e = torch.rand(shape, generator=g, device=DEV) * density
    return e.reshape(-1).contiguous(), _smooth(e, 2).reshape(-1).contiguous()


def _particles(case, seed):
    g = _gen(seed)
    if case["kind"] in ("tet", "batched"):
        return torch.rand((case["n"], 3), generator=g, device=DEV), _values(case["n"], case["F"], g)
    return _bed(case["n"], case["F"], case.get("depth", 1.0), g)


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind == "unet":
        s["net"] = cgd.UNet((case["nx"], case["ny"], case["nz"]), seed=1)
        s["net"].set_params(_unet_params(seed))
        s["x"], s["target"] = _pair(case, seed)
        s["y"] = torch.empty_like(s["x"])
        return s
    s["pos"], s["values"] = _particles(case, seed)
    F = case["F"]
    if kind == "tet":
        xyz, tets = inputs.kuhn_tet_mesh(case["hexes"], 0.2, seed + 3)
        s["mesh"] = cgd.TetMesh(xyz, tets)
        s["b"] = case["bcells"] / case["hexes"]
    elif kind == "rect":
        e = _edges(case)
        per = tuple(bool(case["periodic"] >> a & 1) for a in range(3))
        s["mesh"] = cgd.RectMesh(*e, diffusivity=_diffusivity(case, e), periodic=per)
        s["b"] = _b(case)
    else:
        lo, hi = _box(case)
        s["mesh"] = cgd.HexMesh((case["nx"], case["ny"], case["nz"]), lo, hi)
        s["b"] = _b(case) if "bcells" in case else 0.0
    cells = s["mesh"].cells
    if kind == "batched":
        s["offsets"] = _offsets(case, seed)
        s["field"] = torch.empty((case["snaps"], F, cells), device=DEV)
    else:
        s["field"] = torch.empty((F, cells), device=DEV)
    if kind == "deposit":
        s["acc"] = torch.empty((F, cells), dtype=torch.int64, device=DEV)
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "unet":
        if case["grad"]:
            loss = s["net"].loss_grad(s["x"], s["target"])
            return {"loss": loss, "grads": s["net"].get_grads()}
        return {"y": s["net"].forward(s["x"], s["y"])}
    if kind == "deposit":
        f = cgd.deposit(s["mesh"], s["pos"], s["values"], field=s["field"], acc=s["acc"])
        return {"field": f, "acc": s["acc"]}
    if kind == "batched":
        return {"field": cgd.coarse_grain_batched(s["mesh"], s["offsets"], s["pos"], s["values"], s["b"],
                                                  case["steps"], rtol=1e-6, fields=s["field"],
                                                  scheme=case["scheme"])}
    f, st = cgd.coarse_grain(s["mesh"], s["pos"], s["values"], s["b"], case["steps"], rtol=1e-6, field=s["field"],
                             stats=bool(case.get("stats")), scheme=case["scheme"])
    if st is not None:
        return {"field": f, "iters": np.array(st.iters, dtype=np.int32)}
    return {"field": f}


def work(case):
    """Particles read once, fields written once; one multiply-add per cell,
    step and face at the least.  The network: its convolutions' operations."""
    if case["kind"] == "unet":
        cells = case["nx"] * case["ny"] * case["nz"]
        level = {"1": 1, "2": 8, "3": 64}
        conv = sum(54.0 * ci * co * cells / level[name[1]] for name, ci, co in _LAYERS)
        first = 54.0 * 16 * cells
        if case["grad"]:  # forward, input gradients of all layers but the first, weight gradients
            return {"bytes": 8.0 * cells + 4.0 * 390_000, "flops": 3.0 * conv - first}
        return {"bytes": 8.0 * cells, "flops": conv}
    cells = 6 * case["hexes"] ** 3 if case["kind"] == "tet" else case["nx"] * case["ny"] * case["nz"]
    F = case["F"]
    moved = (12.0 + 4.0 * F) * case["n"] + 4.0 * F * cells * case.get("snaps", 1)
    if case["kind"] == "deposit":
        return {"bytes": moved + 8.0 * F * cells, "flops": 0.0}
    return {"bytes": moved, "flops": 14.0 * F * cells * case["steps"] * case.get("snaps", 1)}


# ------------------------------------------------------------------ float64

def _host_cells(case, pos, edges):
    """Host cell of every particle from the node coordinates (uniform axes: by
    floor((x - lo) s), as the mesh defines it)."""
    lo, hi = _box(case)
    n = (case["nx"], case["ny"], case["nz"])
    idx = []
    for a in range(3):
        x = pos[:, a].double()
        if edges is None:
            i = torch.floor((x - lo[a]) * (n[a] / (hi[a] - lo[a]))).long()
        else:
            i = torch.searchsorted(torch.from_numpy(edges[a]).to(x.device), x, right=True) - 1
        idx.append(i.clamp_(0, n[a] - 1))
    return idx[0] + n[0] * (idx[1] + n[1] * idx[2])


def _sums(cell, values, cells):
    out = torch.zeros((values.shape[0], cells), dtype=torch.float64, device=values.device)
    for f in range(values.shape[0]):
        out[f].index_add_(0, cell, values[f].double())
    return out


def _cosines(n, device):
    k = torch.arange(n, dtype=torch.float64, device=device)
    c = torch.cos(math.pi / n * k[:, None] * (k[None, :] + 0.5)) * math.sqrt(2.0 / n)
    c[0] *= math.sqrt(0.5)
    return c


def _along(mat, e, axis):
    """mat applied along one axis of e [F, nz, ny, nx], a field at a time."""
    for f in range(e.shape[0]):
        e[f] = torch.movedim(torch.matmul(torch.movedim(e[f], axis, -1), mat.T), -1, axis)
    return e


def _diffuse_box(case, e):
    """n steps of the uniform zero-flux box by its cosine modes."""
    lo, hi = _box(case)
    dims = (case["nz"], case["ny"], case["nx"])
    ext = (hi[2] - lo[2], hi[1] - lo[1], hi[0] - lo[0])
    dtau = _b(case) ** 2 / 4.0 / case["steps"]
    e = e.reshape((-1,) + dims)
    lam = 0.0
    mats = []
    for a in range(3):
        k = torch.arange(dims[a], dtype=torch.float64, device=e.device)
        la = 4.0 * (dims[a] / ext[a]) ** 2 * torch.sin(math.pi * k / (2 * dims[a])) ** 2
        lam = lam + la.reshape([-1 if b == a else 1 for b in range(3)])
        mats.append(_cosines(dims[a], e.device))
    gain = 1.0 / (1.0 + dtau * lam) if case["scheme"] == "be" else (1.0 - dtau / 2 * lam) / (1.0 + dtau / 2 * lam)
    gain = gain ** case["steps"]
    for a in range(3):
        e = _along(mats[a], e, a)
    e *= gain
    for a in range(3):
        e = _along(mats[a].T, e, a)
    return e.reshape(e.shape[0], -1)


def _cg(apply_a, b, dot):
    x, r = torch.zeros_like(b), b.clone()
    p, rr = r.clone(), dot(r, r)
    stop = 1e-26 * rr
    for _ in range(3000):
        if bool((rr <= stop).all()):
            break
        q = apply_a(p)
        al = rr / dot(p, q)
        x += al * p
        r -= al * q
        new = dot(r, r)
        p = r + (new / rr) * p
        rr = new
    return x


def _march(case, dtau, mass, stiff, e):
    """Backward Euler or Crank-Nicolson of M de/dt = -K e."""
    half = dtau if case["scheme"] == "be" else 0.5 * dtau
    out = []
    for f in range(e.shape[0]):
        x = e[f]
        for _ in range(case["steps"]):
            if float(x.abs().max()) == 0.0:
                break
            y = _cg(lambda p: mass * p + half * stiff(p), mass * x, lambda u, v: (u * v).sum())
            x = y if case["scheme"] == "be" else 2.0 * y - x
        out.append(x)
    return torch.stack(out)


def _exact_rect(case, seed):
    pos, values = _particles(case, seed)
    edges = _edges(case)
    n = (case["nx"], case["ny"], case["nz"])
    h = [torch.from_numpy(np.diff(e)).to(DEV) for e in edges]
    vol = h[2][:, None, None] * h[1][None, :, None] * h[0][None, None, :]
    d = _diffusivity(case, edges)
    d = torch.ones_like(vol) if d is None else torch.from_numpy(d).to(DEV).double().reshape(vol.shape)
    e = _sums(_host_cells(case, pos, edges), values, vol.numel()).reshape((-1,) + tuple(vol.shape)) / vol
    faces = []
    for a in range(3):
        ax = 2 - a
        area = vol / h[a].reshape([-1 if b == ax else 1 for b in range(3)])
        per = bool(case["periodic"] >> a & 1) and n[a] > 1
        up = torch.roll(d, -1, ax)
        df = torch.where(d + up > 0, 2.0 * d * up / (d + up).clamp_min(1e-300), torch.zeros_like(d))
        dist = 0.5 * (h[a] + torch.roll(h[a], -1))
        c = df * area / dist.reshape([-1 if b == ax else 1 for b in range(3)])
        if not per:
            c.narrow(ax, n[a] - 1, 1).zero_()
        faces.append((ax, c))

    def stiff(p):
        y = torch.zeros_like(p)
        for ax, c in faces:
            flux = c * (p - torch.roll(p, -1, ax))
            y += flux - torch.roll(flux, 1, ax)
        return y

    dtau = _b(case) ** 2 / 4.0 / case["steps"]
    return {"field": _march(case, dtau, vol, stiff, e).reshape(e.shape[0], -1)}


def _exact_tet(case, seed):
    pos, values = _particles(case, seed)
    m = case["hexes"]
    xyz, tets = inputs.kuhn_tet_mesh(m, 0.2, seed + 3)
    xyz = torch.from_numpy(xyz).to(DEV)
    tv = torch.from_numpy(tets).to(DEV).long()
    v = xyz[tv]
    vol = torch.linalg.det(v[:, 1:] - v[:, :1]).abs() / 6.0
    # host tets: the 27 hexes around the particle's lattice hex hold every candidate
    p = pos.double()
    base = (p * m).floor().long().clamp_(0, m - 1)
    best = torch.full((p.shape[0],), -1, dtype=torch.long, device=DEV)
    margin = torch.full((p.shape[0],), -math.inf, dtype=torch.float64, device=DEV)
    inv = torch.linalg.inv((v[:, 1:] - v[:, :1]).transpose(1, 2))
    for off in range(27):
        d = torch.tensor([off % 3 - 1, off // 3 % 3 - 1, off // 9 - 1], device=DEV)
        c = base + d
        ok = ((c >= 0) & (c < m)).all(1)
        c = c.clamp(0, m - 1)
        first = 6 * (c[:, 0] + m * (c[:, 1] + m * c[:, 2]))
        for t in range(6):
            tet = first + t
            w = torch.bmm(inv[tet], (p - v[tet, 0]).unsqueeze(2).contiguous()).squeeze(2)
            low = torch.minimum(w.min(1).values, 1.0 - w.sum(1))
            take = ok & (low > margin)
            margin = torch.where(take, low, margin)
            best = torch.where(take, tet, best)
    e = _sums(best, values, tv.shape[0]) / vol
    # two-point fluxes over the interior faces
    tri = torch.stack([tv[:, [1, 2, 3]], tv[:, [0, 2, 3]], tv[:, [0, 1, 3]], tv[:, [0, 1, 2]]], 1).reshape(-1, 3)
    tri = tri.sort(1).values
    nv = xyz.shape[0]
    order = torch.argsort((tri[:, 0] * nv + tri[:, 1]) * nv + tri[:, 2])
    owner = order // 4
    s = tri[order]
    same = (s[1:] == s[:-1]).all(1)
    i, j, f = owner[:-1][same], owner[1:][same], s[:-1][same]
    area = 0.5 * torch.linalg.norm(torch.cross(xyz[f[:, 1]] - xyz[f[:, 0]], xyz[f[:, 2]] - xyz[f[:, 0]], dim=1), dim=1)
    cen = v.mean(1)
    a = area / torch.linalg.norm(cen[j] - cen[i], dim=1)

    def stiff(q):
        flux = a * (q[i] - q[j])
        y = torch.zeros_like(q)
        y.index_add_(0, i, flux)
        y.index_add_(0, j, -flux)
        return y

    dtau = (case["bcells"] / m) ** 2 / 4.0 / case["steps"]
    return {"field": _march(case, dtau, vol, stiff, e)}


def _conv(x, w, b):
    """3x3x3 correlation with zero padding, channels last, as 27 products."""
    xp = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1, 1, 1))
    d, h, wd, _ = x.shape
    y = b.expand(d, h, wd, -1)
    for t in range(27):
        z, yy, xx = t // 9, t // 3 % 3, t % 3
        y = y + torch.matmul(xp[z:z + d, yy:yy + h, xx:xx + wd], w[:, t].T)
    return torch.relu(y)


def _exact_unet(case, seed):
    x, target = _pair(case, seed)
    shape = (case["nz"], case["ny"], case["nx"], 1)
    x, target = x.double().reshape(shape), target.double().reshape(shape)
    flat = torch.from_numpy(_unet_params(seed)).to(DEV).double().requires_grad_(case["grad"])
    P, o = {}, 0
    for name, ci, co in _LAYERS:
        P[name] = (flat[o:o + co * 27 * ci].reshape(co, 27, ci), flat[o + co * 27 * ci:o + co * 27 * ci + co])
        o += co * 27 * ci + co
    hw, hb = flat[o:o + 16], flat[o + 16]

    def pool(t):
        d, h, w, c = t.shape
        return t.reshape(d // 2, 2, h // 2, 2, w // 2, 2, c).mean(dim=(1, 3, 5))

    def up(t):
        return t.repeat_interleave(2, 0).repeat_interleave(2, 1).repeat_interleave(2, 2)

    with torch.set_grad_enabled(case["grad"]):
        s = x.square().mean().sqrt()
        e1 = _conv(_conv(x / s, *P["e1a"]), *P["e1b"])
        e2 = _conv(_conv(pool(e1), *P["e2a"]), *P["e2b"])
        e3 = _conv(_conv(pool(e2), *P["e3a"]), *P["e3b"])
        u2 = _conv(up(e3), *P["u2"])
        d2 = _conv(_conv(torch.cat([u2, e2], 3), *P["d2a"]), *P["d2b"])
        u1 = _conv(up(d2), *P["u1"])
        d1 = _conv(_conv(torch.cat([u1, e1], 3), *P["d1a"]), *P["d1b"])
        y = x + s * (torch.matmul(d1, hw) + hb).unsqueeze(3)
        if not case["grad"]:
            return {"y": y.reshape(-1)}
        loss = ((y - target) / s).square().mean()
        loss.backward()
    return {"loss": float(loss), "grads": flat.grad.cpu().numpy()}


def exact(case, seed):
    kind = case["kind"]
    if kind == "unet":
        return _exact_unet(case, seed)
    if kind == "tet":
        return _exact_tet(case, seed)
    if kind == "rect":
        return _exact_rect(case, seed)
    pos, values = _particles(case, seed)
    lo, hi = _box(case)
    cells = case["nx"] * case["ny"] * case["nz"]
    vol = math.prod(hi[a] - lo[a] for a in range(3)) / cells
    cell = _host_cells(case, pos, None)
    if kind == "batched":
        off = _offsets(case, seed)
        out = torch.empty((case["snaps"], case["F"], cells), dtype=torch.float64, device=DEV)
        for j in range(case["snaps"]):
            part = slice(int(off[j]), int(off[j + 1]))
            out[j] = _diffuse_box(case, _sums(cell[part], values[:, part], cells) / vol)
        return {"field": out}
    e = _sums(cell, values, cells) / vol
    if kind == "deposit":
        return {"field": e, "acc": None}
    e = _diffuse_box(case, e)
    if case["stats"]:
        return {"field": e, "iters": None}
    return {"field": e}
