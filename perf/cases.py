"""Timed workloads of the tracer, the maps, field preparation and the proposer
network, through the package's public calls.

`listed()` names the workloads, `draw(rng)` gives one more of the same ranges,
`prepare` builds what a program holds before the call (inputs from the seed,
prepared field, plan), `run` is one pass, `work` the bytes and FLOPs a pass
cannot do without, and `exact` the FP64 values of the outputs by plain torch.

Kinds: "trace" (one field, one seed set), "batch" (many fields in one call),
"map" (slice with FLL-jump refinement), "volume" (3D map), "field" (node, brick
and direction records of a new field), "propose" and "train" (the network).
Fields are sub-surface point charges or a flux rope over them, in the box
[-1, 1]^2 x [0, 1], or charges in a spherical wedge.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1609_00724_amd as q
from paper_1609_00724_amd import _abi, learn
from paper_1609_00724_amd.api import MapSpec, QMapPlan, TraceBatchPlan, TracePlan, VolumeSpec, make_opts

DEV = "cuda"
LO, HI = (-1.0, -1.0, 0.0), (1.0, 1.0, 1.0)
WEDGE_LO, WEDGE_HI = (-0.3, -0.3, 1.0), (0.3, 0.3, 1.5)
SLAB = dict(x0=-1.0, x1=1.0, y0=-1.0, y1=1.0)


def _trace(name, n, seeds, **kw):
    c = dict(name=name, kind="trace", field="charges", nx=n[0], ny=n[1], nz=n[2], geometry="cartesian", storage="f32",
             mode="paper", order="linear", stepper="ck54", step_dtype="f32", tol=1e-4, cap=1.0, seeds=seeds,
             where="photosphere", noalloc=False)
    c.update(kw)
    return c


def listed():
    return [
        # an interactive probe of a few hundred lines, scratch owned by the
        # library: launches and latency are the whole cost
        _trace("trace_probe", (64, 64, 64), 300, where="box", noalloc=True),
        # the hyperbolic flux tube at tight tolerance, all FP64, one seed per
        # pixel of a 128^2 raster (the accuracy configuration)
        _trace("trace_flux_tube_f64", (64, 64, 64), 128 * 128, field="hyperbolic", storage="f64",
               mode="interp_normalize", step_dtype="f64", tol=1e-8, where="pixels"),
        # random seeds through the box, a ragged count, the paper's 1-cell cap
        _trace("trace_random", (192, 192, 96), 200003, where="box"),
        # a wedge of a spherical model: longitude, latitude, radius
        _trace("trace_spherical", (97, 97, 65), 40000, geometry="spherical", where="photosphere", cap=1.0),
        # the paper's tricubic kernel
        _trace("trace_cubic", (128, 128, 64), 100000, order="cubic", where="photosphere", cap=4.0, tol=1e-3),
        # many fields of uneven size and seed count in one call
        dict(name="batch_fields", kind="batch", sets=12, layout=1, nmin=64, nmax=192, smin=10000, smax=200000, storage="f32",
             step_dtype="f32", tol=1e-4, cap=1.0),
        # one map of the learned pipeline's size, refined by the rule
        dict(name="map_256", kind="map", nx=256, ny=256, nz=128, level=8, refine=2, z0=0.0, threshold=0.02, tol=1e-4,
             cap=1.0, step_dtype="f32", storage="f32", tilted=False),
        # the photospheric map: 1024^2 base pixels, two refinement levels, the
        # fixed-error settings
        dict(name="map_1024", kind="map", nx=256, ny=256, nz=128, level=10, refine=2, z0=0.0, threshold=0.02, tol=1e-2,
             cap=8.0, step_dtype="f32", storage="f32", tilted=False),
        # the flux-rope volume: 256^3 base cells, two levels, the tuned launch
        # word with brick and direction records
        dict(name="volume_rope", kind="volume", nx=384, ny=384, nz=256, level=8, refine=2, threshold=0.02, tol=1e-2,
             cap=4.0, storage="f32", records=True),
        # a new field made ready for the volume tracer
        dict(name="field_records", kind="field", nx=256, ny=256, nz=128, storage="f32", records=True),
        # the network on one coarse 256^2 map
        dict(name="propose_map", kind="propose", tiles=16, side=64),
        # one training step on a batch of tiles
        dict(name="train_256", kind="train", tiles=256, side=64),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _dims(rng, lo, hi):
    nx = _logint(rng, lo, hi)
    return nx, max(8, nx + rng.randint(-nx // 8, nx // 8)), max(8, nx // 2 + rng.randint(-3, 8))


def draw(rng):
    kind = rng.choice(["trace", "trace", "trace", "geometry", "order", "batch", "map", "map", "volume", "field", "propose",
                       "train"])
    tol = rng.choice([1e-2, 1e-3, 1e-4])
    cap = rng.choice([1.0, 2.0, 4.0])
    if kind == "trace":
        c = _trace("", _dims(rng, 33, 224), _logint(rng, 100, 250000), tol=tol, cap=cap,
                   storage=rng.choice(["f32", "f32", "bf16", "f64"]), step_dtype=rng.choice(["f32", "f32", "f64"]),
                   mode=rng.choice(["paper", "paper", "interp_normalize"]), where=rng.choice(["photosphere", "box"]))
        if rng.random() < 0.2:
            c.update(stepper="euler", cap=0.2)
    elif kind == "geometry":
        c = _trace("", _dims(rng, 33, 128), _logint(rng, 300, 60000), tol=tol, cap=cap,
                   geometry=rng.choice(["spherical", "spherical", "stretched"]), step_dtype=rng.choice(["f32", "f64"]),
                   where=rng.choice(["photosphere", "box"]))
    elif kind == "order":
        c = _trace("", _dims(rng, 33, 160), _logint(rng, 300, 150000), tol=tol, cap=cap,
                   order=rng.choice(["quadratic", "cubic"]), where=rng.choice(["photosphere", "box"]))
    elif kind == "batch":
        c = dict(kind=kind, sets=rng.randint(2, 12), layout=rng.randint(0, 10**6), nmin=rng.randint(33, 80), nmax=rng.randint(96, 192), smin=1000,
                 smax=_logint(rng, 5000, 200000), storage=rng.choice(["f32", "bf16"]),
                 step_dtype=rng.choice(["f32", "f32", "f64"]), tol=tol, cap=1.0)
    elif kind == "map":
        n = _dims(rng, 64, 256)
        c = dict(kind=kind, nx=n[0], ny=n[1], nz=n[2], level=rng.randint(5, 10), refine=rng.randint(0, 3),
                 z0=rng.choice([0.0, 0.0, round(rng.uniform(0.01, 0.3), 3)]), threshold=round(rng.uniform(0.01, 0.1), 3), tol=tol,
                 cap=rng.choice([1.0, 4.0, 8.0]), step_dtype=rng.choice(["f32", "f32", "f64"]),
                 storage=rng.choice(["f32", "f32", "bf16"]), tilted=rng.random() < 0.2)
    elif kind == "volume":
        n = _dims(rng, 48, 224)
        c = dict(kind=kind, nx=n[0], ny=n[1], nz=n[2], level=rng.randint(4, 7), refine=rng.randint(0, 2),
                 threshold=round(rng.uniform(0.01, 0.1), 3), tol=tol, cap=rng.choice([1.0, 4.0]), storage="f32",
                 records=rng.random() < 0.5)
    elif kind == "field":
        n = _dims(rng, 32, 256)
        st = rng.choice(["f32", "f32", "bf16", "f64"])
        c = dict(kind=kind, nx=n[0], ny=n[1], nz=n[2], storage=st, records=st == "f32")
    else:
        c = dict(kind=kind, tiles=_logint(rng, 1, 256), side=rng.choice([32, 64, 64, 96, 128]))
        c["tiles"] = max(1, min(c["tiles"], 256 * 64 * 64 // c["side"] ** 2))
    c.pop("name", None)
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _axes(case):
    """Node coordinates per axis (FP64, device)."""
    n = (case["nx"], case["ny"], case["nz"])
    lo, hi = (WEDGE_LO, WEDGE_HI) if case.get("geometry") == "spherical" else (LO, HI)
    ax = [torch.linspace(lo[d], hi[d], n[d], dtype=torch.float64, device=DEV) for d in range(3)]
    if case.get("geometry") == "stretched":
        for d in range(2):   # denser towards the middle
            ax[d] = torch.linspace(-1, 1, n[d], dtype=torch.float64, device=DEV)
            ax[d] = 0.5 * ax[d] + 0.5 * ax[d] ** 3
        s = torch.linspace(0, 1, n[2], dtype=torch.float64, device=DEV)   # denser towards the bottom
        ax[2] = (torch.exp(1.5 * s) - 1) / (math.exp(1.5) - 1)
        ax[2][0], ax[2][-1] = 0.0, 1.0
        for d in range(2):
            ax[d][0], ax[d][-1] = -1.0, 1.0
    return ax


def _charges(g):
    """2-8 sub-surface charges of zero net charge (rows x, y, z, q)."""
    k = int(g.integers(2, 9))
    pos, dep, mag = g.uniform(-0.5, 0.5, (k, 2)), g.uniform(0.05, 0.15, k), g.uniform(0.5, 1.5, k)
    npos = (k + 1) // 2
    mag[npos:] *= -mag[:npos].sum() / mag[npos:].sum()
    return np.column_stack([pos, -dep, mag])


def _charge_field(ch, X, Y, Z):
    out = [torch.zeros_like(X) for _ in range(3)]
    for cx, cy, cz, w in ch:
        dx, dy, dz = X - cx, Y - cy, Z - cz
        f = w * (dx * dx + dy * dy + dz * dz) ** -1.5
        for o, d in zip(out, (dx, dy, dz)):
            o += d * f
    return out


def _rope_field(g, ax):
    """A ring current below the photosphere with a twisted core, two leg charges
    and a drawn background; FP32 components, in z slabs to bound memory."""
    R, zc, a = 0.3, -0.1, 0.08
    xl = math.sqrt(R * R - zc * zc)
    ch = np.vstack([[[xl, 0, zc, 1.5], [-xl, 0, zc, -1.5]], _charges(g)])
    amp = float(g.uniform(1.0, 2.0))
    th = np.arange(96) * (2 * math.pi / 96)
    parts = []
    for z0 in range(0, ax[2].numel(), 64):
        Z, Y, X = torch.meshgrid(ax[2][z0:z0 + 64], ax[1], ax[0], indexing="ij")
        X, Y, Z = X.contiguous(), Y.contiguous(), Z.contiguous()
        b = _charge_field(ch, X, Y, Z)
        for t in th:
            tx, tz = -R * math.sin(t) * th[1], R * math.cos(t) * th[1]
            rx, rz = X - R * math.cos(t), Z - (zc + R * math.sin(t))
            w = 0.5 * (rx * rx + Y * Y + rz * rz + a * a) ** -1.5
            b[0] -= w * tz * Y
            b[1] += w * (tz * rx - tx * rz)
            b[2] += w * tx * Y
        s = torch.sqrt(X * X + (Z - zc) ** 2)
        rho2 = (s - R) ** 2 + Y * Y
        bt = torch.where(rho2 < a * a, amp * (1 - rho2 / (a * a)), torch.zeros_like(s))
        b[0] -= bt * (Z - zc) / s
        b[2] += bt * X / s
        parts.append([c.float() for c in b])
    return [torch.cat([p[i] for p in parts]) for i in range(3)]


def _components(case, g, ax):
    """B components on the nodes, (nz, ny, nx): FP32, or FP64 for FP64 storage."""
    dt = torch.float64 if case["storage"] == "f64" else torch.float32
    if case.get("field") == "rope":
        return [c.to(dt) for c in _rope_field(g, ax)]
    Z, Y, X = (t.contiguous() for t in torch.meshgrid(ax[2], ax[1], ax[0], indexing="ij"))
    if case.get("field") == "hyperbolic":
        k = float(g.uniform(1.0, 2.5))
        return [(k * X).to(dt), (-k * Y).to(dt), torch.ones_like(Z).to(dt)]
    if case.get("geometry") == "spherical":
        ch = _charges(g)
        # the same charges under the wedge's middle: (z + depth) becomes 1 - depth along x
        ch = np.column_stack([1.0 + ch[:, 2], 0.4 * ch[:, 0], 0.4 * ch[:, 1], ch[:, 3]])
        ct, st, cp, sp = torch.cos(Y), torch.sin(Y), torch.cos(X), torch.sin(X)
        bx, by, bz = _charge_field(ch, Z * ct * cp, Z * ct * sp, Z * st)
        return [(-sp * bx + cp * by).to(dt), (-st * cp * bx - st * sp * by + ct * bz).to(dt),
                (ct * cp * bx + ct * sp * by + st * bz).to(dt)]
    return [c.to(dt) for c in _charge_field(_charges(g), X, Y, Z)]


def _geometry(case, ax):
    n = (case["nx"], case["ny"], case["nz"])
    origin = tuple(float(a[0]) for a in ax)
    spacing = tuple((float(a[-1]) - float(a[0])) / (n[d] - 1) for d, a in enumerate(ax))
    return origin, spacing


def _cell(case, spacing, ax):
    """Smallest cell length: arc length along each axis at the lower boundary."""
    if case.get("geometry") == "stretched":
        return min(float((a[1:] - a[:-1]).min()) for a in ax)
    if case.get("geometry") == "spherical":
        return min(spacing[0] * math.cos(0.3), spacing[1], spacing[2])
    return min(spacing)


def _field(case, g, ax, comps=None):
    origin, spacing = _geometry(case, ax)
    b = comps if comps is not None else _components(case, g, ax)
    kw = {}
    if case.get("geometry") == "spherical":
        kw = dict(geometry="spherical")
    elif case.get("geometry") == "stretched":
        kw = dict(coords=tuple(ax))
    return q.field_init(*b, origin, spacing, storage=case["storage"], mode=case.get("mode", "paper"),
                        order=case.get("order", "linear"), **kw)


def _opts(case, h, launch=0):
    if case.get("stepper") == "euler":
        return make_opts(1e-4, 1e-4, case["cap"] * h, 0.0, stepper="euler", step_dtype=case["step_dtype"])
    return make_opts(case["tol"], case["tol"], 0.1 * h, case["cap"] * h, step_dtype=case.get("step_dtype", "f32"),
                     launch=launch)


def _seeds(case, g, ax):
    """(n, 3) FP64 seeds on the bottom face, on a raster of it or in the box."""
    lo, hi = [float(a[0]) for a in ax], [float(a[-1]) for a in ax]
    n = case["seeds"]
    if case["where"] == "pixels":
        side = math.isqrt(n)
        i = (np.arange(side) + 0.5) / side
        Y, X = np.meshgrid(i, i, indexing="ij")
        p = np.column_stack([X.ravel(), Y.ravel(), np.zeros(side * side)])
    else:
        p = g.uniform(0.0, 1.0, (n, 3))
        if case["where"] == "photosphere":
            p[:, 2] = 0.0
    s = np.array(lo) + p * (np.array(hi) - np.array(lo))
    return torch.from_numpy(s).to(DEV)


def _tiles(case, seed):
    """Smooth random feature tiles, a refine mask and log10 Q with gaps."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    n, s = case["tiles"], case["side"]
    x = torch.rand((n, 3, s // 8, s // 8), generator=g, device=DEV)
    x = torch.nn.functional.interpolate(x, size=(s, s), mode="bilinear", align_corners=False)
    x = (x + 0.1 * torch.randn((n, 3, s, s), generator=g, device=DEV)).permute(0, 2, 3, 1).contiguous()
    mask = (x[..., 1] > 0.6).float()
    logq = 1.0 + 3.0 * x[..., 0]
    logq = torch.where(torch.rand((n, s, s), generator=g, device=DEV) < 0.02, torch.full_like(logq, math.nan), logq)
    return x, mask, logq


def _net(seed):
    """A network in mid-training: He-normal weights, Adam moments of its scale."""
    p = learn.init_params(seed, DEV)
    g = torch.Generator(device=DEV).manual_seed(seed + 1)
    m = 1e-3 * torch.randn(p.shape, generator=g, device=DEV)
    v = 1e-5 * (0.5 + torch.rand(p.shape, generator=g, device=DEV))
    return p, m, v


def prepare(case, seed):
    g = np.random.Generator(np.random.PCG64(seed))
    kind = case["kind"]
    if kind in ("propose", "train"):
        p, m, v = _net(seed)
        net = learn.Proposer(p)
        x, mask, logq = _tiles(case, seed + 2)
        if kind == "propose":
            return dict(kind=kind, net=net, x=x, ws=net.workspace(*x.shape[:3]))
        net.m.copy_(m)
        net.v.copy_(v)
        net.t = 500
        return dict(kind=kind, net=net, x=x, mask=mask, logq=logq)
    if kind == "batch":
        sets = []
        for c in _batch_sets(case):
            ax = _axes(c)
            sets.append((_field(c, g, ax), _seeds(c, g, ax)))
        opts = make_opts(case["tol"], case["tol"], step_dtype=case["step_dtype"])
        return dict(kind=kind, plan=TraceBatchPlan(sets, opts, want=("fp_fwd", "fp_bwd", "fll", "q_perp")))
    if kind == "volume":
        case = dict(case, field="rope")
    ax = _axes(case)
    origin, spacing = _geometry(case, ax)
    if kind == "field":
        return dict(kind=kind, b=_components(case, g, ax), origin=origin, spacing=spacing, case=case)
    field = _field(case, g, ax)
    h = _cell(case, spacing, ax)
    if kind == "trace":
        seeds = _seeds(case, g, ax)
        return dict(kind=kind, field=field, opts=_opts(case, h), soa=seeds.t().contiguous(),
                    plan=TracePlan(seeds.shape[0], seeds.device, noalloc=case["noalloc"]))
    m, r = case["level"], case["refine"]
    if kind == "map":
        plane = None
        if case["tilted"]:
            plane = ((-0.8, -0.9, 0.05), (1.5, 0.1, 0.0), (0.1, 1.4, 0.6))
        spec = MapSpec(case["z0"], **SLAB, base_level=m, refine_levels=r, out_level=m + min(r, 1),
                       threshold=case["threshold"], plane=plane)
        return dict(kind=kind, field=field, opts=_opts(case, h), plan=_map_plan(spec, 4 ** m * min(8, 4 ** r)))
    launch = 0
    if case["records"]:
        field.add_bricks().add_cell_dirs()
        launch = _abi.launch_word(2, 64, _abi.GATHER_BRICKS, refine_gather=_abi.GATHER_DIRS)
    spec = VolumeSpec(**SLAB, z0=0.0, z1=1.0, base_level=m, refine_levels=r, out_level=m, threshold=case["threshold"])
    return dict(kind=kind, field=field, opts=_opts(case, h, launch), plan=_map_plan(spec, 8 ** m * min(2 if m > 7 else 8, 8 ** r)))


def _map_plan(spec, capacity):
    plan = QMapPlan(spec, capacity, DEV)
    for t in (plan.keys, plan.fll, plan.q_perp, plan.status):   # entries past the samples held stay zero
        t.zero_()
    return plan


def _batch_sets(case):
    """The trace case of every set of a batch: grid and seed count by the layout."""
    g = np.random.Generator(np.random.PCG64(case["layout"]))
    for _ in range(case["sets"]):
        nx = int(g.integers(case["nmin"], case["nmax"] + 1))
        n = (nx, int(g.integers(case["nmin"], case["nmax"] + 1)), max(16, nx // 2))
        s = int(round(math.exp(g.uniform(math.log(case["smin"]), math.log(case["smax"])))))
        yield _trace("", n, s, storage=case["storage"])


def run(state):
    kind = state["kind"]
    if kind == "trace":
        return state["plan"].run(state["field"], state["soa"], state["opts"])
    if kind == "batch":
        return state["plan"].run()
    if kind in ("map", "volume"):
        p = state["plan"].run(state["field"], state["opts"])
        return dict(count=p.count, overflow=p.overflow, keys=p.keys, fll=p.fll, q_perp=p.q_perp, status=p.status,
                    q_grid=p.q_grid, fll_grid=p.fll_grid, fledge=p.fledge)
    if kind == "field":
        c = state["case"]
        f = q.field_init(*state["b"], state["origin"], state["spacing"], storage=c["storage"])
        n = c["nx"] * c["ny"] * c["nz"]
        dt = {"f32": torch.float32, "f64": torch.float64, "bf16": torch.bfloat16}[c["storage"]]
        out = dict(nodes=f.ws.view(dt)[:4 * n])
        if c["records"]:
            f.add_bricks().add_cell_dirs()
            out.update(bricks=f.bricks_ws.view(dt), dirs=f.dirs_ws.view(dt))
        return out
    net = state["net"]
    if kind == "propose":
        return net.forward(state["x"], ws=state["ws"])
    loss, grad = net.train_step(state["x"], state["mask"], state["logq"], want_grad=True)
    return dict(loss=loss, grad=grad, params=net.params, m=net.m, v=net.v)


# ---------------------------------------------------------------------------
# work: inputs read once, outputs written once; FLOPs of the method
# ---------------------------------------------------------------------------
# per RHS evaluation at the trilinear / quadratic / cubic kernels, and per
# Cash-Karp attempt of 9 components (FMA = 2)
_EVAL = {"linear": 147, "quadratic": 651, "cubic": 1290}
_ATTEMPT = 600


def _line_flops(case, spacing_min, extent):
    """FLOPs of one line: field lines of these fields run about half the box's
    width; a step takes at most `cap` cells."""
    steps = max(4.0, 0.5 * extent / (case["cap"] * spacing_min)) + 4
    if case.get("stepper") == "euler":
        return steps * (_EVAL[case.get("order", "linear")] + 18)
    return steps * (6 * _EVAL[case.get("order", "linear")] + _ATTEMPT)


_NODE = {"f32": 16, "bf16": 8, "f64": 32}


def work(case):
    kind = case["kind"]
    if kind in ("propose", "train"):
        px = case["tiles"] * case["side"] ** 2
        conv = [9 * ci * co * 2 for ci, co in zip(learn.CHANNELS[:-1], learn.CHANNELS[1:])]
        if kind == "propose":
            return dict(bytes=px * 20, flops=px * sum(conv))
        # forward, weight gradients of four layers, input gradients of three
        return dict(bytes=px * 20 + 19970 * 4 * 8, flops=px * (2 * sum(conv) + sum(conv[1:])))
    if kind == "batch":
        n = (case["nmin"] + case["nmax"]) / 2
        lines = case["sets"] * (case["smax"] - case["smin"]) / math.log(case["smax"] / case["smin"])
        return dict(bytes=case["sets"] * n ** 3 / 2 * _NODE[case["storage"]] + lines * 108,
                    flops=lines * _line_flops(case, 2.0 / n, 2.0))
    nodes = case["nx"] * case["ny"] * case["nz"]
    if kind == "field":
        per = _NODE[case["storage"]]
        b = nodes * (24 if case["storage"] == "f64" else 12) + nodes * per
        return dict(bytes=b + (nodes * (16 + 96) if case["records"] else 0), flops=nodes * 10)
    wedge = case.get("geometry") == "spherical"
    extent = 0.6 if wedge else 2.0
    h = extent / max(case["nx"], case["ny"]) * (0.5 if case.get("geometry") == "stretched" else 1.0)
    if kind == "trace":
        return dict(bytes=nodes * _NODE[case["storage"]] + case["seeds"] * 124,
                    flops=case["seeds"] * _line_flops(case, h, extent))
    dim = 2 if kind == "map" else 3
    lines = 2 ** (dim * case["level"]) * (1.3 if case["refine"] else 1.0)
    grid = 2 ** (dim * (case["level"] + (min(case["refine"], 1) if dim == 2 else 0))) * 8
    return dict(bytes=nodes * _NODE[case["storage"]] + lines * 28 + grid + 2 ** (dim * case["level"]) * 4,
                flops=lines * _line_flops(case, h, extent))


# ---------------------------------------------------------------------------
# FP64 values by plain torch
# ---------------------------------------------------------------------------
_A = [[], [1 / 5], [3 / 40, 9 / 40], [3 / 10, -9 / 10, 6 / 5], [-11 / 54, 5 / 2, -70 / 27, 35 / 27],
      [1631 / 55296, 175 / 512, 575 / 13824, 44275 / 110592, 253 / 4096]]
_B5 = [37 / 378, 0, 250 / 621, 125 / 594, 0, 512 / 1771]
_B4 = [2825 / 27648, 0, 18575 / 48384, 13525 / 55296, 277 / 14336, 1 / 4]


class _Line:
    """The line and deviation equations on the nodes of a case, in FP64."""

    def __init__(self, case, b, ax):
        self.ax, self.paper = ax, case["mode"] == "paper"
        self.uniform = case["geometry"] != "stretched"
        self.sphere = case["geometry"] == "spherical"
        self.order = {"linear": 1, "quadratic": 2, "cubic": 3}[case["order"]]
        B = torch.stack([c.double() for c in b], -1)
        mag = B.norm(dim=-1, keepdim=True)
        v = torch.cat([B / mag, mag], -1) if self.paper else torch.cat([B, mag], -1)
        if self.order > 1:   # a layer beyond each face: 3 f(0) - 3 f(1) + f(2)
            for d in range(3):
                s = [v.select(d, k).unsqueeze(d) for k in (0, 1, 2, -1, -2, -3)]
                v = torch.cat([3 * s[0] - 3 * s[1] + s[2], v, 3 * s[3] - 3 * s[4] + s[5]], d)
        self.dims = v.shape[:3]
        self.v = v.reshape(-1, 4)
        self.lo = torch.tensor([float(a[0]) for a in ax], dtype=torch.float64, device=DEV)
        self.hi = torch.tensor([float(a[-1]) for a in ax], dtype=torch.float64, device=DEV)

    def field(self, x):
        """u (n, 3), G[j][i] = d u_i / d x_j as (n, 3, 3), |B| (n)."""
        idx, ws, ds = [], [], []
        for d in range(3):
            a, p = self.ax[d], x[:, d].contiguous()
            if self.uniform:
                h = (a[-1] - a[0]) / (a.numel() - 1)
                s = (p - a[0]) / h
                c = s.floor().clamp(0, a.numel() - 2)
                t = s - c
                c = c.long()
                h = h.expand_as(t)
            else:
                c = (torch.searchsorted(a, p, right=True) - 1).clamp(0, a.numel() - 2)
                h = a[c + 1] - a[c]
                t = (p - a[c]) / h
            if self.order == 1:
                w, dw = [1 - t, t], [-torch.ones_like(t), torch.ones_like(t)]
            elif self.order == 3:
                t2, t3 = t * t, t * t * t
                w = [(-t3 + 2 * t2 - t) / 2, (3 * t3 - 5 * t2 + 2) / 2, (-3 * t3 + 4 * t2 + t) / 2, (t3 - t2) / 2]
                dw = [(-3 * t2 + 4 * t - 1) / 2, (9 * t2 - 10 * t) / 2, (-9 * t2 + 8 * t + 1) / 2, (3 * t2 - 2 * t) / 2]
            else:
                near = (t >= 0.5).long()
                u = t - near
                c = c + near
                w, dw = [u * (u - 0.5), 1 - 2 * u * u, u * (u + 0.5)], [2 * u - 0.5, -4 * u, 2 * u + 0.5]
            idx.append(c[:, None] + torch.arange(len(w), device=DEV))
            ws.append(torch.stack(w, 1))
            ds.append(torch.stack(dw, 1) / h[:, None])
        K = ws[0].shape[1]
        flat = (idx[2][:, :, None, None] * self.dims[1] + idx[1][:, None, :, None]) * self.dims[2] + idx[0][:, None, None, :]
        v = self.v[flat.reshape(-1)].reshape(-1, K, K, K, 4)
        ex = [(v * w[:, None, None, :, None]).sum(3) for w in (ws[0], ds[0])]
        ey = [(e * w[:, None, :, None]).sum(2) for e, w in ((ex[0], ws[1]), (ex[1], ws[1]), (ex[0], ds[1]))]
        ez = [(e * w[:, :, None]).sum(1) for e, w in ((ey[0], ws[2]), (ey[1], ws[2]), (ey[2], ws[2]), (ey[0], ds[2]))]
        val, G = ez[0], torch.stack([e[:, :3] for e in ez[1:]], 1)
        if self.paper:
            return val[:, :3], G, val[:, 3]
        b = val[:, :3].norm(dim=1, keepdim=True)
        u = val[:, :3] / b
        return u, (G - u[:, None, :] * (G * u[:, None, :]).sum(2, keepdim=True)) / b[:, None], b[:, 0]

    def scale(self, x):
        s = torch.ones_like(x)
        if self.sphere:
            s[:, 0], s[:, 1] = x[:, 2] * torch.cos(x[:, 1]), x[:, 2]
        return s

    def rhs(self, y, sigma):
        u, G, _ = self.field(y[:, :3])
        d = [(G * y[:, k:k + 3, None]).sum(1) for k in (3, 6)]
        f = torch.cat([u] + d, 1) * sigma[:, None]
        return f / self.scale(y[:, :3]).repeat(1, 3) if self.sphere else f

    def step(self, y, sigma, h, euler):
        """End of one step and the error estimate's numerator."""
        K = [self.rhs(y, sigma)]
        if euler:
            return y + h[:, None] * K[0], torch.zeros_like(y)
        for a in _A[1:]:
            K.append(self.rhs(y + h[:, None] * sum(c * k for c, k in zip(a, K)), sigma))
        y5 = y + h[:, None] * sum(c * k for c, k in zip(_B5, K))
        return y5, h[:, None] * sum((c - e) * k for c, e, k in zip(_B5, _B4, K))

    def gap(self, x):
        """Largest signed distance beyond a face, and that face."""
        g = torch.stack([self.lo - x, x - self.hi], 2).reshape(-1, 6)
        return g.max(1)


def _exact_trace(case, seed):
    g = np.random.Generator(np.random.PCG64(seed))
    ax = _axes(case)
    L = _Line(case, _components(case, g, ax), ax)
    x0 = _seeds(case, g, ax)
    h0 = _cell(case, _geometry(case, ax)[1], ax)
    euler = case["stepper"] == "euler"
    n = x0.shape[0]
    u, _, B0 = L.field(x0)
    u = u / u.norm(dim=1, keepdim=True)
    sg = torch.where(u[:, 2] < 0, -1.0, 1.0).double()
    p = -1 / (sg + u[:, 2])
    e1 = torch.stack([1 + sg * u[:, 0] ** 2 * p, sg * u[:, 0] * u[:, 1] * p, -sg * u[:, 0]], 1)
    e2 = torch.stack([u[:, 0] * u[:, 1] * p, sg + u[:, 1] ** 2 * p, -u[:, 1]], 1)
    s0 = L.scale(x0)
    y = torch.cat([x0, e1 / s0, e2 / s0], 1).repeat(2, 1)
    sigma = torch.ones(2 * n, dtype=torch.float64, device=DEV)
    sigma[n:] = -1
    length = torch.zeros_like(sigma)
    face = torch.full((2 * n,), -1, device=DEV)
    for f in range(6):   # a seed on a face whose signed field points out ends there
        d, top = f // 2, f % 2
        out = sigma * u[:, d].repeat(2) * (1 if top else -1) > 0
        on = (x0[:, d] == (L.hi if top else L.lo)[d]).repeat(2)
        face = torch.where((face < 0) & on & out, f, face)
    hmax = case["cap"] * h0
    h = torch.full_like(sigma, hmax if euler else 0.1 * h0)
    act = (face < 0).nonzero()[:, 0]
    pend = torch.zeros_like(sigma)
    for _ in range(20000):
        if not act.numel():
            break
        ya, hs = y[act], h[act].clamp(max=hmax)
        yn, e = L.step(ya, sigma[act], hs, euler)
        err = (e.abs() / (case["tol"] + case["tol"] * torch.maximum(ya.abs(), yn.abs()))).amax(1)
        ok = err <= 1
        out = ok & (L.gap(yn[:, :3])[0] > 0)
        pend[act[out]] = hs[out]
        move = ok & ~out
        y[act[move]] = yn[move]
        length[act[move]] += hs[move]
        if not euler:
            h[act] = torch.where(ok, hs * (0.9 * err.clamp(min=1e-300) ** -0.2).clamp(max=5),
                                 hs * (0.9 * err.clamp(min=1e-300) ** -0.25).clamp(min=0.2))
        act = act[~out]
    # the step that left the box, cut where its end lies on the face
    for i in (pend > 0).nonzero()[:, 0].split(200000):
        yi, si = y[i], sigma[i]
        a, b = torch.zeros_like(si), pend[i].clone()
        ga, gb = L.gap(yi[:, :3])[0], L.gap(L.step(yi, si, b, euler)[0][:, :3])[0]
        side, c = torch.zeros_like(a), b
        for _ in range(80):
            c = torch.where(ga >= 0, a, (a * gb - b * ga) / (gb - ga))
            gc = L.gap(L.step(yi, si, c, euler)[0][:, :3])[0]
            if bool((gc.abs() <= 1e-14).all()):
                break
            up = gc > 0
            ga = torch.where(up, torch.where(side > 0, ga / 2, ga), gc)
            gb = torch.where(up, gc, torch.where(side < 0, gb / 2, gb))
            a, b = torch.where(up, a, c), torch.where(up, c, b)
            side = torch.where(up, 1.0, -1.0).double()
        yl = L.step(yi, si, c, euler)[0]
        f = L.gap(yl[:, :3])[1]
        wall = torch.stack([L.lo, L.hi], 1).reshape(-1)[f]
        yl[torch.arange(yl.shape[0], device=DEV), f // 2] = wall
        y[i], face[i] = yl, f
        length[i] += c
    yF, yB = y[:n], y[n:]
    out = dict(fp_fwd=yF[:, :3].t().contiguous(), fp_bwd=yB[:, :3].t().contiguous(), fll=length[:n] + length[n:])
    if case["step_dtype"] != "f64" or case["storage"] == "bf16":
        # the largest Q set the norm, and there FP32 steps are at the limit of
        # the problem's conditioning: no value to hold them to
        return dict(out, q_perp=None, q_det=None, q_fp=None)
    ends = []
    for yy, f in ((yF, face[:n]), (yB, face[n:])):
        v, _, mag = L.field(yy[:, :3])
        sc = L.scale(yy[:, :3])
        a, b = yy[:, 3:6] * sc, yy[:, 6:9] * sc
        un = v / v.norm(dim=1, keepdim=True)
        perp = [d - un * (un * d).sum(1, keepdim=True) for d in (a, b)]
        k = (f // 2)[:, None]
        plane = [d - v * (d.gather(1, k) / v.gather(1, k)) for d in (a, b)]
        ends.append((perp, plane, mag))

    def bracket(F, K):
        dot = lambda s, t: (s * t).sum(1)  # noqa: E731
        br = (dot(F[0], F[0]) * dot(K[1], K[1]) + dot(K[0], K[0]) * dot(F[1], F[1])
              - 2 * dot(K[0], K[1]) * dot(F[0], F[1]))
        area = torch.linalg.cross(F[0], F[1]).norm(dim=1) * torch.linalg.cross(K[0], K[1]).norm(dim=1)
        return br, area

    br, area = bracket(ends[0][0], ends[1][0])
    bf, af = bracket(ends[0][1], ends[1][1])
    return dict(out, q_perp=ends[0][2] * ends[1][2] / B0 ** 2 * br, q_det=br / area, q_fp=bf / af)


def _network(params, x):
    """(n, h, w, 2) outputs of the network in FP64 from an FP64 parameter vector."""
    h, w = x.shape[1:3]
    for layer, (wo, bo) in enumerate(learn.param_offsets()):
        ci, co = learn.CHANNELS[layer], learn.CHANNELS[layer + 1]
        W = params[wo:bo].reshape(9, ci, co)
        xp = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
        y = params[bo:bo + co]
        for tap in range(9):
            dy, dx = tap // 3, tap % 3
            y = y + xp[:, dy:dy + h, dx:dx + w, :].reshape(-1, ci).matmul(W[tap]).reshape(*x.shape[:3], co)
        x = torch.relu(y) if layer < 3 else y
    return x


def _exact_net(case, seed):
    p, m, v = _net(seed)
    x, mask, logq = _tiles(case, seed + 2)
    if case["kind"] == "propose":
        with torch.no_grad():
            return _network(p.double(), x.double())
    P = mask.numel()
    pd = p.double()
    grad, loss = torch.zeros_like(pd), torch.zeros((), dtype=torch.float64, device=DEV)
    for i in range(0, x.shape[0], 64):   # tiles in groups, to bound the graph's memory
        pg = pd.clone().requires_grad_(True)
        out = _network(pg, x[i:i + 64].double())
        z, t, tq = out[..., 0], mask[i:i + 64].double(), logq[i:i + 64].double()
        ok = torch.isfinite(tq)
        dq = torch.where(ok, out[..., 1] - torch.where(ok, tq, torch.zeros_like(tq)), torch.zeros_like(tq))
        part = (torch.nn.functional.softplus(z, threshold=1e9) - t * z + 0.1 * dq * dq).sum() / P
        part.backward()
        grad += pg.grad
        loss += part.detach()
    m = 0.9 * m.double() + 0.1 * grad
    v = 0.999 * v.double() + 0.001 * grad * grad
    pd = pd - 1e-3 * (m / (1 - 0.9 ** 501)) / ((v / (1 - 0.999 ** 501)).sqrt() + 1e-8)
    return dict(loss=loss, grad=grad, params=pd, m=m, v=v)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("propose", "train"):
        return _exact_net(case, seed)
    if kind == "trace":
        return _exact_trace(case, seed)
    if kind == "field":
        g = np.random.Generator(np.random.PCG64(seed))
        ax = _axes(case)
        B = torch.stack([c.double() for c in _components(case, g, ax)], -1)
        mag = B.norm(dim=-1, keepdim=True)
        nodes = torch.cat([B / mag, mag], -1)
        if not case["records"]:
            return dict(nodes=nodes.reshape(-1))
        nz, ny, nx = nodes.shape[:3]
        pad = torch.nn.functional.pad(nodes, (0, 0, 0, nx % 2, 0, ny % 2, 0, nz % 2))
        s = pad.shape
        bricks = pad.reshape(s[0] // 2, 2, s[1] // 2, 2, s[2] // 2, 2, 4).permute(0, 2, 4, 1, 3, 5, 6)
        dirs = torch.stack([nodes[c:nz - 1 + c, b:ny - 1 + b, a:nx - 1 + a, :3]
                            for c in (0, 1) for b in (0, 1) for a in (0, 1)], 3)
        return dict(nodes=nodes.reshape(-1), bricks=bricks.reshape(-1), dirs=dirs.reshape(-1))
    return None   # which samples a map keeps depends on the traced lengths themselves
