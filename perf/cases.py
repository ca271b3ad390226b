"""The work that users of this framework have it do, as cases that can be timed and compared.

A case is a dict of plain values.  ``listed()`` names the standing ones, ``draw(rng)`` makes
another of the same ranges, ``prepare(case, seed)`` builds what a program holds before the call
(inputs on the GPU, plans), ``run(state)`` is one pass through the public entry points,
``work(case)`` the bytes and operations a pass cannot do without, and ``exact(case, seed)`` the
same results in plain 64-bit torch.

Kinds of case and what they stand for:

  call     the one-shot functions on a small mesh: capacities counted, buffers allocated, leaf
           and pyramid built, all within the call (an asset imported once)
  sphere   a closed mesh re-voxelized through kept plans (an animated asset); at the finer
           grids its triangles span many voxels
  weave    a woven fabric of explicit fibers through kept plans, or replayed from a graph
  metal    a height field with triangles of about a voxel, with merged lobes (K = 4)
  patches  many fabric patches of uneven size in one batched build
  fit      one optimisation step of the two-lobe fit: loss and gradients
  codes    eigen-fit and 6-byte SGGX code of a level's voxels, and the decode
  samples  the sampling voxelizer
  occupancy  sub-voxel occupancy of a pyramid's levels
  sggxh    the histogram-distance lobe reduction over a pyramid
"""
from __future__ import annotations

import math
import zlib
from dataclasses import dataclass

import numpy as np
import torch

import paper_2604_13191_amd as vx

DEV = "cuda"
F64 = torch.float64
LATTICE = 1 << 23                    # lattice units per grid extent
RADIUS = 0.5                         # fiber radius in voxels, as everywhere in this repository


@dataclass
class Grid:
    bmin: tuple
    extent: float
    log2_res: int


# ------------------------------------------------------------------------------------------------
# the cases
# ------------------------------------------------------------------------------------------------

def listed():
    return [
        # an asset imported once: 20,480 triangles at 64^3, all counting and allocation in the call
        {"name": "sphere_call", "kind": "call", "subdiv": 5, "log2_res": 6, "levels": 7, "K": 1},
        # a strand of 64 fibers re-voxelized every frame from a captured graph: launches count
        {"name": "strand_graph", "kind": "weave", "fibers": 64, "points": 257, "log2_res": 10, "levels": 11, "K": 1,
         "graph": True},
        # a closed mesh whose triangles span many voxels, with merged lobes
        {"name": "sphere_fine", "kind": "sphere", "subdiv": 5, "log2_res": 9, "levels": 8, "K": 4},
        # a fabric swatch of explicit fibers, full pyramid
        {"name": "weave", "kind": "weave", "fibers": 2000, "points": 257, "log2_res": 10, "levels": 11, "K": 1,
         "graph": False},
        # an odd-sized piece of a brushed surface
        {"name": "metal_piece", "kind": "metal", "window": 777, "log2_res": 12, "levels": 8, "K": 4},
        # the whole surface: 33.5 M triangles
        {"name": "metal", "kind": "metal", "window": 4096, "log2_res": 12, "levels": 8, "K": 4},
        # a garment's patches, 100 to 2,500 fibers each, in one build
        {"name": "patches", "kind": "patches", "patches": 14, "low": 100, "high": 2500, "levels": 8, "K": 4},
        # one optimisation step (forward and backward) on a fabric of 500 fibers
        {"name": "fit", "kind": "fit", "fibers": 500, "points": 257, "log2_res": 10, "lo": 1, "hi": 6},
        # the storage code of a leaf
        {"name": "codes", "kind": "codes", "n": 5131046},
        # the paper's sampler at 16 samples for the largest triangle
        {"name": "samples", "kind": "samples", "window": 1537, "log2_res": 12, "N": 16},
        # densities of a surface piece, leaf and seven coarser levels
        {"name": "occupancy", "kind": "occupancy", "window": 1025, "log2_res": 12, "levels": 8},
        # the paper's lobe reduction, 5,000 samples a lobe
        {"name": "sggxh", "kind": "sggxh", "window": 257, "log2_res": 12, "levels": 8, "K": 4, "samples": 5000},
    ]


def draw(rng):
    def log(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    kind = rng.choice(["call", "sphere", "weave", "weave", "metal", "metal", "patches", "fit", "codes", "samples",
                       "occupancy", "sggxh"])
    if kind == "call":
        l2 = rng.randint(5, 8)
        return {"kind": kind, "subdiv": rng.randint(2, 5), "log2_res": l2, "levels": rng.randint(2, min(l2 + 1, 8)),
                "K": rng.choice([1, 1, 4])}
    if kind == "sphere":
        return {"kind": kind, "subdiv": rng.randint(3, 6), "log2_res": rng.randint(7, 9),
                "levels": rng.randint(4, 8), "K": rng.choice([1, 2, 4])}
    if kind == "weave":
        l2 = rng.randint(8, 11)
        K = rng.choice([1, 1, 4])
        return {"kind": kind, "fibers": log(17, 3000), "points": log(33, 400), "log2_res": l2,
                "levels": l2 + 1 if K == 1 and l2 < 11 else rng.randint(5, 8), "K": K,
                "graph": rng.random() < 0.3}
    if kind == "metal":
        return {"kind": kind, "window": log(33, 2100), "log2_res": rng.randint(11, 12), "levels": rng.randint(5, 8),
                "K": rng.choice([1, 2, 4, 4])}
    if kind == "patches":
        low = log(30, 300)
        return {"kind": kind, "patches": rng.randint(2, 24), "low": low, "high": low * rng.randint(2, 6),
                "levels": rng.randint(5, 8), "K": rng.choice([1, 4])}
    if kind == "fit":
        return {"kind": kind, "fibers": log(20, 1500), "points": log(33, 300), "log2_res": rng.randint(8, 10),
                "lo": rng.randint(1, 2), "hi": rng.randint(3, 6)}
    if kind == "codes":
        return {"kind": kind, "n": log(1000, 6000000)}
    if kind == "samples":
        if rng.random() < 0.5:
            return {"kind": kind, "window": log(65, 2100), "log2_res": 12, "N": log(2, 24)}
        return {"kind": kind, "fibers": log(20, 2500), "points": log(33, 300), "log2_res": rng.randint(8, 11),
                "chords": rng.randint(1, 5), "per_chord": rng.randint(1, 5)}
    if kind == "occupancy":
        if rng.random() < 0.5:
            return {"kind": kind, "window": log(65, 1500), "log2_res": 12, "levels": rng.randint(3, 8)}
        return {"kind": kind, "fibers": log(20, 1000), "points": log(33, 300), "log2_res": rng.randint(8, 10),
                "levels": rng.randint(3, 8)}
    return {"kind": kind, "window": log(33, 257), "log2_res": rng.randint(11, 12), "levels": rng.randint(3, 8),
            "K": rng.choice([2, 4]), "samples": rng.choice([500, 2000, 5000])}


# ------------------------------------------------------------------------------------------------
# inputs, from the seed alone
# ------------------------------------------------------------------------------------------------
# A case's geometry is drawn once from the case's own values; a seed turns it (an axis permutation
# and mirrors, exact on the lattice) and starts its primitives elsewhere, so that every seed has
# other coordinates, keys and orders but as many voxels, and results of two seeds have one shape.

def own_seed(case):
    return zlib.crc32(repr(sorted((k, v) for k, v in case.items() if k != "name")).encode())


TURNS = ((0, 1, 2), (1, 0, 2), (0, 2, 1), (2, 0, 1), (1, 2, 0), (2, 1, 0))


def turned(p, extent, turn, odd=False):
    """Points rounded to the lattice of [0, extent]^3 (odd: to its odd places, so that no point
    lies on a voxel's face, where a clipped length has no derivative) and turned (48 ways), as float32."""
    p = p.to(F64) * (LATTICE / extent)
    p = (2.0 * torch.round(0.5 * (p - 1.0)) + 1.0 if odd else torch.round(p)) * (extent / LATTICE)
    axes = [p[..., a] for a in TURNS[turn % 6]]
    axes = [extent - x if (turn // 6 >> a) & 1 else x for a, x in enumerate(axes)]
    return torch.stack(axes, -1).float().contiguous()


def sphere_mesh(case, seed):
    """Icosahedron subdivided onto a sphere of radius 0.45 in the unit cube, jittered per vertex,
    as a soup of float32 triangles."""
    t = (1.0 + math.sqrt(5.0)) / 2.0
    v = np.array([[-1, t, 0], [1, t, 0], [-1, -t, 0], [1, -t, 0], [0, -1, t], [0, 1, t], [0, -1, -t], [0, 1, -t],
                  [t, 0, -1], [t, 0, 1], [-t, 0, -1], [-t, 0, 1]], dtype=np.float64)
    f = np.array([[0, 11, 5], [0, 5, 1], [0, 1, 7], [0, 7, 10], [0, 10, 11], [1, 5, 9], [5, 11, 4], [11, 10, 2],
                  [10, 7, 6], [7, 1, 8], [3, 9, 4], [3, 4, 2], [3, 2, 6], [3, 6, 8], [3, 8, 9], [4, 9, 5],
                  [2, 4, 11], [6, 2, 10], [8, 6, 7], [9, 8, 1]], dtype=np.int64)
    v /= np.linalg.norm(v, axis=1, keepdims=True)
    for _ in range(case["subdiv"]):
        e = np.sort(f[:, [[0, 1], [1, 2], [2, 0]]].reshape(-1, 2), axis=1)
        u, inv = np.unique(e, axis=0, return_inverse=True)
        m = v[u[:, 0]] + v[u[:, 1]]
        ab, bc, ca = (inv.reshape(-1, 3) + len(v)).T
        v = np.concatenate([v, m / np.linalg.norm(m, axis=1, keepdims=True)])
        a, b, c = f.T
        f = np.stack([a, ab, ca, b, bc, ab, c, ca, bc, ab, bc, ca], 1).reshape(-1, 3)
    rng = np.random.default_rng(own_seed(case))
    p = 0.5 + 0.45 * v + rng.normal(0.0, 1e-3, v.shape)
    tris = turned(torch.as_tensor(p[f]).to(DEV), 1.0, seed % 48)
    return torch.roll(tris, 97 * seed % len(f), 0).contiguous(), Grid((0.0, 0.0, 0.0), 1.0, case["log2_res"])


def metal_field(case, seed):
    """Height field with ridges (wavelength about 8 cells along x and 256 along y, amplitude 2
 triangles per cell, the first window^2 vertices of a one-voxel lattice."""
    rng = np.random.default_rng(own_seed(case))
    n_waves = 16
    fx = rng.uniform(0.9, 1.1, n_waves) / 8.0
    fy = rng.choice([-1.0, 1.0], n_waves) * rng.uniform(0.5, 1.5, n_waves) / 256.0
    ph = rng.uniform(0.0, 2.0 * math.pi, n_waves)
    n, res = case["window"], 1 << case["log2_res"]
    n = min(n, res)
    x = torch.arange(n, dtype=F64, device=DEV)[:, None] + 0.5
    y = torch.arange(n, dtype=F64, device=DEV)[None, :] + 0.5
    h = torch.zeros((n, n), dtype=F64, device=DEV)
    for a in range(n_waves):
        h += torch.cos(2.0 * math.pi * (fx[a] * x + fy[a] * y) + ph[a])
    z = res / 2.0 + 2.0 * h / h.abs().max()
    # a sample on a voxel's face belongs to the upper one: sampled fields are not mirrored
    p = turned(torch.stack([x.expand(n, n), y.expand(n, n), z], -1), float(res),
               seed % (6 if case["kind"] == "samples" else 48))
    v00, v10, v01, v11 = p[:-1, :-1], p[1:, :-1], p[:-1, 1:], p[1:, 1:]
    tris = torch.stack([torch.stack([v00, v10, v11], 2), torch.stack([v00, v11, v01], 2)], 2)
    tris = tris.reshape(-1, 3, 3)
    tris = torch.roll(tris, 9973 * seed % len(tris), 0).contiguous()
    return tris, Grid((0.0, 0.0, 0.0), float(res), case["log2_res"])


def weave_points(n_fibers, n_points, log2_res, gen, seed):
    """Plain weave in voxel units, its fibers in the order and turn of the seed: half of them along
    x, half along y, grouped in yarns of pitch 32 with crimp 4, helical twist up to 5 degrees and
    0.3 voxel of jitter."""
    res = 1 << log2_res

    def uniform(a, b):
        return a + (b - a) * torch.rand(n_fibers, 1, dtype=F64, device=DEV, generator=gen)

    f = torch.arange(n_fibers, device=DEV)[:, None]
    j = f % max(1, res // 32)
    centre = 16.0 + 32.0 * j
    r = uniform(0.0, 1.0).sqrt()
    a0 = uniform(0.0, 2.0 * math.pi)
    theta = uniform(-5.0, 5.0) * (math.pi / 180.0)
    s = 2.0 + (res - 4.0) * torch.arange(n_points, dtype=F64, device=DEV)[None, :] / (n_points - 1)
    rho = torch.hypot(10.0 * r * torch.cos(a0), 2.5 * r * torch.sin(a0))
    alpha = a0 + s * torch.tan(theta) / rho.clamp_min(1.0)
    across = centre + 10.0 * r * torch.cos(alpha)
    phase = math.pi * (s - 16.0) / 32.0 + math.pi * j
    warp = f < n_fibers // 2
    p = torch.empty((n_fibers, n_points, 3), dtype=F64, device=DEV)
    p[..., 0] = torch.where(warp, s.expand_as(across), across)
    p[..., 1] = torch.where(warp, across, s.expand_as(across))
    p[..., 2] = res / 2.0 + torch.where(warp, 4.0, -4.0) * torch.cos(phase) + 2.5 * r * torch.sin(alpha)
    p += 0.3 * torch.randn(p.shape, dtype=F64, device=DEV, generator=gen)
    offsets = torch.arange(0, n_fibers * n_points + 1, n_points, dtype=torch.int64, device=DEV)
    p = torch.roll(turned(p, float(res), seed % 48, odd=True), 7 * seed % n_fibers, 0)
    return p.reshape(-1, 3).contiguous(), offsets


def generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def fabric(case, seed):
    pts, offsets = weave_points(case["fibers"], case["points"], case["log2_res"], generator(own_seed(case)), seed)
    return pts, offsets, Grid((0.0, 0.0, 0.0), float(1 << case["log2_res"]), case["log2_res"])


def patch_list(case, seed):
    """(points, offsets, grid) of every patch: fiber counts uniform in their logarithm, grids of
    256^3 to 1024^3."""
    gen = generator(own_seed(case))
    out = []
    for i in range(case["patches"]):
        # the spread of sizes is the case's, not the seed's: every seed builds as much
        t = (i + 0.5) / case["patches"]
        n = int(round(math.exp(math.log(case["low"]) + t * math.log(case["high"] / case["low"]))))
        l2 = 8 + (2 * i) % 3
        out.append(weave_points(n, 257, l2, gen, seed + i) + (Grid((0.0, 0.0, 0.0), float(1 << l2), l2),))
    return out


def fit_params(rows, seed):
    """Lobe factors near an isotropic start, one [rows, 12] tensor a level."""
    g = generator(seed + 1)
    base = torch.tensor([0.45, 0.0, 0.45, 0.0, 0.0, 0.45] * 2, dtype=torch.float32, device=DEV)
    return [base + 0.05 * torch.randn((n, 12), dtype=torch.float32, device=DEV, generator=g) for n in rows]


def code_inputs(case, seed):
    """Weights and moments of a fabric's leaf: one to four fiber pieces a voxel, some voxels only
    touched (weight 0)."""
    g = generator(seed)
    n = case["n"]
    w = torch.zeros(n, dtype=F64, device=DEV)
    S = torch.zeros((6, n), dtype=F64, device=DEV)
    pieces = torch.randint(0, 5, (n,), device=DEV, generator=g)
    for k in range(4):
        t = torch.randn((3, n), dtype=F64, device=DEV, generator=g)
        t /= t.norm(dim=0, keepdim=True)
        length = torch.rand(n, dtype=F64, device=DEV, generator=g) * (pieces > k)
        w += length
        S[:3] += length * (1.0 - t * t)
        S[3] -= length * t[0] * t[1]
        S[4] -= length * t[0] * t[2]
        S[5] -= length * t[1] * t[2]
    return w.float(), S.float().contiguous()


# ------------------------------------------------------------------------------------------------
# prepare and run
# ------------------------------------------------------------------------------------------------

def pyramid_plans(kind, grid, data, levels, K, offsets=None, radius=0.0):
    """The plans of one asset with its level buffers at their true sizes, as a program that
    rebuilds the asset keeps them."""
    plan = vx.VoxelizePlan(kind, grid, data, offsets=offsets, radius=radius)
    leaf = plan.run().check()
    sizes = [max(v.n, 1) for v in vx.LodPlan(grid, leaf, plan.stats[2:3], levels).run().check()[1:]]
    return plan, vx.LodPlan(grid, leaf, plan.stats[2:3], levels, K=K, iters=2, caps=sizes)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "call":
        tris, grid = sphere_mesh(case, seed)
        return {"case": case, "tris": tris, "grid": grid}
    if kind in ("sphere", "metal"):
        tris, grid = sphere_mesh(case, seed) if kind == "sphere" else metal_field(case, seed)
        plan, lod = pyramid_plans(0, grid, tris, case["levels"], case["K"])
        return {"case": case, "plan": plan, "lod": lod}
    if kind == "weave":
        pts, offsets, grid = fabric(case, seed)
        plan, lod = pyramid_plans(1, grid, pts, case["levels"], case["K"], offsets, RADIUS)
        state = {"case": case, "plan": plan, "lod": lod}
        if case["graph"]:
            torch.cuda.synchronize()
            state["graph"] = vx.capture(lambda s: (plan.run(s), lod.run(s)), torch.cuda.Stream())
        return state
    if kind == "patches":
        patches = [vx.Patch(g, p, o, RADIUS) for p, o, g in patch_list(case, seed)]
        return {"case": case, "batch": vx.BatchPlan(patches, K=case["K"], levels=case["levels"])}
    if kind == "fit":
        pts, offsets, grid = fabric(case, seed)
        plan = vx.FitPlan(grid, pts, offsets, RADIUS, lo=case["lo"], hi=case["hi"])
        params = fit_params([n for n, _ in plan.param_shapes()], seed)
        return {"case": case, "plan": plan, "pts": pts.requires_grad_(True),
                "params": [p.requires_grad_(True) for p in params]}
    if kind == "codes":
        w, S = code_inputs(case, seed)
        return {"case": case, "w": w, "S": S}
    if kind == "samples":
        if "window" in case:
            tris, grid = metal_field(case, seed)
            plan = vx.SamplePlan(0, grid, tris, N=case["N"])
        else:
            pts, offsets, grid = fabric(case, seed)
            plan = vx.SamplePlan(1, grid, pts, offsets=offsets, chords=case["chords"], per_chord=case["per_chord"])
        return {"case": case, "plan": plan}
    if kind == "occupancy":
        if "window" in case:
            data, grid = metal_field(case, seed)
            how = (0, grid, data, None, 0.0)
        else:
            data, offsets, grid = fabric(case, seed)
            how = (1, grid, data, offsets, RADIUS)
        plan, lod = pyramid_plans(how[0], grid, data, case["levels"], 1, how[3], how[4])
        plan.run()
        lod.run().check()
        return {"case": case, "plan": plan, "lod": lod,
                "occupancy": vx.OccupancyPlan(how[0], grid, data, lod, offsets=how[3], radius=how[4])}
    tris, grid = metal_field(case, seed)
    plan, lod = pyramid_plans(0, grid, tris, case["levels"], 1)
    plan.run()
    lod.run().check()
    return {"case": case, "plan": plan, "lod": lod,
            "sggxh": vx.SggxhPlan(lod, K=case["K"], samples=case["samples"])}


def voxel_outputs(v, n=None):
    n = v.cap if n is None else n
    out = {"keys": v.keys[:n], "count": v.count[:n], "w": v.w[:n], "S": v.S[:, :n]}
    if v.mask is not None:
        out["mask"] = v.mask[:n]
    return out


def lobe_outputs(lobes):
    return [{"nl": lb.nl, "w": lb.w, "S": lb.S} for lb in lobes]


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "call":
        leaf = vx.voxelize_triangles(state["tris"], state["grid"])
        levels, lobes = vx.build_lod(state["grid"], leaf, case["levels"], K=case["K"], return_lobes=True)
        return {"levels": [voxel_outputs(v, v.n) for v in levels],
                "lobes": [{"nl": b.nl[:b.n], "w": b.w[:, :b.n], "S": b.S[:, :, :b.n]} for b in lobes]}
    if kind in ("sphere", "metal", "weave"):
        plan, lod = state["plan"], state["lod"]
        if "graph" in state:
            state["graph"].replay(torch.cuda.current_stream())
        else:
            plan.run()
            lod.run()
        return {"levels": [voxel_outputs(v) for v in [plan.out] + lod.out], "lobes": lobe_outputs(lod.lobes)}
    if kind == "patches":
        batch = state["batch"].run()
        return {"levels": [voxel_outputs(v) for v in batch.out], "lobes": lobe_outputs(batch.lobes),
                "table": batch.patch_table}
    if kind == "fit":
        loss = vx.lobe_fit(state["plan"], state["pts"], state["params"])
        grads = torch.autograd.grad(loss, [state["pts"]] + state["params"])
        return {"loss": loss.detach(), "dpts": grads[0], "dparams": list(grads[1:])}
    if kind == "codes":
        lam, vec, code = vx.sggx_compact(state["w"], state["S"])
        return {"lam": lam, "vec": vec, "code": code, "S": vx.sggx_decode(code)}
    if kind == "samples":
        return voxel_outputs(state["plan"].run().out)
    if kind == "occupancy":
        return [{"mask": o.mask, "hits": o.hits} for o in state["occupancy"].run().occ]
    return lobe_outputs(state["sggxh"].run().lobes)


# ------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ------------------------------------------------------------------------------------------------

def _key_bytes(case):
    return 8 if case.get("log2_res", 12) > 10 or case["kind"] == "patches" else 4


def _surface(case):
    """(triangles, leaf voxels, pairs): about 1.3 leaf voxels per voxel of area; a triangle of
    area a voxels touches about 3 + 2.6 a of them."""
    if case["kind"] in ("sphere", "call"):
        n = 20 * 4 ** case["subdiv"]
        area = 4.0 * math.pi * (0.45 * (1 << case["log2_res"])) ** 2
        return n, 1.5 * area, 3.0 * n + 2.6 * area
    m = min(case["window"], 1 << case["log2_res"]) - 1
    return 2 * m * m, 1.3 * m * m, 8.9 * m * m


def _fibers(case):
    """(points, leaf voxels, pairs): a strand of radius 1/2 touches about 6.3 voxels per voxel of
    its length; strands of a yarn share voxels."""
    n, m, res = case["fibers"], case["points"], 1 << case["log2_res"]
    length = n * (res + 0.6 * m)
    area = 2.0 * min(n / 2.0, res / 32.0) * res * 21.0
    return n * m, min(4.0 * length, 8.0 * area), 6.3 * length


def _pyramid_bytes(case, leaf):
    kb, K = _key_bytes(case), case.get("K", 1)
    above = leaf * sum(0.28 ** L for L in range(1, case["levels"]))
    return (kb + 32) * leaf + (kb + 33 + (1 + 28 * K if K > 1 else 0)) * above


def work(case):
    """Inputs read once and outputs written once; operations: an exact box test and a clip per
    pair (about 300 for a triangle, 120 for a fiber), a handful per sample."""
    kind = case["kind"]
    if kind in ("call", "sphere", "metal"):
        n, leaf, pairs = _surface(case)
        return {"bytes": 36.0 * n + _pyramid_bytes(case, leaf), "flops": 300.0 * pairs}
    if kind == "weave":
        m, leaf, pairs = _fibers(case)
        return {"bytes": 12.0 * m + 8.0 * case["fibers"] + _pyramid_bytes(case, leaf), "flops": 120.0 * pairs}
    if kind == "patches":
        total = {"bytes": 0.0, "flops": 0.0}
        for i in range(case["patches"]):
            t = (i + 0.5) / case["patches"]
            n = math.exp(math.log(case["low"]) + t * math.log(case["high"] / case["low"]))
            c = {**case, "fibers": n, "points": 257, "log2_res": 8 + (2 * i) % 3}
            m, leaf, pairs = _fibers(c)
            total["bytes"] += 12.0 * m + _pyramid_bytes(c, leaf)
            total["flops"] += 120.0 * pairs
        return total
    if kind == "fit":
        m, leaf, pairs = _fibers(case)
        above = leaf * sum(0.22 ** L for L in range(case["lo"], case["hi"] + 1))
        # per direction: the target from the children below and two lobes, and their gradients
        return {"bytes": 24.0 * m + 96.0 * above, "flops": 240.0 * pairs + 128 * (40.0 * leaf + 80.0 * above)}
    if kind == "codes":
        return {"bytes": 112.0 * case["n"], "flops": 500.0 * case["n"]}
    if kind == "samples":
        if "window" in case:
            n, leaf, _ = _surface(case)
            smp = 0.55 * case["N"] * n
            return {"bytes": 36.0 * n + 40.0 * leaf, "flops": 60.0 * smp}
        m, leaf, _ = _fibers(case)
        smp = float(m * case["chords"] * case["per_chord"])
        return {"bytes": 12.0 * m + 40.0 * min(leaf, smp), "flops": 60.0 * smp}
    if kind == "occupancy":
        if "window" in case:
            n, leaf, pairs = _surface(case)
            inp = 36.0 * n
        else:
            n, leaf, pairs = _fibers(case)
            inp = 12.0 * n
        above = leaf * sum(0.28 ** L for L in range(1, case["levels"]))
        # per pair about 70 of its voxel's 512 sub-cells lie in the primitive's box
        return {"bytes": inp + (_key_bytes(case) + 72.0) * (leaf + above), "flops": 10.0 * 70 * pairs}
    n, leaf, _ = _surface(case)
    above = leaf * sum(0.28 ** L for L in range(1, case["levels"]))
    # a third of the coarse voxels hold more than K lobes, eight or so each; some 25 operations a sample
    return {"bytes": 28.0 * leaf + 29.0 * case["K"] * above, "flops": 25.0 * 8 * case["samples"] * above / 3}


# ------------------------------------------------------------------------------------------------
# the same in 64 bits: plain torch, none of the framework's code
# ------------------------------------------------------------------------------------------------

CHUNK = 4_000_000                    # candidates at a time


def spread3(v):
    x = v & 0x1FFFFF
    for shift, mask in ((32, 0x1F00000000FFFF), (16, 0x1F0000FF0000FF), (8, 0x100F00F00F00F00F),
                        (4, 0x10C30C30C30C30C3), (2, 0x1249249249249249)):
        x = (x | (x << shift)) & mask
    return x


def morton(v):
    return spread3(v[:, 0]) | (spread3(v[:, 1]) << 1) | (spread3(v[:, 2]) << 2)


def snap(p, grid):
    """Points on the integer lattice (as int64)."""
    b = torch.tensor(grid.bmin, dtype=F64, device=DEV)
    return torch.round((p.to(F64) - b) * (LATTICE / grid.extent)).to(torch.int64)


def candidates(mn, mx, s, res):
    """(primitive, voxel) of every closed box that meets a primitive's bounds, in chunks."""
    lo = (-torch.div(-mn, s, rounding_mode="floor") - 1).clamp_min(0)
    hi = torch.div(mx, s, rounding_mode="floor").clamp_max(res - 1)
    ext = (hi - lo + 1).clamp_min(0)
    cnt = ext.prod(1)
    ends = torch.cumsum(cnt, 0)
    total = int(ends[-1]) if len(ends) else 0
    p0 = 0
    done = 0
    while done < total:
        p1 = int(torch.searchsorted(ends, torch.tensor([done + CHUNK], device=DEV), right=True))
        p1 = max(p1, p0 + 1)
        c = cnt[p0:p1]
        prim = torch.repeat_interleave(torch.arange(p0, p1, device=DEV), c)
        i = torch.arange(len(prim), device=DEV) - torch.repeat_interleave(torch.cumsum(c, 0) - c, c)
        e, l = ext[prim], lo[prim]
        x = i % e[:, 0]
        y = (i // e[:, 0]) % e[:, 1]
        z = i // (e[:, 0] * e[:, 1])
        yield prim, l + torch.stack([x, y, z], 1)
        done = int(ends[p1 - 1])
        p0 = p1


def triangle_touch(q, v, s):
    """Separating-axis test of triangles [n, 3, 3] and closed boxes, in doubled integers."""
    t = 2 * q - (2 * v + 1)[:, None, :] * s                        # box centre at 0, half side s
    hit = ((t.min(1).values <= s) & (t.max(1).values >= -s)).all(1)
    e = torch.stack([q[:, 1] - q[:, 0], q[:, 2] - q[:, 1], q[:, 0] - q[:, 2]], 1)
    n = torch.linalg.cross(e[:, 0], e[:, 1])
    hit &= (n * t[:, 0]).sum(1).abs() <= s * n.abs().sum(1)
    for a in range(3):
        b, c = (a + 1) % 3, (a + 2) % 3
        for k in range(3):
            p = t[:, :, c] * e[:, k, b, None] - t[:, :, b] * e[:, k, c, None]
            r = s * (e[:, k, b].abs() + e[:, k, c].abs())
            hit &= (p.min(1).values <= r) & (p.max(1).values >= -r)
    return hit


def clipped_area(q, v, s):
    """Area (voxels^2) of triangles inside their boxes: the polygon cut plane by plane."""
    p = (q - v[:, None, :] * s).to(F64) / s                        # the box is [0, 1]^3
    flat = ((q.max(1).values == q.min(1).values) & (q[:, 0] == (v + 1) * s)).any(1)
    for a in range(3):
        for sign, off in ((1.0, 0.0), (-1.0, 1.0)):
            m = p.shape[1]
            d = sign * p[:, :, a] + off                            # inside: d >= 0
            d2, p2 = torch.roll(d, -1, 1), torch.roll(p, -1, 1)
            inside, cross = d >= 0, (d >= 0) != (d2 >= 0)
            t = torch.where(cross, d / torch.where(cross, d - d2, 1.0), 0.0)
            x = p + t[:, :, None] * (p2 - p)
            pts = torch.stack([p, x], 2).reshape(len(p), 2 * m, 3)
            keep = torch.stack([inside, cross], 2).reshape(len(p), 2 * m)
            pos = torch.cumsum(keep, 1) - 1
            cnt = keep.sum(1)
            out = torch.zeros((len(p), m + 2, 3), dtype=F64, device=DEV)
            idx = torch.where(keep, pos, m + 1).clamp_max(m + 1)
            out.scatter_(1, idx[:, :, None].expand(-1, -1, 3), pts)
            out = out[:, :m + 1]
            pad = torch.arange(m + 1, device=DEV)[None, :] >= cnt[:, None]
            p = torch.where(pad[:, :, None], out[:, :1], out)      # the first vertex again closes it
            p = torch.where((cnt > 0)[:, None, None], p, 0.0)
    w = p - p[:, :1]
    n = torch.linalg.cross(w[:, 1:-1], w[:, 2:]).sum(1)
    return torch.where(flat, 0.0, 0.5 * n.norm(dim=1))


def segment_touch(A, B, v, s, rho):
    """Whether segments come within rho of closed boxes: the least of a convex function of the
    segment parameter, bisected on its slope."""
    c = (A - v * s).to(F64) - 0.5 * s
    d = (B - A).to(F64)
    t0, t1 = torch.zeros(len(c), dtype=F64, device=DEV), torch.ones(len(c), dtype=F64, device=DEV)

    def gap(t):
        x = c + t[:, None] * d
        return torch.sign(x) * (x.abs() - 0.5 * s).clamp_min(0.0)

    for _ in range(56):
        t = 0.5 * (t0 + t1)
        up = (gap(t) * d).sum(1) < 0
        t0, t1 = torch.where(up, t, t0), torch.where(up, t1, t)
    best = torch.minimum((gap(t0) ** 2).sum(1), (gap(t1) ** 2).sum(1))
    for end in (0.0, 1.0):
        best = torch.minimum(best, (gap(torch.full_like(t0, end)) ** 2).sum(1))
    return best <= float(rho) ** 2


def clipped_length(a, d, v):
    """Length of a + t d, t in [0, 1] (voxel units), inside the half-open box at v."""
    moving = d != 0
    safe = torch.where(moving, d, torch.ones_like(d))
    u, w = (v - a) / safe, (v + 1 - a) / safe
    inside = (a >= v) & (a < v + 1)
    one, zero = torch.ones_like(a), torch.zeros_like(a)
    enter = torch.where(moving, torch.minimum(u, w), zero).max(1).values.clamp_min(0.0)
    leave = torch.where(moving, torch.maximum(u, w), one).min(1).values.clamp_max(1.0)
    ok = (moving | inside).all(1) & (leave > enter)
    return torch.where(ok, (leave - enter) * d.norm(dim=1), torch.zeros_like(enter))


def outer6(t):
    x, y, z = t.unbind(1)
    return torch.stack([x * x, y * y, z * z, x * y, x * z, y * z], 0)


IDENTITY6 = (1.0, 1.0, 1.0, 0.0, 0.0, 0.0)


def sums(key, w, S):
    """Sums of w and S by key, keys ascending."""
    uk, inv = torch.unique(key, return_inverse=True)
    return (uk, torch.zeros(len(uk), dtype=F64, device=DEV).index_add_(0, inv, w),
            torch.zeros((6, len(uk)), dtype=F64, device=DEV).index_add_(1, inv, S))


def exact_triangles(tris, grid):
    s, res = LATTICE >> grid.log2_res, 1 << grid.log2_res
    q = snap(tris, grid)
    n = torch.linalg.cross(q[:, 1] - q[:, 0], q[:, 2] - q[:, 0]).to(F64)
    n = n / n.norm(dim=1, keepdim=True).clamp_min(1e-300)
    got = []
    for prim, v in candidates(q.min(1).values, q.max(1).values, s, res):
        hit = triangle_touch(q[prim], v, s)
        prim, v = prim[hit], v[hit]
        w = clipped_area(q[prim], v, s)
        got.append(sums(morton(v), w, w * outer6(n[prim])))
    return sums(*(torch.cat(part, -1) for part in zip(*got)))


def fiber_pairs(pts, offsets, grid):
    """(first point, voxel) of every touching pair."""
    s, res = LATTICE >> grid.log2_res, 1 << grid.log2_res
    q = snap(pts, grid)
    first = torch.ones(len(q), dtype=torch.bool, device=DEV)
    first[offsets[1:] - 1] = False
    seg = first.nonzero()[:, 0]
    A, B = q[seg], q[seg + 1]
    rho = round(RADIUS * LATTICE / grid.extent)
    ps, vs = [], []
    for k, v in candidates(torch.minimum(A, B) - rho, torch.maximum(A, B) + rho, s, res):
        hit = segment_touch(A[k], B[k], v, s, rho)
        ps.append(seg[k[hit]])
        vs.append(v[hit])
    return torch.cat(ps), torch.cat(vs)


def fiber_terms(pts, p, v):
    """Clipped length and moment I - t t^T of every pair, points in voxel units."""
    a, d = pts[p], pts[p + 1] - pts[p]
    t = d / d.norm(dim=1, keepdim=True)
    return clipped_length(a, d, v.to(F64)), torch.tensor(IDENTITY6, dtype=F64, device=DEV)[:, None] - outer6(t)


def exact_fibers(pts, offsets, grid):
    s = LATTICE >> grid.log2_res
    p, v = fiber_pairs(pts, offsets, grid)
    w, M = fiber_terms(snap(pts, grid).to(F64) / s, p, v)
    return sums(morton(v), w, w * M)


def exact_levels(leaf, levels):
    out = [leaf]
    for _ in range(1, levels):
        k, w, S = out[-1]
        out.append(sums(k >> 3, w, S))
    return out


def level_values(levels):
    # keys, counts and masks are whole numbers
    return [{"keys": None, "count": None, "w": w, "S": S, "mask": None} for _, w, S in levels]


def exact_samples(case, seed):
    if "window" in case:
        tris, grid = metal_field(case, seed)
        g = tris.to(F64) * ((1 << grid.log2_res) / grid.extent)
        c = torch.linalg.cross(g[:, 1] - g[:, 0], g[:, 2] - g[:, 0])
        sq = (c * c).sum(1)
        N, top = case["N"], sq.max()
        n = torch.ones(len(sq), dtype=torch.int64, device=DEV)
        for k in range(2, N + 1):
            n += (k * k * top <= N * N * sq).long()
        t = torch.repeat_interleave(torch.arange(len(n), device=DEV), n)
        k = torch.arange(len(t), device=DEV) - torch.repeat_interleave(torch.cumsum(n, 0) - n, n)
        u1 = (k.to(F64) + 0.5) / n[t]
        u2 = sum(((k >> b) & 1).to(F64) * 2.0 ** -(b + 1) for b in range(8))
        low = u2 > u1
        b0 = torch.where(low, 0.5 * u1, u1 - 0.5 * u2)
        b1 = torch.where(low, u2 - 0.5 * u1, 0.5 * u2)
        x = (g[t, 2] + b1[:, None] * (g[t, 1] - g[t, 2])) + b0[:, None] * (g[t, 0] - g[t, 2])
        area = sq.sqrt()
        M = outer6(c / area[:, None].clamp_min(1e-300))[:, t]
        w = 0.5 * area[t] / n[t]
    else:
        pts, offsets, grid = fabric(case, seed)
        g = pts.to(F64) * ((1 << grid.log2_res) / grid.extent)
        m, per = case["chords"], case["per_chord"]
        g = g.reshape(case["fibers"], case["points"], 3)
        P = torch.cat([g[:, :1], g, g[:, -1:]], 1)
        P0, P1, P2, P3 = (P[:, i:i + case["points"] - 1].reshape(-1, 1, 3) for i in range(4))
        u = (torch.arange(m + 1, dtype=F64, device=DEV) / m)[None, :, None]
        curve = P1 + u * (0.5 * (P2 - P0) + u * ((P0 - 2.5 * P1 + 2.0 * P2 - 0.5 * P3) +
                                                   u * (0.5 * (P3 - P0) + 1.5 * (P1 - P2))))
        a, d = curve[:, :-1].reshape(-1, 1, 3), (curve[:, 1:] - curve[:, :-1]).reshape(-1, 1, 3)
        f = ((torch.arange(per, dtype=F64, device=DEV) + 0.5) / per)[None, :, None]
        x = (a + f * d).reshape(-1, 3)
        length = d[:, 0].norm(dim=1)
        tangent = d[:, 0] / length[:, None].clamp_min(1e-300)
        M = (torch.tensor(IDENTITY6, dtype=F64, device=DEV)[:, None] - outer6(tangent)).repeat_interleave(per, 1)
        w = (length / per).repeat_interleave(per)
    v = x.floor()
    ok = ((v >= 0) & (v < (1 << grid.log2_res))).all(1)
    _, W, S = sums(morton(v[ok].long()), w[ok], w[ok] * M[:, ok])
    return {"keys": None, "count": None, "w": W, "S": S}


def exact_fit(case, seed):
    pts, offsets, grid = fabric(case, seed)
    scale = (1 << grid.log2_res) / grid.extent
    x = pts.to(F64).requires_grad_(True)
    p, v = fiber_pairs(pts, offsets, grid)
    w, M = fiber_terms(x * scale, p, v)
    key, inv = torch.unique(morton(v), return_inverse=True)
    W = [torch.zeros(len(key), dtype=F64, device=DEV).index_add(0, inv, w)]
    S = [torch.zeros((6, len(key)), dtype=F64, device=DEV).index_add(1, inv, w * M)]
    parent = [None]
    for _ in range(case["hi"]):
        key, inv = torch.unique(key >> 3, return_inverse=True)
        parent.append(inv)
        W.append(torch.zeros(len(key), dtype=F64, device=DEV).index_add(0, inv, W[-1]))
        S.append(torch.zeros((6, len(key)), dtype=F64, device=DEV).index_add(1, inv, S[-1]))
    span = range(case["lo"], case["hi"] + 1)
    params = [q.to(F64).requires_grad_(True) for q in fit_params([len(W[L]) for L in span], seed)]
    k = torch.arange(128, dtype=F64)
    z = 1.0 - (2.0 * k + 1.0) / 128
    phi = k * (math.pi * (3.0 - math.sqrt(5.0)))
    r = torch.sqrt(1.0 - z * z)
    dirs = torch.stack([r * torch.cos(phi), r * torch.sin(phi), z], 1).float().to(DEV).to(F64)
    cW = [t.detach().requires_grad_(True) for t in W]
    cS = [t.detach().requires_grad_(True) for t in S]
    total = 0.0
    for L, q in zip(span, params):
        for d in dirs.split(16):
            quad = torch.cat([d * d, 2 * d[:, :1] * d[:, 1:2], 2 * d[:, :1] * d[:, 2:], 2 * d[:, 1:2] * d[:, 2:]], 1)
            area2 = cW[L - 1] * (quad @ cS[L - 1])
            ok = (area2 > 0) & (cW[L - 1] > 0)
            area = torch.where(ok, torch.where(ok, area2, 1.0).sqrt(), 0.0)
            tau = torch.zeros((len(d), len(W[L])), dtype=F64, device=DEV).index_add(1, parent[L], area)
            mass = torch.zeros(len(W[L]), dtype=F64, device=DEV).index_add(0, parent[L], cW[L - 1])
            has = mass > 0
            f = 0.0
            for j in (0, 6):
                l00, l10, l11, l20, l21, l22 = (q[:, j + i] for i in range(6))
                ox, oy, oz = (d[:, i:i + 1] for i in range(3))
                f = f + ((l00 * ox + l10 * oy + l20 * oz) ** 2 + (l11 * oy + l21 * oz) ** 2 + (l22 * oz) ** 2).sqrt()
            gap = torch.where(has, f - tau / torch.where(has, mass, 1.0), 0.0)
            loss = (gap * gap).sum() / len(dirs)
            loss.backward()
            total += float(loss.detach())
    made = [(t, g.grad) for t, g in zip(W + S, cW + cS) if g.grad is not None]
    torch.autograd.backward([t for t, _ in made], [g for _, g in made])
    return {"loss": torch.tensor(total, dtype=F64), "dpts": x.grad, "dparams": [q.grad for q in params]}


def exact_codes(case, seed):
    w, S = (t.to(F64) for t in code_inputs(case, seed))
    ok = w > 0
    A = torch.where(ok, S / torch.where(ok, w, 1.0), torch.tensor(IDENTITY6, dtype=F64, device=DEV)[:, None])
    m = [[A[0], A[3], A[4]], [A[3], A[1], A[5]], [A[4], A[5], A[2]]]
    for _ in range(8):                                             # cyclic Jacobi rotations
        for p, q in ((0, 1), (0, 2), (1, 2)):
            r = 3 - p - q
            h = 0.5 * (m[q][q] - m[p][p])
            apq = m[p][q]
            sign = torch.where(h < 0, -1.0, 1.0)
            t = torch.where(apq != 0, sign * apq / (h.abs() + torch.hypot(h, apq)).clamp_min(1e-300), 0.0)
            c = 1.0 / torch.sqrt(1.0 + t * t)
            s = t * c
            m[p][p], m[q][q] = m[p][p] - t * apq, m[q][q] + t * apq
            m[p][q] = m[q][p] = torch.zeros_like(apq)
            m[r][p], m[r][q] = c * m[r][p] - s * m[r][q], s * m[r][p] + c * m[r][q]
            m[p][r], m[q][r] = m[r][p], m[r][q]
    lam = torch.stack([m[0][0], m[1][1], m[2][2]]).sort(0, descending=True).values
    lam = torch.maximum(lam, 1e-3 * lam[:1])
    # eigenvectors of (nearly) equal eigenvalues have no one value; the code's bytes are whole numbers
    return {"lam": lam, "vec": None, "code": None, "S": None}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("call", "sphere", "metal"):
        tris, grid = metal_field(case, seed) if kind == "metal" else sphere_mesh(case, seed)
        # merged lobes come from decisions between near-equal costs: no one value in 64 bits
        return {"levels": level_values(exact_levels(exact_triangles(tris, grid), case["levels"])), "lobes": None}
    if kind == "weave":
        return {"levels": level_values(exact_levels(exact_fibers(*fabric(case, seed)), case["levels"])), "lobes": None}
    if kind == "patches":
        parts = [exact_fibers(p, o, g) for p, o, g in patch_list(case, seed)]
        parts = [(k | (i << 33), w, S) for i, (k, w, S) in enumerate(parts)]   # the patch above the voxel
        levels = [tuple(torch.cat(part, -1) for part in zip(*parts))]
        for _ in range(1, case["levels"]):
            k, w, S = levels[-1]
            up = (k >> 33 << 33) | ((k & ((1 << 33) - 1)) >> 3)
            levels.append(sums(up, w, S))
        return {"levels": level_values(levels), "lobes": None, "table": None}
    if kind == "fit":
        return exact_fit(case, seed)
    if kind == "codes":
        return exact_codes(case, seed)
    if kind == "samples":
        return exact_samples(case, seed)
    # occupancy masks and counts are whole numbers; the histogram reduction merges by counts of
    # pseudo-random samples
    return None
