"""Performance cases: whole calls of the library as a program that meshes point clouds makes
them, from a thousand points to thirty million.

A case names a `kind` and its sizes:

* cloud   - one triangulation on a context the program keeps: clear, insert (in `calls` calls),
            export of tetrahedra and neighbours
* noalloc - the entry point that allocates no device memory, into buffers the program holds
* batch   - independent clouds in one call, each exported on its own
* refine  - a triangulation refined by circumcentre insertion, its mesh and points exported

The library leaves the order of the exported rows open, so a pass brings them into one: each
tetrahedron's vertices ascending, the tetrahedra sorted.  Neighbours are returned in that
numbering up to 65536 points; beyond, they are exported with the tetrahedra, as a program that
walks the mesh has them, and the tetrahedra, which determine them, are returned.  How many there are
depends on the points, so results stand in buffers of a fixed size, unused places -1.
"""
import math

import numpy as np
import torch

from paper_1805_08831_amd import Triangulation, dt_get_tets, dt_get_tets_batch
from paper_1805_08831_amd.dt import dt_get_points, dt_refine, dt_triangulate_noalloc

SMALL = 65536  # indices below this pack four to an int64
TETS_PER_POINT = 7.0  # room for a cloud's tetrahedra (uniform clouds have up to 6.8 per point)
GAIN = {0.4: 5.9, 0.5: 3.1, 0.7: 1.4}  # final points per input point of a refinement, by spacing


def listed():
    return [
        # a mesh of a part or a molecule inside another program: host arrays in and out
        dict(name="host_1k", kind="cloud", points=1000, dist="uniform", buffers="host", calls=1, index_bits=0,
             adaptive=False),
        # a serving loop over small clouds that must not allocate
        dict(name="noalloc_4k", kind="noalloc", points=4099),
        # one cloud of the batch recipe's middle size, on its own
        dict(name="cloud_20k", kind="cloud", points=20011, dist="uniform", buffers="device", calls=1, index_bits=0,
             adaptive=False),
        # the largest cloud of the entry point that does not allocate
        dict(name="noalloc_64k", kind="noalloc", points=65536),
        # the benchmark's small configuration
        dict(name="cloud_100k", kind="cloud", points=100_000, dist="uniform", buffers="device", calls=1,
             index_bits=0, adaptive=False),
        # points that arrive in portions, the mesh kept between the calls
        dict(name="append_300k", kind="cloud", points=300_007, dist="uniform", buffers="device", calls=6,
             index_bits=0, adaptive=False),
        # 64-bit adjacency codes, the layout of the largest pools
        dict(name="wide_1m", kind="cloud", points=1_000_000, dist="uniform", buffers="device", calls=1,
             index_bits=64, adaptive=False),
        # the non-uniform recipe (lattice, clusters, thin shell): exact predicates, huge cavities
        dict(name="mix_1m", kind="cloud", points=1_000_000, dist="mix", buffers="device", calls=1, index_bits=0,
             adaptive=False),
        # clouds of log-uniform sizes in one call
        dict(name="batch_64", kind="batch", clouds=64, nmin=1000, nmax=200_000),
        # the refinement benchmark
        dict(name="refine_250k", kind="refine", points=250_000, spacing=0.4),
        # the headline benchmark
        dict(name="cloud_10m", kind="cloud", points=10_000_000, dist="uniform", buffers="device", calls=1,
             index_bits=0, adaptive=False),
        # a scan-sized cloud, memory-bound throughout
        dict(name="cloud_30m", kind="cloud", points=30_000_000, dist="uniform", buffers="device", calls=1,
             index_bits=0, adaptive=False),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["cloud", "cloud", "cloud", "append", "mix", "noalloc", "batch", "refine"])
    if kind == "noalloc":
        return dict(kind="noalloc", points=_log(rng, 200, SMALL))
    if kind == "batch":
        return dict(kind="batch", clouds=_log(rng, 4, 64), nmin=_log(rng, 200, 2000), nmax=_log(rng, 5000, 200_000))
    if kind == "refine":
        return dict(kind="refine", points=_log(rng, 5000, 250_000), spacing=rng.choice([0.4, 0.5, 0.7]))
    case = dict(kind="cloud", points=_log(rng, 500, 10_000_000), dist="uniform", buffers="device", calls=1,
                index_bits=rng.choice([0, 0, 0, 64]), adaptive=False)
    if kind == "append":
        case.update(points=_log(rng, 3000, 2_000_000), calls=rng.randint(2, 8))
    elif kind == "mix":
        case.update(points=_log(rng, 3000, 1_000_000), dist="mix", adaptive=rng.random() < 0.5)
    elif case["points"] < 20_000:
        case.update(buffers=rng.choice(["host", "device"]))
    return case


# ---------------------------------------------------------------- inputs


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _uniform(n, g):
    return torch.rand((n, 3), dtype=torch.float64, device="cuda", generator=g)


def _normal(n, k, g):
    return torch.randn((n, k), dtype=torch.float64, device="cuda", generator=g)


def _mix(n, g):
    """40 % distinct nodes of a dyadic lattice, 30 % in 50 rotated Gaussian clusters of unequal
    axes, 30 % within 1e-4 of the unit sphere, shuffled."""
    nl = 4 * n // 10
    nc = 3 * n // 10
    ns = n - nl - nc
    side = int(math.ceil((1.024 * nl) ** (1 / 3))) + 1
    nodes = torch.randperm(side ** 3, device="cuda", generator=g)[:nl]
    ijk = torch.stack([nodes // (side * side), nodes // side % side, nodes % side], dim=1).double()
    scale = 2.0 ** math.ceil(math.log2(3.2 * side))
    lattice = (2 * ijk - (side - 1)) / scale
    k = 50
    centres = _normal(k, 3, g)
    centres = 0.9 * centres / centres.norm(dim=1, keepdim=True) * _uniform(k, g)[:, :1] ** (1 / 3)
    sigma = torch.exp(math.log(0.002) + _uniform(k, g) * math.log(0.05 / 0.002))
    rot = torch.linalg.qr(_normal(3 * k, 3, g).view(k, 3, 3).cpu()).Q.cuda()
    own = torch.arange(nc, device="cuda") % k
    z = _normal(nc, 3, g) * sigma[own]
    clusters = centres[own] + (z[:, None, :] * rot[own]).sum(dim=2)
    d = _normal(ns, 3, g)
    shell = d / d.norm(dim=1, keepdim=True) * (1 + (2 * _uniform(ns, g)[:, :1] - 1) * 1e-4)
    pts = torch.cat([lattice, clusters, shell])
    return pts[torch.randperm(n, device="cuda", generator=g)].contiguous()


def _sizes(case):
    q = (torch.arange(case["clouds"], dtype=torch.float64) + 0.5) / case["clouds"]
    return torch.exp(math.log(case["nmin"]) + q * math.log(case["nmax"] / case["nmin"])).round().long()


def _clouds(case, g):
    """Points of all clouds and their offsets: sizes evenly spread in their logarithm and
    shuffled, each cloud uniform in its own axis-aligned box."""
    k = case["clouds"]
    sizes = _sizes(case).cuda()[torch.randperm(k, device="cuda", generator=g)]
    u = torch.rand((k, 7), dtype=torch.float64, device="cuda", generator=g)
    offsets = np.concatenate([[0], np.cumsum(sizes.cpu().numpy())]).astype(np.uint64)
    own = torch.repeat_interleave(torch.arange(k, device="cuda"), sizes)
    lo = -10 + 20 * u[:, 1:4]
    extent = torch.exp(math.log(0.1) + u[:, 4:7] * math.log(100.0))
    return (lo[own] + _uniform(int(offsets[-1]), g) * extent[own]).contiguous(), offsets


def _room(points):
    return int(TETS_PER_POINT * points) + 64


def prepare(case, seed):
    g = _generator(seed)
    # the library and torch work on one stream, so that buffers pass between them in order
    state = dict(case=case, stream=torch.cuda.Stream())
    stream = state["stream"].cuda_stream
    if case["kind"] == "noalloc":
        n = case["points"]
        state["xyz"] = _uniform(n, g)
        state["capacity"] = _room(n)
        state["tets"] = torch.empty((state["capacity"], 4), dtype=torch.int32, device="cuda")
        state["nbrs"] = torch.empty((state["capacity"], 4), dtype=torch.int64, device="cuda")
    elif case["kind"] == "batch":
        state["xyz"], state["offsets"] = _clouds(case, g)
        state["tri"] = Triangulation(stream=stream)
    elif case["kind"] == "refine":
        state["xyz"] = _uniform(case["points"], g)
        state["h"] = case["spacing"] * case["points"] ** (-1 / 3)
        state["tri"] = Triangulation(stream=stream)
    else:
        n = case["points"]
        xyz = _mix(n, g) if case["dist"] == "mix" else _uniform(n, g)
        parts = list(torch.tensor_split(xyz, case["calls"]))
        state["parts"] = [p.cpu().numpy() if case["buffers"] == "host" else p for p in parts]
        state["tri"] = Triangulation(stream=stream, index_bits=case["index_bits"], adaptive_curve=case["adaptive"])
    torch.cuda.synchronize()
    return state


# ---------------------------------------------------------------- passes


def _padded(x, rows):
    return torch.nn.functional.pad(x, (0, 0) * (x.dim() - 1) + (0, rows - len(x)), value=-1)


def _ordered_with_neighbours(tets, nbrs, rows):
    """Tetrahedra of at most 65536 vertices as one int64 each, ascending, and the neighbour
    across the facet opposite each vertex, vertices ascending, in that numbering."""
    v, column = torch.sort(tets, dim=1)
    v = v.long()
    key, order = torch.sort((v[:, 0] << 48) | (v[:, 1] << 32) | (v[:, 2] << 16) | v[:, 3])
    place = torch.empty_like(order)
    place[order] = torch.arange(len(order), device=order.device)
    across = nbrs.gather(1, column)[order]
    across = torch.where(across >= 0, place[across.clamp(min=0)], across)
    return _padded(key, rows), _padded(across, rows)


def _ordered(tets, rows):
    """Tetrahedra as two packed int64 each (vertices ascending), in the order of a mixed key,
    which one sort establishes for any number of them."""
    a, b, c, d = tets.t().contiguous().unbind(0)
    a, b = torch.minimum(a, b), torch.maximum(a, b)
    c, d = torch.minimum(c, d), torch.maximum(c, d)
    a, c = torch.minimum(a, c), torch.maximum(a, c)
    b, d = torch.minimum(b, d), torch.maximum(b, d)
    b, c = torch.minimum(b, c), torch.maximum(b, c)
    hi = (a.long() << 32) | b
    lo = (c.long() << 32) | d
    order = torch.sort(hi * -7046029254386353131 + lo * -4417276706812531889).indices
    return _padded(hi[order], rows), _padded(lo[order], rows)


def _run_cloud(state):
    case, tri = state["case"], state["tri"]
    tri.clear()
    for part in state["parts"]:
        tri.insert(part)
    tets, nbrs = tri.tets(device_tensors=case["buffers"] == "device")
    if case["buffers"] == "host":
        tets, nbrs = torch.from_numpy(tets.view(np.int32)), torch.from_numpy(nbrs)
    if case["points"] <= SMALL:
        return _ordered_with_neighbours(tets, nbrs, _room(case["points"]))
    return _ordered(tets, _room(case["points"]))


def _run_noalloc(state):
    count = dt_triangulate_noalloc(state["xyz"], state["tets"], state["nbrs"], state["capacity"],
                                   stream=state["stream"].cuda_stream)
    return _ordered_with_neighbours(state["tets"][:count], state["nbrs"][:count], state["capacity"])


def _run_batch(state):
    tri, offsets = state["tri"], state["offsets"]
    tri.clear()
    tri.insert_batch(state["xyz"], offsets)
    total = tri.num_tets()
    tets = torch.empty((total, 4), dtype=torch.int32, device="cuda")
    nbrs = torch.empty((total, 4), dtype=torch.int64, device="cuda")
    row = 0
    for k in range(len(offsets) - 1):
        count = dt_get_tets_batch(tri.ctx, k)
        dt_get_tets_batch(tri.ctx, k, tets[row:], nbrs[row:], total - row)
        tets[row:row + count] += int(offsets[k])  # one numbering for all clouds
        row += count
    return _ordered(tets, _room(int(offsets[-1])))


def _run_refine(state):
    tri = state["tri"]
    tri.clear()
    tri.insert(state["xyz"])
    added, steps = dt_refine(tri.ctx, state["h"])
    count = dt_get_tets(tri.ctx)
    tets = torch.empty((count, 4), dtype=torch.int32, device="cuda")
    nbrs = torch.empty((count, 4), dtype=torch.int64, device="cuda")
    dt_get_tets(tri.ctx, tets, nbrs, count)
    final = int(1.2 * GAIN[state["case"]["spacing"]] * state["case"]["points"])
    points, passes = dt_get_points(tri.ctx), np.full((100, 2), -1, dtype=np.int64)
    passes[:len(steps)] = steps
    return (_ordered(tets, _room(final)), np.pad(points, ((0, final - len(points)), (0, 0)), constant_values=-1.0),
            passes, added)


def run(state):
    run_kind = {"cloud": _run_cloud, "noalloc": _run_noalloc, "batch": _run_batch, "refine": _run_refine}
    with torch.cuda.stream(state["stream"]):
        return run_kind[state["case"]["kind"]](state)


# ---------------------------------------------------------------- accounting


def work(case):
    """Bytes: coordinates read, tetrahedra and neighbours written once.  Operations: the
    insphere tests of an average insertion (its 20 cavity tetrahedra and the 27 around them,
    each about 100 operations)."""
    n = int(_sizes(case).sum()) if case["kind"] == "batch" else case["points"]
    final = GAIN[case["spacing"]] * n if case["kind"] == "refine" else n
    written = 48 * 6.7 * final + (24 * final if case["kind"] == "refine" else 0)
    return {"bytes": 24 * n + written, "flops": final * 47 * 100.0}


def exact(case, seed):
    # the outputs are whole numbers, which are compared as they are; the refinement's points
    # are the result of thousands of dependent decisions with no short form in plain torch
    return None
