"""The workloads this library's speed is judged on: grid builds of every size it is used at (one
small build, builds of the bench's scenes, batches, a served request), the build with false
intersections removed, ray casting over a built grid and the standalone radix sort.

Scenes follow the shapes of ``paper_2403_10647_amd/scenes.py`` (small, uniform, mixed, arch and
hairball soups) plus an indexed surface mesh, drawn on the GPU.  A case's triangles and bounds are
its own; the seed gives their order and, where the bounds are alike, which axis is which, so that
every seed has the same pair count and outputs of one shape.
"""
import math

import torch

from paper_2403_10647_amd import _lib as G


def listed():
    return [
        # a single small object: 4096 triangles on 32^3 cells, rebuilt each frame; launches and latency
        {"name": "small_4096", "do": "build", "scene": "small", "tris": 4096, "lam": 8.0},
        # one request of a build server that arrives alone: counted, sized, then built
        {"name": "request_alone", "do": "request", "grids": 1, "tmin": 14001, "tmax": 14001, "lam": 4.0},
        # a new scene of odd size built once: nothing prepared, so the count sizes fresh outputs
        {"name": "first_build_150k", "do": "first", "scene": "uniform", "tris": 150_001, "lam": 4.0},
        # an indexed surface mesh in file order (shared vertices, neighbours adjacent, most cells empty)
        {"name": "mesh_2m", "do": "build", "scene": "mesh", "tris": 2_000_000, "lam": 4.0},
        # many small and some very large triangles, a frame of a dynamic scene
        {"name": "mixed_1m", "do": "build", "scene": "mixed", "tris": 1_000_000, "lam": 4.0},
        # the headline workload: the 10M-triangle architectural scene
        {"name": "arch_10m", "do": "build", "scene": "arch", "tris": 10_000_000, "lam": 2.0},
        # long thin diagonal triangles: hundreds of cells per box
        {"name": "hairball_400k", "do": "build", "scene": "hairball", "tris": 400_000, "lam": 4.0},
        # a small batch, as the server forms under moderate load
        {"name": "batch_32", "do": "batch", "grids": 32, "tmin": 1000, "tmax": 200_000, "lam": 4.0},
        # the 512-grid batch of the benchmark
        {"name": "batch_512", "do": "batch", "grids": 512, "tmin": 1000, "tmax": 200_000, "lam": 4.0},
        # false intersections removed on the scene that needs it
        {"name": "culled_hairball_1m", "do": "culled", "scene": "hairball", "tris": 1_000_000, "lam": 4.0},
        # a million rays over the architectural grid
        {"name": "raycast_1m", "do": "raycast", "scene": "arch", "tris": 10_000_000, "lam": 2.0, "rays": 1_000_000},
        # the radix sort as a building block: 25-bit keys, as an arch build has
        {"name": "sort_16m", "do": "sort", "pairs": 16_000_003, "bits": 25},
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# the largest plain build drawn of each scene: each stays below the largest listed case's cost
_MOST = {"small": 65_536, "uniform": 8_000_000, "mesh": 8_000_000, "mixed": 1_500_000, "arch": 10_000_000,
         "hairball": 500_000}


def draw(rng):
    do = rng.choice(("build", "build", "build", "first", "request", "batch", "culled", "raycast", "sort"))
    lam = rng.choice((1.0, 2.0, 4.0, 8.0))
    if do in ("build", "first"):
        scene = rng.choice(("uniform", "mesh", "mixed", "arch", "hairball"))
        return {"do": do, "scene": scene, "tris": _logint(rng, 1000, _MOST[scene] // (2 if lam == 8.0 else 1)), "lam": lam}
    if do == "request":
        return {"do": do, "grids": rng.randint(1, 8), "tmin": 1000, "tmax": _logint(rng, 2000, 200_000), "lam": 4.0}
    if do == "batch":
        return {"do": do, "grids": _logint(rng, 2, 500), "tmin": 1000, "tmax": _logint(rng, 2000, 190_000), "lam": 4.0}
    if do == "culled":
        scene = rng.choice(("mixed", "arch", "hairball"))
        return {"do": do, "scene": scene, "tris": _logint(rng, 2000, 900_000), "lam": rng.choice((1.0, 2.0, 4.0))}
    if do == "raycast":
        return {"do": do, "scene": rng.choice(("uniform", "mesh", "arch")), "tris": _logint(rng, 2000, 2_000_000),
                "lam": rng.choice((2.0, 4.0)), "rays": _logint(rng, 1000, 500_000)}
    return {"do": do, "pairs": _logint(rng, 1000, 60_000_000), "bits": rng.randint(8, 32)}


# ---------------------------------------------------------------------------
# scenes
# ---------------------------------------------------------------------------
def _uniform(gen, shape, lo=0.0, hi=1.0):
    return torch.rand(shape, device="cuda", generator=gen) * (hi - lo) + lo


def _logu(gen, shape, lo, hi):
    return torch.exp(_uniform(gen, shape, math.log(lo), math.log(hi)))


def _sphere(gen, n, k=1):
    u = torch.randn((n, k, 3), device="cuda", generator=gen)
    return u / u.norm(dim=-1, keepdim=True).clamp_min(1e-12)


def _soup(scene, n, gen):
    """Vertices [n, 3, 3] of an unindexed soup."""
    if scene == "small":
        return _uniform(gen, (n, 1, 3)) + _uniform(gen, (n, 3, 3), -0.02, 0.02)
    if scene == "uniform":
        return _uniform(gen, (n, 1, 3), 0.0, 10.0) + _uniform(gen, (n, 3, 3), -0.05, 0.05)
    if scene == "mixed":
        big = n // 20
        off = _uniform(gen, (n, 3, 3), -1.0, 1.0)
        half = torch.full((n, 1, 3), 0.05, device="cuda")
        half[:big] = _logu(gen, (big, 1, 3), 0.05, 3.0)
        half = half[torch.randperm(n, device="cuda", generator=gen)]
        return _uniform(gen, (n, 1, 3), 0.0, 10.0) + off * half
    if scene == "hairball":
        a = _uniform(gen, (n, 1, 3), 0.0, 10.0)
        b = a + _logu(gen, (n, 1, 1), 0.3, 3.0) * _sphere(gen, n)
        c = b + _logu(gen, (n, 1, 1), 0.003, 0.03) * _sphere(gen, n)
        return torch.cat([a, b, c], 1)
    if scene == "arch":
        walls = max(2, n // 1000)
        box = torch.tensor([100.0, 10.0, 100.0], device="cuda")
        axis = torch.randint(0, 3, (walls,), device="cuda", generator=gen)
        p0 = _uniform(gen, (walls, 3)) * box
        p1 = torch.minimum(p0 + _logu(gen, (walls, 3), 1.0, 50.0), box)
        flat = torch.nn.functional.one_hot(axis, 3).bool()
        p1 = torch.where(flat, p0, p1)          # a rectangle on the plane of its axis
        first = torch.nn.functional.one_hot((axis == 0).long(), 3).bool()   # the first in-plane axis: y on x planes, else x
        q1, q3 = torch.where(first, p1, p0), torch.where(first, p0, p1)
        rect = torch.cat([torch.stack([p0, q1, p1], 1), torch.stack([p0, p1, q3], 1)])
        m = n - rect.shape[0]
        centre = _uniform(gen, (max(1, n // 5000), 3)) * box
        which = torch.randint(0, centre.shape[0], (m,), device="cuda", generator=gen)
        mid = centre[which] + 0.5 * torch.randn((m, 3), device="cuda", generator=gen)
        r = torch.exp(math.log(0.02) + 0.5 * torch.randn((m, 3, 1), device="cuda", generator=gen))
        soup = torch.cat([rect, mid[:, None, :] + r * _sphere(gen, m, 3)])
        return soup[torch.randperm(n, device="cuda", generator=gen)]
    raise ValueError(scene)


def _mesh(n, gen):
    """A bumpy closed surface: vertices [V, 3] and shared indices [n, 3], in rows of its grid."""
    rows = max(2, int(math.ceil(math.sqrt(n / 2.0))))
    u = torch.linspace(0.0, math.pi, rows + 1, device="cuda")[:, None].expand(rows + 1, rows + 1)
    v = torch.linspace(0.0, 2 * math.pi, rows + 1, device="cuda")[None, :].expand(rows + 1, rows + 1)
    wave = torch.randint(2, 9, (2,), device="cuda", generator=gen).float()
    r = 5.0 * (1.0 + 0.15 * torch.sin(wave[0] * u) * torch.cos(wave[1] * v))
    r = r * (1.0 + 0.2 / rows * torch.randn(r.shape, device="cuda", generator=gen))
    p = torch.stack([r * torch.sin(u) * torch.cos(v), r * torch.sin(u) * torch.sin(v), r * torch.cos(u)], -1).reshape(-1, 3)
    i = torch.arange(rows * rows, device="cuda")
    c = (i // rows) * (rows + 1) + i % rows
    quads = torch.stack([c, c + 1, c + rows + 2, c, c + rows + 2, c + rows + 1], 1).reshape(-1, 3)
    return p, quads[:n]


# bounds of each scene: all of it but a few clutter triangles, which the grid clamps
_BOUNDS = {"small": ((0.0,) * 3, (1.0,) * 3), "uniform": ((-0.05,) * 3, (10.05,) * 3), "mixed": ((-3.0,) * 3, (13.0,) * 3),
           "hairball": ((-3.03,) * 3, (13.03,) * 3), "mesh": ((-5.8,) * 3, (5.8,) * 3),
           "arch": ((-1.5, -1.5, -1.5), (101.5, 11.5, 101.5))}


def _resolution(lo, hi, n, lam, cap):
    k = (lam * max(n, 1) / math.prod(h - l for l, h in zip(lo, hi))) ** (1.0 / 3.0)
    return [min(cap, max(1, int(math.ceil((h - l) * k)))) for l, h in zip(lo, hi)]


def _input(scene, n, lam, seed, turn=True, key=0):
    """A scene of n triangles; the seed orders them and (turn) permutes the axes."""
    base, gen = _gen(n + 7919 * key), _gen(seed * 1000 + key)
    if scene == "mesh":
        p, t = _mesh(n, base)
        # file order, started anywhere
        t = t.roll(int(torch.randint(0, n, (1,), device="cuda", generator=gen)), 0)
    else:
        v = _soup(scene, n, base)
        p = v[torch.randperm(n, device="cuda", generator=gen)].reshape(3 * n, 3)
        t = torch.arange(3 * n, device="cuda").reshape(n, 3)
    if turn:
        axes = [[2, 1, 0], [0, 1, 2]] if scene == "arch" else [[0, 1, 2], [1, 2, 0], [2, 0, 1], [0, 2, 1], [1, 0, 2], [2, 1, 0]]
        p = p[:, axes[int(torch.randint(0, len(axes), (1,), device="cuda", generator=gen))]]
    lo, hi = _BOUNDS[scene]
    res = _resolution(lo, hi, n, lam, 1024 if scene == "arch" else 512)
    if scene == "small":
        res = [max(1, int(round((lam * n) ** (1.0 / 3.0))))] * 3
    return G.GridInput(p.T.contiguous(), t.to(torch.int32).contiguous(), list(lo), list(hi), res)


def _gen(seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return gen


def _grids(case, seed):
    n = case["grids"]
    u = torch.rand(n, device="cuda", generator=_gen(n)).tolist()
    lo, hi = math.log(case["tmin"]), math.log(case["tmax"])
    return [_input("mixed", int(math.exp(lo + (hi - lo) * x) + 0.5), case["lam"], seed, key=i) for i, x in enumerate(u)]


def _batch_outputs(inputs, caps):
    """The batch's outputs carved out of three tensors, each grid's part aligned to 256 bytes."""
    def carve(sizes):
        at = [0]
        for x in sizes:
            at.append(at[-1] + -(-max(x, 1) // 64) * 64)
        whole = torch.zeros(at[-1], dtype=torch.int32, device="cuda")
        return whole, [whole[o:o + max(x, 1)] for o, x in zip(at, sizes)]
    cells, c = carve(caps)
    objs, o = carve(caps)
    ranges, r = carve([2 * g.ncells for g in inputs])
    return [cells, objs, ranges], [G.GridResult(*x, 0) for x in zip(c, o, r)]


def _rays(g, n, gen):
    """70% from inside the box in any direction, 30% from outside towards a point inside."""
    lo, hi = torch.tensor(g.lo, device="cuda"), torch.tensor(g.hi, device="cuda")
    out = int(round(0.3 * n))
    inside = lo + _uniform(gen, (n, 3)) * (hi - lo)
    d = _sphere(gen, n)[:, 0]
    o = torch.where(torch.arange(n, device="cuda")[:, None] < out, (lo + hi) / 2 + d * (hi - lo).norm(), inside)
    target = lo + _uniform(gen, (n, 3)) * (hi - lo)
    d = torch.where(torch.arange(n, device="cuda")[:, None] < out, target - o, d)
    return torch.cat([o.T, d.T]).contiguous()


# ---------------------------------------------------------------------------
# the measured calls
# ---------------------------------------------------------------------------
def _outputs(r):
    return [r.cells[: r.npairs], r.objs[: r.npairs], r.ranges]


def prepare(case, seed):
    gen = _gen(seed)
    do = case["do"]
    st = {"do": do, "ws": G.Workspace()}
    if do == "sort":
        high = 1 << case["bits"]
        st["keys"] = torch.randint(0, high, (case["pairs"],), device="cuda", generator=gen).to(torch.int32)
        st["vals"] = torch.arange(case["pairs"], device="cuda", dtype=torch.int32)
        st["bits"] = case["bits"]
        return st
    if do in ("request", "batch"):
        inputs = _grids(case, seed)
        st["inputs"] = inputs
        if do == "batch":
            st["out"], outs = _batch_outputs(inputs, G.count_batched(inputs, st["ws"]))
            st["build"] = G.BatchedBuild(inputs, outs, st["ws"])
        else:
            n = len(inputs)
            # a server's slot: a workspace for the most pairs it admits, pinned staging and counts
            st["bytes"] = 1 << 30
            st["ws"].get(st["bytes"])
            st["staging"] = torch.empty(2 * int(G.lib().grid_batch_staging_size(n)), dtype=torch.uint8, pin_memory=True)
            st["counts"] = torch.zeros(n + 1, dtype=torch.int64, pin_memory=True)
        return st
    g = _input(case["scene"], case["tris"], case["lam"], seed, turn=do != "culled")
    st["g"] = g
    if do == "first":
        return st
    n, _ = G.count(g, st["ws"])
    if do == "culled":
        # the outputs hold the pairs kept, known to a program from its last frame
        kept = G.build_culled(g, n, ws=st["ws"])[0].npairs
        out = G.alloc_results([g], [kept])[0]
        st["build"] = G.CulledBuild(g, out, n, st["ws"])
        return st
    out = G.alloc_results([g], [n])[0]
    if do == "build":
        st["build"] = G.PlainBuild(g, out, st["ws"])
        return st
    st["grid"] = G.build(g, out=out, ws=st["ws"])
    st["rays"] = _rays(g, case["rays"], gen)
    return st


def run(st):
    do = st["do"]
    if do == "build":
        return _outputs(st["build"]())
    if do == "first":
        return _outputs(G.build(st["g"], ws=st["ws"]))
    if do == "batch":
        st["build"]()
        return st["out"]
    if do == "request":
        n = len(st["inputs"])
        G.count_batched_async(st["inputs"], st["ws"], st["bytes"], st["staging"], st["counts"])
        torch.cuda.current_stream().synchronize()   # the exact counts size the outputs
        caps = st["counts"].tolist()
        outs = G.alloc_results(st["inputs"], caps[:n])
        G.build_batched_counted(st["inputs"], outs, caps[:n], st["ws"], st["bytes"], st["staging"])
        return [t for r in outs for t in _outputs(r)]
    if do == "culled":
        r, _ = st["build"]()
        return _outputs(r)
    if do == "raycast":
        return list(G.raycast(st["g"], st["grid"], st["rays"]))
    keys, vals = st["keys"].clone(), st["vals"].clone()   # the sort works in place
    return list(G.sort_pairs(keys, vals, st["bits"], st["ws"]))


def work(case):
    """Bytes one pass cannot do without: every input read once, every output written once."""
    if case["do"] == "sort":
        return {"bytes": 16 * case["pairs"], "flops": 0}
    st = prepare(case, 0)
    inputs = st["inputs"] if "inputs" in st else [st["g"]]
    read = sum(4 * (g.verts.numel() + g.tris.numel()) for g in inputs)
    if case["do"] == "raycast":
        # the rays, their hits, and a scene of which each ray's walk sees a part: the rays alone are certain
        return {"bytes": 32 * case["rays"], "flops": 0}
    return {"bytes": read + sum(4 * t.numel() for t in run(st)), "flops": 0}


def exact(case, seed):
    """Every output is a whole number, but for the rays' hit distances, whose closest-hit search over
    all triangles in 64 bits takes far longer than the measurement allows."""
    return None
