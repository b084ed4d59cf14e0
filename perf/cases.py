"""Workloads of the geometric-search library, for timing and for comparing two versions' results.

Each case is one pass of a user's program through the public entry points, with the inputs already
on the GPU.  Most passes build their index first: a simulation or a clustering rebuilds its tree
whenever its points move, and then asks it one or a few questions.  The smallest case keeps its tree,
as a service answering small requests does.

All inputs are float32 (the library's one coordinate type), drawn on the GPU from the seed.  Radii
come from the closed forms of the package's input module for a target mean number of neighbours.
"""
import math

import numpy as np
import torch

import paper_2507_23700_amd as ax
from paper_2507_23700_amd import inputs

DEV = "cuda"
COMPONENTS, SIGMA = 64, 0.02  # Gaussian mixture
NOISE = 1e-3                  # radial noise of the hollow sphere
RAY_BOX = 1.4                 # longest edge of a ray-traced box in units of the mean spacing n^(-1/3)


def listed():
    return [
        # a service that answers requests of a thousand points against a small tree it keeps
        {"name": "knn_request", "op": "request", "dist": "cube", "dim": 3, "n": 20_000, "m": 1_000, "k": 10},
        # a small simulation step, bound by latency: every kind of radius and nearest query once
        {"name": "step_20k", "op": "step", "dist": "cube", "dim": 3, "n": 20_000, "m": 20_000, "k": 10, "mean": 10.0},
        # the paper's headline: all results of a radius search stored
        {"name": "radius_cube_10m", "op": "radius", "dist": "cube", "dim": 3, "n": 10_000_000, "m": 10_000_000,
         "mean": 10.0},
        # neighbourhoods of fixed size (normals, local densities) of a large cloud
        {"name": "knn_cube_10m", "op": "knn", "dist": "cube", "dim": 3, "n": 10_000_000, "m": 10_000_000, "k": 16},
        # counting in a callback, on a surface, an odd number of points
        {"name": "count_shell_5m", "op": "count", "dist": "shell", "dim": 3, "n": 5_000_011, "m": 4_999_999,
         "mean": 10.0},
        # feature space: clustered points in six dimensions, nearest and radius with per-match distances
        {"name": "knn_gmm6_2m", "op": "knn", "dist": "gmm", "dim": 6, "n": 2_000_000, "m": 2_000_000, "k": 8},
        {"name": "radius_gmm6_500k", "op": "distances", "dist": "gmm", "dim": 6, "n": 500_009, "m": 500_009,
         "mean": 20.0},
        # density-based clustering of a large cloud, a radius for ten neighbours
        {"name": "dbscan_cube_5m", "op": "dbscan", "dist": "cube", "dim": 3, "n": 5_000_000, "mean": 10.0,
         "min_pts": 10},
        # rays through a scene of small boxes: what each meets first, and everything it meets
        {"name": "rays_boxes_1m", "op": "rays", "dist": "boxes", "dim": 3, "n": 1_000_000, "m": 300_000, "k": 1},
        # broad-phase collision of boxes in the plane
        {"name": "overlap_boxes2d_1m", "op": "overlap", "dist": "boxes", "dim": 2, "n": 1_000_003, "m": 1_000_003,
         "mean": 8.0},
        # many uneven trees, batches of queries aimed at them: build, distance sums, nearest
        {"name": "forest_32", "op": "forest", "trees": 32, "lo": 10_000, "hi": 1_000_000, "batches": 512,
         "blo": 100, "bhi": 100_000, "k": 8},
        # a training loss over pairs of clouds: forward and backward
        {"name": "chamfer_128", "op": "chamfer", "pairs": 128, "lo": 1_000, "hi": 32_768},
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))))) | rng.randrange(2)

    op = rng.choice(["request", "step", "radius", "radius", "knn", "knn", "count", "knn6", "distances", "dbscan",
                     "rays", "overlap", "forest", "chamfer"])
    mean = round(rng.uniform(4.0, 16.0), 2)
    flat = rng.choice([2, 3, 3, 3])
    dist = "cube" if flat == 2 else rng.choice(["cube", "shell"])
    if op == "request":
        return {"op": op, "dist": dist, "dim": flat, "n": size(2_000, 1_000_000), "m": size(64, 20_000),
                "k": rng.choice([1, 4, 8, 10, 16, 32])}
    if op == "step":
        return {"op": op, "dist": dist, "dim": flat, "n": size(1_000, 500_000), "m": size(1_000, 500_000),
                "k": rng.choice([4, 8, 10, 16]), "mean": mean}
    if op == "radius":
        n = size(20_000, 8_000_000)
        return {"op": op, "dist": dist, "dim": flat, "n": n, "m": min(n, size(20_000, 8_000_000)), "mean": mean}
    if op == "knn":
        n = size(20_000, 8_000_000)
        return {"op": op, "dist": dist, "dim": flat, "n": n, "m": min(n, size(20_000, 8_000_000)),
                "k": rng.choice([1, 4, 8, 10, 16])}
    if op == "count":
        return {"op": op, "dist": dist, "dim": flat, "n": size(20_000, 8_000_000), "m": size(20_000, 8_000_000),
                "mean": mean}
    if op == "knn6":
        return {"op": "knn", "dist": "gmm", "dim": 6, "n": size(20_000, 2_000_000), "m": size(20_000, 1_500_000),
                "k": rng.choice([4, 8, 16])}
    if op == "distances":
        six = rng.random() < 0.5
        n = size(20_000, 500_000 if six else 4_000_000)
        return {"op": op, "dist": "gmm" if six else "cube", "dim": 6 if six else 3, "n": n, "m": n,
                "mean": round(rng.uniform(8.0, 20.0), 2)}
    if op == "dbscan":
        return {"op": op, "dist": dist, "dim": flat, "n": size(20_000, 5_000_000), "mean": mean,
                "min_pts": rng.choice([2, 5, 10])}
    if op == "rays":
        return {"op": op, "dist": "boxes", "dim": 3, "n": size(20_000, 1_000_000), "m": size(10_000, 250_000),
                "k": rng.choice([1, 4])}
    if op == "overlap":
        return {"op": op, "dist": "boxes", "dim": rng.choice([2, 3]), "n": size(20_000, 1_000_000),
                "m": size(20_000, 1_000_000), "mean": round(rng.uniform(2.0, 8.0), 2)}
    if op == "forest":
        return {"op": op, "trees": rng.randrange(4, 33), "lo": 2_000, "hi": size(20_000, 800_000),
                "batches": rng.randrange(16, 513), "blo": 50, "bhi": size(1_000, 80_000), "k": rng.choice([4, 8])}
    return {"op": "chamfer", "pairs": rng.randrange(2, 129), "lo": 500, "hi": size(2_000, 30_000)}


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------

def _generator(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1_000_003 + stream) & 0x7FFFFFFFFFFFFFFF)
    return g


def _cube(n, dim, g):
    return torch.rand((n, dim), generator=g, device=DEV)


def _shell(n, g):
    v = torch.randn((n, 3), generator=g, device=DEV, dtype=torch.float64)
    v /= v.norm(dim=1, keepdim=True)
    v *= 1.0 + NOISE * torch.randn((n, 1), generator=g, device=DEV, dtype=torch.float64)
    return v.float()


def _points(case, n, seed, stream):
    g = _generator(seed, stream)
    if case["dist"] == "cube":
        return _cube(n, case["dim"], g)
    if case["dist"] == "shell":
        return _shell(n, g)
    centres = torch.rand((COMPONENTS, case["dim"]), generator=_generator(seed, 99), device=DEV)
    which = torch.randint(0, COMPONENTS, (n,), generator=g, device=DEV)
    return centres[which] + SIGMA * torch.randn((n, case["dim"]), generator=g, device=DEV)


def _radius(case):
    n, mean = case["n"], case["mean"]
    if case["dist"] == "cube":
        return float(inputs.radius_cube(n, mean, case["dim"]))
    if case["dist"] == "shell":
        return float(inputs.radius_shell(n, mean, NOISE))
    return float(inputs.radius_gmm(n, min(mean, n / (2.0 * COMPONENTS)), case["dim"], COMPONENTS, SIGMA))


def _boxes(n, dim, edge, seed, stream):
    """Boxes in the unit cube with edges uniform in (0, edge)."""
    g = _generator(seed, stream)
    lo = torch.rand((n, dim), generator=g, device=DEV)
    return torch.stack([lo, lo + edge * torch.rand((n, dim), generator=g, device=DEV)], dim=1).contiguous()


def _log_sizes(rng, lo, hi, count):
    return np.rint(np.exp(rng.uniform(math.log(lo), math.log(max(hi, lo + 1)), count))).astype(np.int64)


def _forest_sizes(case):
    """Tree sizes, batch sizes and the tree each batch searches: of the case, not of the seed, so that
    passes on other inputs cost the same."""
    rng = np.random.default_rng([case["trees"], case["batches"], case["hi"], case["bhi"]])
    tree = _log_sizes(rng, case["lo"], case["hi"], case["trees"])
    batch = _log_sizes(rng, case["blo"], case["bhi"], case["batches"])
    return tree, batch, rng.integers(0, case["trees"], case["batches"]).astype(np.int32)


def _offsets(sizes):
    return np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)


def _chamfer_sizes(case):
    rng = np.random.default_rng([case["pairs"], case["lo"], case["hi"]])
    return (rng.integers(case["lo"], case["hi"] + 1, case["pairs"]),
            rng.integers(case["lo"], case["hi"] + 1, case["pairs"]))


def _clouds(sizes, seed, stream):
    """Noisy surfaces of random ellipsoids, one per cloud, packed."""
    g = _generator(seed, stream)
    total = int(sizes.sum())
    axes = 0.5 + torch.rand((len(sizes), 3), generator=g, device=DEV, dtype=torch.float64)
    rot = torch.linalg.qr(torch.randn((len(sizes), 3, 3), generator=g, device=DEV, dtype=torch.float64).cpu())[0].to(DEV)
    of = torch.repeat_interleave(torch.arange(len(sizes), device=DEV), torch.from_numpy(sizes).to(DEV),
                                 output_size=total)
    u = torch.randn((total, 3), generator=g, device=DEV, dtype=torch.float64)
    u /= u.norm(dim=1, keepdim=True)
    u = (u * axes[of]).unsqueeze(1)
    p = (u * rot[of]).sum(dim=2)
    p += 0.01 * torch.randn((total, 3), generator=g, device=DEV, dtype=torch.float64)
    return p.float()


def _matches(case):
    """About how many matches a search of this case has."""
    if case["op"] == "rays":  # a random ray crosses about 0.6 of the cube; a box shows it 3/8 edge^2 on average
        return 0.6 * 0.375 * RAY_BOX ** 2 * case["n"] ** (1.0 / 3.0) * case["m"]
    return case.get("mean", 0.0) * case["m"]


def _room(case):
    return torch.full((int(1.5 * _matches(case)) + 65_536,), -1, dtype=torch.int32, device=DEV)


def prepare(case, seed):
    op = case["op"]
    if op == "chamfer":
        na, nb = _chamfer_sizes(case)
        return {"op": op, "a": _clouds(na, seed, 1).requires_grad_(), "a_off": _offsets(na),
                "b": _clouds(nb, seed, 2).requires_grad_(), "b_off": _offsets(nb),
                "grad": 0.5 + torch.rand(case["pairs"], generator=_generator(seed, 3), device=DEV)}
    if op == "forest":
        tree, batch, aim = _forest_sizes(case)
        values = [_cube(int(n), 3, _generator(seed, 100 + t)) if t % 2 == 0 else _shell(int(n), _generator(seed, 100 + t))
                  for t, n in enumerate(tree)]
        queries = [_cube(int(n), 3, _generator(seed, 10_000 + b)) if aim[b] % 2 == 0
                   else _shell(int(n), _generator(seed, 10_000 + b)) for b, n in enumerate(batch)]
        radius = np.array([inputs.radius_cube(int(n), 10.0) if t % 2 == 0 else inputs.radius_shell(int(n), 10.0)
                           for t, n in enumerate(tree)], dtype=np.float32)
        return {"op": op, "values": torch.cat(values), "tree_offsets": _offsets(tree), "queries": torch.cat(queries),
                "batch_offsets": torch.from_numpy(_offsets(batch)).to(DEV),
                "batch_tree": torch.from_numpy(aim).to(DEV), "batch_radius": torch.from_numpy(radius[aim]).to(DEV),
                "k": case["k"]}
    if op == "rays":
        g = _generator(seed, 2)
        origin = torch.rand((case["m"], case["dim"]), generator=g, device=DEV)
        direction = torch.randn((case["m"], case["dim"]), generator=g, device=DEV)
        return {"op": op, "values": _boxes(case["n"], case["dim"], RAY_BOX * case["n"] ** (-1.0 / case["dim"]), seed, 1),
                "rays": torch.stack([origin, direction], dim=1).contiguous(), "k": case["k"], "room": _room(case)}
    if op == "overlap":
        # two boxes with edges uniform in (0, e) overlap per dimension with probability about e
        edge = (case["mean"] / case["n"]) ** (1.0 / case["dim"])
        return {"op": op, "values": _boxes(case["n"], case["dim"], edge, seed, 1),
                "queries": _boxes(case["m"], case["dim"], edge, seed, 2), "room": _room(case)}
    state = {"op": op, "values": _points(case, case["n"], seed, 1)}
    if op == "dbscan":
        state.update(radius=_radius(case), min_pts=case["min_pts"])
        return state
    state["queries"] = _points(case, case["m"], seed, 2)
    state["k"] = case.get("k")
    if "mean" in case:
        state["radius"] = _radius(case)
    if op in ("step", "radius", "distances"):
        state["room"] = _room(case)
    if op == "distances":
        state["room_d2"] = _room(case).float()
    if op == "request":
        state["bvh"] = ax.BVH(state["values"])
    return state


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------

def _keep(room, rows):
    """The rows of a search copied into the program's own array, sized once for every pass (the number of
    matches changes from input to input); the rest of the array stays as it is."""
    n = min(rows.numel(), room.numel())
    room[:n].copy_(rows[:n])
    return room


def run(s):
    op = s["op"]
    if op == "request":
        d2, idx = s["bvh"].knn(s["queries"], s["k"])
        return {"d2": d2, "index": idx}
    if op == "chamfer":
        loss = ax.chamfer(s["a"], s["a_off"], s["b"], s["b_off"])
        ga, gb = torch.autograd.grad(loss, (s["a"], s["b"]), s["grad"])
        return {"loss": loss, "grad_a": ga, "grad_b": gb}
    if op == "forest":
        f = ax.arborx_forest_build(s["values"], s["tree_offsets"])
        count, total = f.reduce(s["queries"], s["batch_offsets"], s["batch_tree"], s["batch_radius"])
        d2, idx = f.knn(s["queries"], s["batch_offsets"], s["batch_tree"], s["k"])
        return {"count": count, "sum": total, "d2": d2, "index": idx}
    if op in ("rays", "overlap"):
        bvh = ax.BVH(s["values"], ax.BOXES)
        if op == "overlap":
            offsets, idx = bvh.intersects(s["queries"])
            return {"offsets": offsets, "index": _keep(s["room"], idx)}
        t, first = bvh.ray_nearest(s["rays"], s["k"])
        offsets, idx = ax.arborx_query_ray_intersect(bvh.tree, s["rays"])
        return {"t": t, "first": first, "offsets": offsets, "index": _keep(s["room"], idx)}
    bvh = ax.BVH(s["values"])
    if op == "dbscan":
        return {"labels": bvh.dbscan(s["radius"], s["min_pts"])}
    if op == "radius":
        offsets, idx = bvh.spatial(s["queries"], s["radius"])
        return {"offsets": offsets, "index": _keep(s["room"], idx)}
    if op == "distances":
        offsets, idx, d2 = bvh.spatial_with_distances(s["queries"], s["radius"])
        return {"offsets": offsets, "index": _keep(s["room"], idx), "d2": _keep(s["room_d2"], d2)}
    if op == "count":
        count = bvh.count(s["queries"], s["radius"])
        same, total = bvh.count_sumdist(s["queries"], s["radius"])
        near = bvh.count_up_to(s["queries"], s["radius"], 4)
        return {"count": count, "again": same, "sum": total, "near": near}
    if op == "knn":
        d2, idx = bvh.knn(s["queries"], s["k"])
        return {"d2": d2, "index": idx}
    offsets, idx = bvh.spatial(s["queries"], s["radius"])  # step
    count, total = bvh.count_sumdist(s["queries"], s["radius"])
    d2, near = bvh.knn(s["queries"], s["k"])
    return {"offsets": offsets, "index": _keep(s["room"], idx), "count": count, "sum": total, "d2": d2, "near": near}


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------

def work(case):
    op = case["op"]
    if op == "chamfer":
        na, nb = _chamfer_sizes(case)
        n = int(na.sum() + nb.sum())
        # points, gradients and the neighbours that the backward reads; a nearest distance and a gradient per point
        return {"bytes": 12 * n + 12 * n + 4 * n, "flops": 8 * n + 12 * n}
    if op == "forest":
        tree, batch, _ = _forest_sizes(case)
        n, m = int(tree.sum()), int(batch.sum())
        return {"bytes": 12 * n + 12 * m + 12 * m + 8 * case["k"] * m, "flops": 8 * m * (10 + case["k"])}
    dim, n, m = case["dim"], case["n"], case.get("m", case["n"])
    pair = 3 * dim - 1  # operations of one squared distance
    if op == "rays":
        met = _matches(case)
        return {"bytes": 8 * dim * n + 8 * dim * m + 8 * case["k"] * m + 8 * m + 4 * met, "flops": 6 * dim * met}
    if op == "overlap":
        met = _matches(case)
        return {"bytes": 8 * dim * n + 8 * dim * m + 8 * m + 4 * met, "flops": 2 * dim * met}
    points = 4 * dim * n
    if op == "dbscan":
        return {"bytes": points + 4 * n, "flops": pair * n * case["mean"] / 2}
    queries = 4 * dim * m
    met = case.get("mean", 0.0) * m
    near = 8 * case.get("k", 0) * m
    if op == "request":
        return {"bytes": points + queries + near, "flops": pair * m * case["k"]}
    if op == "radius":
        return {"bytes": points + queries + 8 * m + 4 * met, "flops": pair * met}
    if op == "distances":
        return {"bytes": points + queries + 8 * m + 8 * met, "flops": pair * met}
    if op == "count":
        return {"bytes": points + queries + 20 * m, "flops": pair * met}
    if op == "knn":
        return {"bytes": points + queries + near, "flops": pair * m * case["k"]}
    return {"bytes": points + queries + 8 * m + 4 * met + 12 * m + near, "flops": pair * (2 * met + m * case["k"])}


# --------------------------------------------------------------------------
# the computed numbers in 64 bits
# --------------------------------------------------------------------------

def _nearest(values, queries, k, budget=1 << 27):
    """(k smallest squared distances, their indices) per query, by brute force in float64."""
    v, q = values.double(), queries.double()
    k2 = min(k, v.shape[0])
    d2 = torch.full((q.shape[0], k), math.inf, dtype=torch.float64, device=q.device)
    idx = torch.full((q.shape[0], k), -1, dtype=torch.int64, device=q.device)
    rows = max(1, budget // max(1, v.shape[0]))
    for i in range(0, q.shape[0], rows):
        d = torch.zeros((min(rows, q.shape[0] - i), v.shape[0]), dtype=torch.float64, device=q.device)
        for c in range(v.shape[1]):
            d += (q[i:i + rows, c, None] - v[None, :, c]).square_()
        if k2 == 1:
            a, b = d.min(dim=1, keepdim=True)
        else:
            a, b = torch.topk(d, k2, dim=1, largest=False, sorted=True)
        d2[i:i + rows, :k2], idx[i:i + rows, :k2] = a, b
    return d2, idx


def exact(case, seed):
    op = case["op"]
    if op == "chamfer":
        s = prepare(case, seed)
        a, b = s["a"].detach(), s["b"].detach()
        ga, gb = torch.zeros(a.shape, dtype=torch.float64, device=DEV), torch.zeros(b.shape, dtype=torch.float64, device=DEV)
        loss = torch.zeros(case["pairs"], dtype=torch.float64, device=DEV)
        for p in range(case["pairs"]):
            sa, sb = slice(*map(int, s["a_off"][p:p + 2])), slice(*map(int, s["b_off"][p:p + 2]))
            x, y, g = a[sa].double(), b[sb].double(), 2.0 * s["grad"][p].double()
            d_ab, i_ab = _nearest(b[sb], a[sa], 1)
            d_ba, i_ba = _nearest(a[sa], b[sb], 1)
            i_ab, i_ba = i_ab[:, 0], i_ba[:, 0]
            loss[p] = d_ab.sum() + d_ba.sum()
            ga[sa] += g * (x - y[i_ab])
            gb[sb] += g * (y - x[i_ba])
            ga[sa].index_add_(0, i_ba, g * (x[i_ba] - y))
            gb[sb].index_add_(0, i_ab, g * (y[i_ab] - x))
        return {"loss": loss, "grad_a": ga, "grad_b": gb}
    if op in ("request", "step", "knn") and case["n"] * case["m"] <= 20_000_000_000:
        s = prepare({**case, "op": "knn"}, seed)
        d2, _ = _nearest(s["values"], s["queries"], case["k"])
        rest = {"offsets": None, "index": None, "count": None, "sum": None, "near": None} if op == "step" else {"index": None}
        return {"d2": d2, **rest}
    return None
