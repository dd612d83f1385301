"""The work a user of this package has it do, as cases that can be timed.

Five kinds of pass, each through the public entry points of paper_2305_04359_amd.binding:
  search   a batch of k-NN queries on a built graph (`noalloc`: the serving entry point, which
           allocates nothing); the graph is what the user's program holds before the call
  build    a flat graph over points in device memory
  stream   a flat graph over the first points, then the rest in a few unequal additions
  layered  a layered index over the points, then a batch of queries on it
  cluster  a graph by the clustering-based builder
Points and queries are drawn on the GPU from the distributions of workloads.py: uint8 rows from
1,024 centres with about a third zeros, int8 rows from 1,024 Gaussians, float32 unit vectors from
512 centres on the sphere, whose inner-product queries come from centres turned by 30 degrees.
"""
from __future__ import annotations

import math

import torch

from paper_2305_04359_amd import binding as A

TYPES = {"u8": torch.uint8, "i8": torch.int8, "f32": torch.float32}
METRICS = {"l2": A.L2SQ, "ip": A.MIPS}


def listed():
    return [
        # one question of an interactive user: latency alone
        {"name": "search-1", "op": "search", "dtype": "u8", "metric": "l2", "n": 1_000_000, "d": 128, "R": 64, "Lb": 128,
         "nq": 1, "k": 10, "L": 40, "eps": -1.0, "noalloc": True},
        # a small serving batch on padded int8 rows, with the (1 + eps) rule
        {"name": "search-37", "op": "search", "dtype": "i8", "metric": "l2", "n": 200_003, "d": 100, "R": 32, "Lb": 64,
         "nq": 37, "k": 10, "L": 60, "eps": 0.1, "noalloc": False},
        # the 10,000-query batch at the beam of recall 0.95
        {"name": "search-10k", "op": "search", "dtype": "u8", "metric": "l2", "n": 1_000_000, "d": 128, "R": 64, "Lb": 128,
         "nq": 10_000, "k": 10, "L": 16, "eps": -1.0, "noalloc": False},
        # inner-product queries on float rows, at the beam of recall 0.90
        {"name": "search-f32", "op": "search", "dtype": "f32", "metric": "ip", "n": 1_000_000, "d": 200, "R": 64, "Lb": 128,
         "nq": 10_000, "k": 10, "L": 50, "eps": -1.0, "noalloc": False},
        # a stream of queries with a wide beam on a graph well beyond the caches
        {"name": "search-100k", "op": "search", "dtype": "u8", "metric": "l2", "n": 5_000_000, "d": 128, "R": 64, "Lb": 96,
         "nq": 100_000, "k": 10, "L": 100, "eps": -1.0, "noalloc": False},
        # a small collection: dozens of short batches
        {"name": "build-10k", "op": "build", "dtype": "u8", "metric": "l2", "n": 10_000, "d": 128, "R": 32, "L": 64},
        # a million points, the usual benchmark
        {"name": "build-1m", "op": "build", "dtype": "u8", "metric": "l2", "n": 1_000_000, "d": 128, "R": 64, "L": 128},
        # int8 rows of a size that is no multiple of 16 bytes, an odd number of them
        {"name": "build-i8", "op": "build", "dtype": "i8", "metric": "l2", "n": 150_001, "d": 100, "R": 64, "L": 128},
        # float embeddings under the inner product: the largest build
        {"name": "build-f32", "op": "build", "dtype": "f32", "metric": "ip", "n": 1_000_000, "d": 200, "R": 64, "L": 128},
        # a collection that grows after its first build
        {"name": "stream", "op": "stream", "dtype": "u8", "metric": "l2", "n": 100_001, "d": 128, "R": 64, "L": 128,
         "first": 40_000, "adds": 4},
        # the layered index, built and asked
        {"name": "layered", "op": "layered", "dtype": "u8", "metric": "l2", "n": 200_000, "d": 128, "m": 32, "efc": 128,
         "nq": 10_000, "k": 10, "L": 13},
        # the clustering-based builder at the paper's parameters
        {"name": "cluster", "op": "cluster", "dtype": "u8", "metric": "l2", "n": 1_000_000, "d": 128, "T": 30, "Ls": 1000,
         "s": 3, "l": 10, "R": 64},
    ]


def _between(rng, lo, hi):
    """A whole number of [lo, hi], even over the logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(["search", "search", "search", "search", "build", "build", "build", "stream", "layered", "cluster"])
    dtype = rng.choice(["u8", "u8", "i8", "f32"])
    metric = rng.choice(["l2", "ip"]) if dtype == "f32" else "l2"
    if dtype == "f32":
        d = 4 * _between(rng, 12, 50)
    else:
        d = rng.choice([128, 128, _between(rng, 48, 128)]) if op == "cluster" else rng.choice([128, 128, _between(rng, 48, 256)])
    esz = 4 if dtype == "f32" else 1
    case = {"op": op, "dtype": dtype, "metric": metric, "d": d}
    if op == "search":
        room = 640_000_000 // (d * esz)  # points
        case.update(n=_between(rng, 10_000, min(room, 5_000_000)), R=rng.choice([32, 48, 64]), Lb=rng.choice([64, 96]))
        case.update(nq=_between(rng, 1, 100_000), k=rng.choice([1, 10, 10, 100]))
        # (queries x beam stays below the largest listed search, a fifth of it for float rows)
        most = (10_000_000 if esz == 1 else 2_000_000) // case["nq"]
        case["L"] = max(case["k"], min(_between(rng, 10, 200), most))
        if case["L"] * case["nq"] > 10_000_000 // esz:
            case.update(k=10, L=max(10, most))
        case["eps"] = rng.choice([-1.0, -1.0, 0.05, 0.25])
        case["noalloc"] = case["nq"] <= 1000 and rng.random() < 0.5
    elif op in ("build", "stream"):
        room = 128_000_000 // (d * esz)
        case.update(n=_between(rng, 2_000, min(room, 1_000_000) if op == "build" else min(room, 200_000)))
        case.update(R=rng.choice([32, 48, 64]), L=rng.choice([64, 96, 128]))
        if op == "stream":
            case.update(first=max(500, int(case["n"] * rng.uniform(0.3, 0.9))), adds=rng.randint(1, 5))
    elif op == "layered":
        room = 40_000_000 // (d * esz)
        case.update(n=_between(rng, 2_000, min(room, 300_000)), m=rng.choice([16, 24, 32]), efc=rng.choice([64, 96, 128]))
        case.update(nq=_between(rng, 1, 20_000), k=10, L=rng.randint(10, 60))
    else:
        room = 128_000_000 // (d * esz)
        case.update(n=_between(rng, 5_000, min(room, 1_000_000) if esz == 1 else min(room, 200_000)))
        case.update(T=rng.randint(5, 30), Ls=rng.choice([250, 500, 1000]), s=3, l=rng.choice([8, 10]), R=rng.choice([32, 64]))
    return case


def _rows(g, n, d, centers, sigma, lo, hi, dtype):
    k = torch.randint(centers.shape[0], (n,), generator=g, device="cuda")
    out = torch.empty((n, d), dtype=dtype, device="cuda")
    for a in range(0, n, 1 << 20):
        kk = k[a:a + (1 << 20)]
        x = centers[kk].add_(torch.randn((kk.shape[0], d), generator=g, device="cuda"), alpha=sigma)
        out[a:a + (1 << 20)] = x.round_().clamp_(lo, hi).to(dtype)
    return out


def _unit(x):
    return x.div_(x.norm(dim=1, keepdim=True))


def _unit_rows(g, n, d, centers, sigma):
    k = torch.randint(centers.shape[0], (n,), generator=g, device="cuda")
    return _unit(centers[k].add_(torch.randn((n, d), generator=g, device="cuda"), alpha=sigma))


def _inputs(case, seed):
    """(points, queries) on the GPU; queries is None where the case asks nothing."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    n, d, nq = case["n"], case["d"], case.get("nq", 0)
    if case["dtype"] == "f32":
        c = _unit(torch.randn((512, d), generator=g, device="cuda"))
        sigma = 0.05 * math.sqrt(200.0 / d)  # per coordinate: the same angle whatever d
        points = _unit_rows(g, n, d, c, sigma)
        if case["metric"] == "ip":  # queries out of the points' distribution
            u = torch.randn((512, d), generator=g, device="cuda")
            u = _unit(u - (u * c).sum(1, keepdim=True) * c)
            c = math.cos(math.pi / 6) * c + math.sin(math.pi / 6) * u
        return points, _unit_rows(g, nq, d, c, sigma) if nq else None
    if case["dtype"] == "u8":
        c = 40.0 * torch.empty((1024, d), device="cuda").exponential_(1.0, generator=g) - 16.0
        sigma, lo, hi = 12.0, 0, 255
    else:
        c = 40.0 * torch.randn((1024, d), generator=g, device="cuda")
        sigma, lo, hi = 25.0, -127, 127
    t = TYPES[case["dtype"]]
    return _rows(g, n, d, c, sigma, lo, hi, t), _rows(g, nq, d, c, sigma, lo, hi, t) if nq else None


def _alpha(case):
    return 1.0 if case["metric"] == "ip" else 1.2


def prepare(case, seed):
    points, queries = _inputs(case, seed)
    s = {"case": case, "seed": seed, "points": points, "queries": queries}
    if case["op"] == "search":
        s["graph"] = A.ann_build(points, case["R"], case["Lb"], _alpha(case), seed=seed, metric=METRICS[case["metric"]])
        if case["noalloc"]:  # a serving loop brings its own results
            s["ids"] = torch.empty((case["nq"], case["k"]), dtype=torch.int32, device="cuda")
            s["dists"] = torch.empty((case["nq"], case["k"]), device="cuda",
                                     dtype=torch.float32 if case["dtype"] == "f32" else torch.int32)
    return s


class _Rows:
    """A graph's adjacency rows in device memory, as torch takes them; keeps the graph alive."""

    def __init__(self, graph):
        gi = graph.info()
        self.graph = graph
        self.__cuda_array_interface__ = {"shape": (int(gi.n), int(gi.R)), "typestr": "<i4", "version": 2,
                                         "data": (int(A.lib().ann_graph_device_rows(graph.handle)), False)}


def _graph_out(graph):
    """The rows, where they lie, and the start vertex."""
    return [torch.as_tensor(_Rows(graph), device="cuda"), int(graph.info().start)]


def run(s):
    c, pts, qs, seed = s["case"], s["points"], s["queries"], s["seed"]
    metric, alpha = METRICS[c["metric"]], _alpha(c)
    if c["op"] == "search":
        if c["noalloc"]:
            A.ann_search_noalloc(s["graph"], pts, qs, c["k"], c["L"], s["ids"], s["dists"], eps=c["eps"])
            return [s["ids"], s["dists"]]
        if c["eps"] >= 0:
            return list(A.ann_search_eps(s["graph"], pts, qs, c["k"], c["L"], c["eps"]))
        return list(A.ann_search(s["graph"], pts, qs, c["k"], c["L"]))
    if c["op"] == "build":
        return _graph_out(A.ann_build(pts, c["R"], c["L"], alpha, seed=seed, metric=metric))
    if c["op"] == "stream":
        g = A.ann_build(pts[:c["first"]], c["R"], c["L"], alpha, seed=seed, metric=metric)
        left, w = c["n"] - c["first"], c["adds"] * (c["adds"] + 1) // 2
        at = c["first"]
        for i in range(c["adds"]):  # additions of 1, 2, 3, ... shares of what is left
            at = c["n"] if i + 1 == c["adds"] else at + left * (i + 1) // w
            A.ann_insert_points(g, pts[:at], c["L"], alpha, seed=seed + i)
        return _graph_out(g)
    if c["op"] == "layered":
        h = A.ann_hnsw_build(pts, c["m"], c["efc"], alpha, seed=seed, metric=metric)
        return list(A.ann_hnsw_search(h, pts, qs, c["k"], c["L"]))
    return _graph_out(A.ann_hcnng_build(pts, c["T"], c["Ls"], c["s"], c["l"], c["R"], alpha, seed=seed, metric=metric))


def work(case):
    """Bytes: points and queries read once, rows and results written (or, for a search, the rows
    and vectors it has to visit read) once.  Operations: two per element of every distance that
    cannot be left out.  A greedy search with beam L expands a little over L vertices and meets,
    for each, about 8 (beams of 100) to 24 (beams of 10) vertices it has not met before."""
    n, d = case["n"], case["d"]
    vec = d * (4 if case["dtype"] == "f32" else 1)

    def searches(count, L, R):  # (bytes gathered, distances taken)
        hops = L + 6
        met = hops * max(8.0, 28.0 - 9.0 * math.log10(L))
        return count * (hops * 4 * R + met * vec), count * met

    op = case["op"]
    if op == "search":
        gathered, dist = searches(case["nq"], case["L"], case["R"])
        return {"bytes": min(gathered, n * (vec + 4 * case["R"])) + case["nq"] * (vec + 8 * case["k"]), "flops": 2.0 * d * dist}
    if op in ("build", "stream"):
        _, dist = searches(n, case["L"], case["R"])
        return {"bytes": n * (vec + 4 * case["R"]), "flops": 2.0 * d * (dist + n * case["R"] ** 2 / 2)}
    if op == "layered":
        _, dist = searches(n, case["efc"], 2 * case["m"])
        _, more = searches(case["nq"], case["L"], 2 * case["m"])
        return {"bytes": n * (vec + 8 * case["m"]) + case["nq"] * (vec + 8 * case["k"]),
                "flops": 2.0 * d * (dist + more + n * (2 * case["m"]) ** 2 / 2)}
    # every point against its leaf, and against two pivots on each level above it
    levels = max(1.0, math.log2(n / case["Ls"]))
    return {"bytes": n * (vec + 4 * case["R"]), "flops": 2.0 * d * n * case["T"] * (case["Ls"] / 2 + 2 * levels)}


def tolerance(case):
    """Integer rows: everything is whole numbers, decided under one total order.  Float rows: fp32
    sums, so two nearly equal candidates may change places and with one of them the rest of a
    row, of a result list or (in the cluster trees) of a leaf.  Measured with the sums in another
    order (the columns of points and queries permuted): up to 1e-3 of a search's ids differ (and,
    where a query ends elsewhere, its distances: 6e-3 of all in the 2-norm, 0.6 for one), 7e-5 of
    a graph's entries, 1.3e-2 of a clustering-based graph's."""
    if case["dtype"] != "f32":
        return "exact"
    if case["op"] in ("build", "stream"):
        return {"rel": 1e-5, "differ": 1e-3}
    if case["op"] == "cluster":
        return {"rel": 1e-5, "differ": 1e-2}
    return {"rel": 2e-2, "max": 0.99, "differ": 5e-3}
