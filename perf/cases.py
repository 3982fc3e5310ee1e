"""Performance cases of the rope-LBVH library.

Each case is one piece of work that a program using the library has it do,
through the package's public functions (``build``,
``query_count`` and ``query_fill``, ``query_first``, ``build_batched``, the
batched count and fill), with the library's default knobs.  The program
keeps its workspaces, a buffer for the hits (grown when a count exceeds it)
and, where it rebuilds the same scene size again and again, the tree's
arrays; everything else a call needs is part of the pass.

Sizes and distributions are those of ``workloads``: uniform points, the
clustered boxes, spheres of a given expected neighbour number, query boxes,
rays and segments aimed at the boxes, batches of scenes of log-uniform size
and the serving requests.  Inputs are drawn on the GPU from the seed.
"""

import math
import random

import torch

import paper_2402_00665_amd as lb

DEV = "cuda"
MEAN_SIDE = math.exp(-7.0 + 0.125)   # of a clustered box: lognormal(-7, 0.5)
NODE = 32


def listed():
    return [
        # the smallest request of the serving stream: a thousand points,
        # where only launches and latency count
        dict(name="build_1k", do="build", prims="uniform", n=1000, bits=63),
        # the small build that a program repeats every frame
        dict(name="build_16k", do="build", prims="uniform", n=16384, bits=30),
        # ... and its queries
        dict(name="spheres_1k_on_16k", do="query", prims="uniform", n=16384, bits=30, q="spheres",
             m=1024, neighbours=0.55),
        # one serving request at the middle of its size range, odd sized:
        # build and query in one call
        dict(name="request_63k", do="request", prims="uniform", n=63241, bits=63, q="spheres",
             m=10000, neighbours=8.0),
        # an ordinary scene of boxes, odd sized, with the long codes
        dict(name="build_boxes_1m", do="build", prims="clustered", n=1000003, bits=63),
        # the two large builds: points with long codes, boxes with short
        # codes (many equal)
        dict(name="build_points_8m", do="build", prims="uniform", n=1 << 23, bits=63),
        dict(name="build_boxes_16m", do="build", prims="clustered", n=1 << 24, bits=30),
        # neighbour search: light, even queries
        dict(name="spheres_1m_on_8m", do="query", prims="uniform", n=1 << 23, bits=63, q="spheres",
             m=1 << 20, neighbours=16.0),
        # overlap queries: most hit nothing, a few hit 10^4 and more
        dict(name="boxes_1m_on_16m", do="query", prims="clustered", n=1 << 24, bits=30, q="boxes",
             m=1 << 20, side=0.01),
        # ray casting: the first box each ray meets
        dict(name="rays_1m_on_16m", do="rays_first", prims="clustered", n=1 << 24, bits=30, m=1 << 20),
        # all the boxes that short segments meet: hundreds of hits each
        dict(name="segments_1m_on_16m", do="query", prims="clustered", n=1 << 24, bits=30,
             q="segments", m=1 << 20, length=0.002),
        # thousands of scenes built together, and their queries together
        dict(name="scenes_4096", do="batch", prims="uniform", scenes=4096, least=32, most=65536,
             bits=63, m=64, radius=0.05),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    """One more case: sizes log-uniform over the ranges of the listed ones."""
    do = rng.choice(["build", "build", "query", "query", "query", "rays_first", "request", "batch"])
    bits = rng.choice([30, 63])
    if do == "batch":
        return dict(do="batch", prims=rng.choice(["uniform", "uniform", "clustered"]),
                    scenes=_log_int(rng, 2, 4000), least=32, most=_log_int(rng, 500, 65536), bits=bits,
                    m=_log_int(rng, 1, 64), radius=0.05)
    if do == "request":
        return dict(do="request", prims="uniform", n=_log_int(rng, 1000, 4000000), bits=63, q="spheres",
                    m=10000, neighbours=8.0)
    prims = rng.choice(["uniform", "clustered", "hollow"])
    if do == "rays_first":
        prims = "clustered"
    n = _log_int(rng, 1000, 1 << 24 if prims == "clustered" else 1 << 23)
    case = dict(do=do, prims=prims, n=n, bits=bits)
    if do == "build":
        return case
    case["m"] = _log_int(rng, 64, 1 << 20)
    if do == "query":
        q = rng.choice(["spheres", "boxes", "segments"] if prims == "clustered" else ["spheres", "boxes"])
        case["q"] = q
        if q == "segments":
            case["length"] = round(rng.uniform(0.0005, 0.002), 5)
        elif prims == "clustered":
            case["side"] = round(rng.uniform(0.002, 0.015), 5)
        else:
            case["neighbours"] = round(math.exp(rng.uniform(math.log(0.5), math.log(32.0))), 2)
    return case


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _uniform(n, width, g):
    return torch.rand((n, width), generator=g, device=DEV)


def _clustered(n, g, components=64, sigma=0.005):
    """Boxes around the points of a Gaussian mixture, lognormal sides."""
    means = torch.rand((components, 3), generator=g, device=DEV, dtype=torch.float64)
    comp = torch.randint(0, components, (n,), generator=g, device=DEV)
    c = means[comp]
    del comp
    c += torch.randn((n, 3), generator=g, device=DEV, dtype=torch.float64) * sigma
    c.clamp_(0.0, 1.0 - 2.0 ** -24)
    half = 0.5 * torch.exp(-7.0 + 0.5 * torch.randn((n, 3), generator=g, device=DEV, dtype=torch.float64))
    out = torch.empty((n, 6), device=DEV)
    out[:, :3] = c - half
    out[:, 3:] = c + half
    return out


def _hollow(n, g):
    """Points on the faces of the unit cube, point k on face k mod 6."""
    p = _uniform(n, 3, g)
    k = torch.arange(n, device=DEV)
    p[k, (k % 6) // 2] = (k % 2).to(torch.float32)
    return p


def _prims(case, g):
    return {"uniform": lambda: _uniform(case["n"], 3, g), "hollow": lambda: _hollow(case["n"], g),
            "clustered": lambda: _clustered(case["n"], g)}[case["prims"]]()


def _in_boxes(boxes, m, g):
    """m points, each uniform inside a box drawn uniformly."""
    pick = boxes[torch.randint(0, boxes.shape[0], (m,), generator=g, device=DEV)].double()
    u = torch.rand((m, 3), generator=g, device=DEV, dtype=torch.float64)
    return pick[:, :3] + u * (pick[:, 3:] - pick[:, :3])


def _rays(boxes, m, g):
    """From origins uniform in the unit cube through a point of a random box, [0, +inf)."""
    o = torch.rand((m, 3), generator=g, device=DEV, dtype=torch.float64)
    q = torch.zeros((m, 8), device=DEV)
    q[:, :3] = o
    q[:, 4:7] = _in_boxes(boxes, m, g) - o
    q[:, 7] = math.inf
    return q


def _segments(boxes, m, length, g):
    """From a point of a random box, uniform direction, [0, 1]."""
    u = torch.randn((m, 3), generator=g, device=DEV, dtype=torch.float64)
    q = torch.zeros((m, 8), device=DEV)
    q[:, :3] = _in_boxes(boxes, m, g)
    q[:, 4:7] = length * u / u.norm(dim=1, keepdim=True)
    q[:, 7] = 1.0
    return q


def _extent(case):
    """Radius of the spheres of a case."""
    if "neighbours" in case:
        return (case["neighbours"] / (case["n"] * 4.0 * math.pi / 3.0)) ** (1.0 / 3.0)
    return 0.5 * case["side"]


def _queries(case, prims, g):
    m, q = case["m"], case["q"]
    if q == "segments":
        return _segments(prims, m, case["length"], g)
    c = torch.rand((m, 3), generator=g, device=DEV)
    r = _extent(case)
    if q == "spheres":
        return torch.cat([c, torch.full((m, 1), r, device=DEV)], 1)
    return torch.cat([c - r, c + r], 1)


def _sizes(case):
    """Scene sizes of a batch: part of the case, whatever the seed."""
    r = random.Random(case["scenes"] * 65537 + case["most"])
    lo, hi = math.log(case["least"]), math.log(case["most"])
    return [int(math.exp(r.uniform(lo, hi))) for _ in range(case["scenes"])]


QKIND = {"spheres": lb.SPHERES, "boxes": lb.QBOXES, "segments": lb.RAYS}


def _hit_buffer(size):
    return torch.zeros(int(size) + 1024, dtype=torch.int32, device=DEV)


def prepare(case, seed):
    g = _gen(seed)
    s = {"do": case["do"], "bits": case["bits"], "ws": lb.Workspace(DEV), "qws": lb.Workspace(DEV)}
    if case["do"] == "batch":
        sizes = _sizes(case)
        s["max_scene"] = case["most"]
        seg = torch.zeros(len(sizes) + 1, dtype=torch.int64)
        seg[1:] = torch.cumsum(torch.tensor(sizes, dtype=torch.int64), 0)
        total = int(seg[-1])
        s["prims"] = _clustered(total, g) if case["prims"] == "clustered" else _uniform(total, 3, g)
        s["seg"] = seg.to(DEV)
        s["batch"] = lb.alloc_batch(s["seg"], case["bits"], case["most"], DEV, total_n=total)
        s["batch"].nodes.zero_()   # two slots a primitive, one of which a scene leaves unused
        m = case["m"] * case["scenes"]
        s["queries"] = torch.cat([_uniform(m, 3, g), torch.full((m, 1), case["radius"], device=DEV)], 1)
        s["qseg"] = torch.arange(case["scenes"] + 1, device=DEV) * case["m"]
        s["hits"] = _hit_buffer(2.0 * work(case)["hits"] + 2 * total)
        return s
    s["prims"] = _prims(case, g)
    if case["do"] == "build":
        s["tree"] = lb.alloc_tree(case["n"], case["bits"], DEV)
        return s
    if case["do"] == "rays_first":
        s["queries"] = _rays(s["prims"], case["m"], g)
    else:
        s["queries"] = _queries(case, s["prims"], g)
        s["qkind"] = QKIND[case["q"]]
        s["hits"] = _hit_buffer(1.5 * case["m"] * _hits(case) + 4 * case["n"])
    if case["do"] != "request":
        s["tree"] = lb.build(s["prims"], case["bits"], workspace=s["ws"])
        del s["prims"]
    return s


def _room(s, offsets):
    """The hit buffer, after the one read of the number of hits."""
    total = int(offsets[-1].item())
    if s["hits"].numel() < total:
        s["hits"] = _hit_buffer(total)
    return s["hits"]


def _query(s, tree):
    offsets = lb.query_count(tree, s["queries"], s["qkind"], s["qws"])
    return offsets, lb.query_fill(tree, s["queries"], s["qkind"], _room(s, offsets), s["qws"])


def run(s):
    do = s["do"]
    if do == "build":
        t = lb.build(s["prims"], s["bits"], workspace=s["ws"], tree=s["tree"])
        return t.nodes, t.codes, t.leaf_perm
    if do == "query":
        return _query(s, s["tree"])
    if do == "rays_first":
        return lb.query_first(s["tree"], s["queries"], workspace=s["qws"])
    if do == "request":
        t = lb.build(s["prims"], s["bits"], workspace=s["ws"])
        return (t.nodes, t.leaf_perm) + _query(s, t)
    b = lb.build_batched(s["prims"], s["seg"], s["bits"], s["max_scene"], workspace=s["ws"], batch=s["batch"])
    offsets = lb.query_batched_count(b, s["queries"], s["qseg"], lb.SPHERES, s["qws"])
    hits = lb.query_batched_fill(b, s["queries"], s["qseg"], lb.SPHERES, offsets, _room(s, offsets), s["qws"])
    return b.nodes, b.codes, b.leaf_perm, offsets, hits


# ------------------------------------------------------------- bookkeeping

def _hits(case):
    """Expected hits of one query."""
    n = case["n"]
    if "neighbours" in case:
        return case["neighbours"] * (1.0 if case["q"] == "spheres" else 6.0 / math.pi)
    if case.get("q") == "segments":
        return 216.0 * (n / 2.0 ** 24) * (case["length"] / 0.002)
    if "side" in case:   # mixture density averages to n over the unit cube
        share = math.pi / 6.0 if case["q"] == "spheres" else 1.0
        return n * share * (case["side"] + MEAN_SIDE) ** 3
    return 1.0


def _build_bytes(case, n):
    width = 24 if case["prims"] == "clustered" else 12
    return n * (width + 2 * NODE + (4 if case["bits"] == 30 else 8) + 4)


def work(case):
    """Inputs once, outputs once; of a tree that a query reads, its hits'
    leaves and one path per query, or the whole tree if that is less."""
    if case["do"] == "batch":
        n = sum(_sizes(case))
        m = case["m"] * case["scenes"]
        hits = case["m"] * n * 4.0 / 3.0 * math.pi * case["radius"] ** 3
        return {"bytes": _build_bytes(case, n) + m * 24 + 4 * hits, "flops": 30.0 * n + 20.0 * hits, "hits": hits}
    n = case["n"]
    built = _build_bytes(case, n) if case["do"] in ("build", "request") else 0
    if case["do"] == "build":
        return {"bytes": built, "flops": 30.0 * n}
    m, hits = case["m"], case["m"] * _hits(case)
    width = {"spheres": 16, "boxes": 24}.get(case.get("q"), 32)
    tree = min(2 * n * NODE, (hits + m * math.log2(n)) * NODE)
    out = 8 * m if case["do"] == "rays_first" else 8 * (m + 1) + 4 * hits
    return {"bytes": built + m * width + out + (0 if built else tree), "flops": 20.0 * (hits + m * math.log2(n))}


def exact(case, seed):
    """Entry parameters of the first hits by brute force in 64 bits; every
    other output is whole numbers or bit patterns."""
    if case["do"] != "rays_first" or case["m"] * case["n"] > 1 << 33:
        return None
    g = _gen(seed)
    boxes = _prims(case, g)
    q = _rays(boxes, case["m"], g).double()
    boxes = boxes.double()
    best = torch.full((case["m"],), math.inf, dtype=torch.float64, device=DEV)
    step = max(1, (1 << 25) // case["m"])
    for b in boxes.split(step):
        t_in = q[:, 3:4].expand(-1, b.shape[0])
        t_out = q[:, 7:8].expand(-1, b.shape[0])
        met = torch.ones((case["m"], b.shape[0]), dtype=torch.bool, device=DEV)
        for a in range(3):
            o, d = q[:, a:a + 1], q[:, 4 + a:5 + a]
            flat = d == 0
            inv = 1.0 / torch.where(flat, torch.ones_like(d), d)
            t1, t2 = (b[:, a] - o) * inv, (b[:, 3 + a] - o) * inv
            inside = (b[:, a] <= o) & (o <= b[:, 3 + a])
            met &= torch.where(flat, inside, torch.ones_like(inside))
            t_in = torch.where(flat, t_in, torch.maximum(t_in, torch.minimum(t1, t2)))
            t_out = torch.where(flat, t_out, torch.minimum(t_out, torch.maximum(t1, t2)))
        met &= t_in <= t_out
        best = torch.minimum(best, torch.where(met, t_in, torch.full_like(t_in, math.inf)).amin(1))
    return None, best
