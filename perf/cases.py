"""The work that users of this library have it do, as cases that can be timed
and compared: searches from one query to large batches, the projection tables
alone, the serving loop, a captured batch of uneven requests, and index builds.

A case is a dict of plain values.  listed() gives the fixed ones, draw(rng) one
more of the same ranges, prepare(case, seed) what a program holds before the
call, run(state) one pass through the public entry points, work(case) the bytes
and operations the pass cannot do without, and exact(case, seed) its outputs in
64 bits, from torch alone.

The collection that is searched (vectors, graph, directions) and its index
depend on the case alone: a program builds them once and then sees new queries,
which are what the seed draws.  The last three of each are kept, as such a
program keeps its own.  Where the build is the case, the seed draws the vectors
and their graph.

Vectors come from the recipes of the workloads: floored exponential mixtures
(integers 0..255), overlapping clusters on the sphere with a decaying
spectrum, and correlated clusters on a 48-dimensional subspace.  The graph is
an approximate nearest-neighbour graph (random partitions, two rounds of
neighbours of neighbours), pruned by the relative-neighbourhood rule, with
reverse edges and two random long-range edges per node.
"""
import collections
import math

import numpy as np
import torch

import paper_2402_11354_amd as P

FLAGS_PRECISION = P.PEOS_FLAG_BF16_BASE | P.PEOS_FLAG_FP16


def _search_case(name, kind, n, d, **kw):
    case = dict(name=name, op="search", kind=kind, n=n, d=d, R=32, L=8, m=16, flags=0, nq=1000, k=10,
                ef=64, rule="hnsw", eps=0.1, mode=P.PEOS_MODE_PEOS)
    case.update(kw)
    return case


def listed():
    return [
        # the smallest call: one query of a 1M-vector collection, latency and
        # launches are all it is
        _search_case("one_query", "counts", 1_000_000, 128, nq=1),
        # a serving loop: a handful of host requests of odd sizes, each with
        # its own k and ef, submitted and polled to completion
        dict(name="requests", op="serve", kind="sphere", n=200_000, d=256, R=32, L=8, m=16, flags=0,
             requests=9, mix=1, eps=0.1),
        # the ordinary batch at recall@10 of about 0.95
        _search_case("batch_10k", "counts", 1_000_000, 128, nq=10_000, eps=0.2),
        # the same collection with the routing test off, at its own ef
        _search_case("exhaustive_10k", "counts", 1_000_000, 128, nq=10_000, ef=60,
                     mode=P.PEOS_MODE_EXHAUSTIVE),
        # many results per query, the directions per subspace (128) of the
        # published experiments
        _search_case("k100_m128", "counts", 1_000_000, 128, nq=4_000, k=100, ef=200, m=128),
        # the compact index (256 bytes a node), an odd batch
        _search_case("compact_3001", "counts", 1_000_000, 128, nq=3_001, ef=96, L=2,
                     flags=P.PEOS_FLAG_COMPACT),
        # long vectors in the precision form, searched for many results
        _search_case("long_precision", "lowrank", 100_000, 960, nq=1_000, k=100, ef=384, L=16,
                     flags=FLAGS_PRECISION),
        # a large batch of requests of uneven k and ef with a queue of twice
        # each list, captured once and replayed
        dict(name="uneven_graph", op="graph", kind="sphere", n=1_000_000, d=96, R=32, L=8, m=16,
             flags=0, nq=20_000, eps=0.1),
        # the unbounded queue of the printed algorithm
        _search_case("unbounded_1000", "counts", 1_000_000, 128, nq=1_000, ef=24, rule="unbounded"),
        # the projection tables alone, long vectors and 128 directions
        dict(name="tables_m128", op="tables", d=960, L=16, m=128, nq=2_049),
        # the index build (edge codes and scalars) of 400k ordinary vectors
        dict(name="build_d128", op="build", kind="counts", n=400_000, d=128, R=32, L=8, m=16, flags=0),
        # and of long vectors in the precision form
        dict(name="build_d960", op="build", kind="lowrank", n=20_000, d=960, R=32, L=16, m=16,
             flags=FLAGS_PRECISION),
    ]


# dimension -> numbers of subspaces whose blocks are multiples of 4
_SHAPES = {("counts", 128): (4, 8, 16), ("counts", 32): (2, 4, 8), ("sphere", 96): (4, 8, 12),
           ("sphere", 256): (8, 16), ("lowrank", 384): (8, 12, 16), ("lowrank", 960): (8, 15, 16)}


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind, d = rng.choice(sorted(_SHAPES))
    L = rng.choice(_SHAPES[kind, d])
    m = rng.choice((16, 16, 16, 32, 128))
    R = rng.choice((16, 32, 32, 48))
    op = rng.choice(("search", "search", "search", "search", "graph", "serve", "tables", "build"))
    n = _log_int(rng, 3_000, 300_000 if d <= 256 else 40_000)
    flags = rng.choice((0, 0, P.PEOS_FLAG_BF16_BASE, P.PEOS_FLAG_FP16, FLAGS_PRECISION,
                        P.PEOS_FLAG_COMPACT))
    if flags == P.PEOS_FLAG_COMPACT:
        L = rng.choice((2, 4))
    eps = rng.choice((0.05, 0.1, 0.2, 0.3))
    if op == "tables":
        return dict(op=op, d=d, L=L, m=m, nq=_log_int(rng, 1, 20_000))
    shape = dict(kind=kind, n=n, d=d, R=R, L=L, m=m, flags=flags)
    if op == "build":
        shape["n"] = min(n, 400_000 * 128 * 16 * 32 // (d * m * R))
        return dict(op=op, **shape)
    if op == "serve":
        return dict(op=op, requests=rng.randint(1, 24), mix=rng.randint(0, 999), eps=eps, **shape)
    if op == "graph":
        return dict(op=op, nq=_log_int(rng, 20, 4_000), eps=eps, **shape)
    ef = _log_int(rng, 10, 500)
    rule = rng.choice(("hnsw", "hnsw", "hnsw", "twice", "unbounded"))
    nq = _log_int(rng, 1, 10_000)
    if rule == "unbounded":
        ef = min(ef, 64)
        nq = min(nq, 1_000)
    nq = max(1, min(nq, int(4e8 / (ef * (d + 128)))))
    return dict(op=op, nq=nq, k=rng.randint(1, min(ef, 100)), ef=ef, rule=rule, eps=eps,
                mode=rng.choice((P.PEOS_MODE_PEOS, P.PEOS_MODE_PEOS, P.PEOS_MODE_EXHAUSTIVE)), **shape)


# ---------------------------------------------------------------------------
# vectors
# ---------------------------------------------------------------------------
def _generator(*seeds):
    g = torch.Generator(device="cuda")
    s = 0
    for v in seeds:
        s = (s * 1_000_003 + int(v) + 1) % (1 << 62)
    g.manual_seed(s)
    return g


def _metric(kind):
    return P.PEOS_METRIC_ANGULAR if kind == "sphere" else P.PEOS_METRIC_L2


def _vectors(kind, d, count, model_seed, draw_seed):
    """count x d float32 draws of the mixture that model_seed fixes."""
    g = _generator(1, model_seed, d)
    r = _generator(2, model_seed, draw_seed)
    dev = dict(device="cuda")
    out = torch.empty((count, d), dtype=torch.float32, **dev)
    clusters = {"counts": 100, "sphere": 500, "lowrank": 256}[kind]
    if kind == "counts":
        means = torch.exp(math.log(2.0) + (math.log(64.0) - math.log(2.0))
                          * torch.rand((clusters, d), generator=g, **dev))
        weight = 1.0 / torch.arange(1, clusters + 1, dtype=torch.float32, **dev)
    elif kind == "sphere":
        centers = torch.randn((clusters, d), generator=g, **dev)
        centers /= centers.norm(dim=1, keepdim=True)
        spec = torch.arange(1, d + 1, dtype=torch.float32, **dev) ** -0.8
        spec *= 2.5 / spec.norm()
        weight = torch.ones(clusters, **dev)
    else:
        centers = 0.5 * torch.randn((clusters, d), generator=g, **dev)
        factors = torch.randn((48, d), generator=g, **dev)
        factors /= factors.norm(dim=1, keepdim=True)
        spec = torch.arange(1, 49, dtype=torch.float32, **dev) ** -0.5
        spec *= 24.0 / spec.norm()
        latent = spec * torch.exp(0.3 * torch.randn((clusters, 48), generator=g, **dev))
        weight = torch.ones(clusters, **dev)
    edges = torch.cumsum(weight / weight.sum(), 0)
    for s in range(0, count, 1 << 17):
        c = min(1 << 17, count - s)
        z = torch.searchsorted(edges, torch.rand(c, generator=r, **dev)).clamp_(max=clusters - 1)
        if kind == "counts":
            u = torch.rand((c, d), generator=r, **dev).clamp_(min=1e-7)
            x = torch.floor(-torch.log(u) * means[z]).clamp_(max=255.0)
        elif kind == "sphere":
            x = centers[z] + spec * torch.randn((c, d), generator=r, **dev)
            x /= x.norm(dim=1, keepdim=True)
        else:
            x = centers[z] + (latent[z] * torch.randn((c, 48), generator=r, **dev)) @ factors
            x += 0.05 * torch.randn((c, d), generator=r, **dev)
        out[s:s + c] = x
    return out


# ---------------------------------------------------------------------------
# graph (an input of the search)
# ---------------------------------------------------------------------------
_NONE = (1 << 63) - 1  # key of no candidate


def _keys(dist, ids):
    """(distance, id) as one sortable integer."""
    return (dist.clamp(min=0).contiguous().view(torch.int32).to(torch.int64) << 32) | ids


def _unique_smallest(keys, count):
    """The count smallest keys of each row, an id once."""
    ids = keys & 0xFFFFFFFF
    ids, order = torch.sort(ids, dim=1, stable=True)
    keys = torch.gather(keys, 1, order)
    again = torch.zeros_like(keys, dtype=torch.bool)
    again[:, 1:] = ids[:, 1:] == ids[:, :-1]
    keys = torch.where(again, torch.full_like(keys, _NONE), keys)
    return torch.sort(keys, dim=1)[0][:, :count]


def _partition_neighbours(x, count, block, g):
    """Each row's nearest rows within its block of a random balanced partition."""
    n, d = x.shape
    pad = -(-n // block) * block
    order = torch.randperm(n, generator=g, device=x.device)
    # a last block that is not full holds some rows again, marked by n more
    order = torch.cat([order, order[:pad - n] + n]) if pad > n else order
    parts = 1
    while pad // parts > block:
        # sort each part by its projection on a fresh direction, then halve
        p = x[order % n] @ torch.randn(d, generator=g, device=x.device)
        size = -(-(pad // block) // parts) * block
        part = torch.div(torch.arange(pad, device=x.device), size, rounding_mode="floor")
        p = (p - p.min()) / (p.max() - p.min() + 1e-20)
        rank = torch.sort(part.to(torch.float64) * 2 + p.to(torch.float64), stable=True)[1]
        order = order[rank]
        parts *= 2
    blocks = order.view(-1, block)
    got = torch.full((n, count), _NONE, dtype=torch.int64, device=x.device)
    step = max(1, (1 << 27) // (block * block))
    for s in range(0, blocks.shape[0], step):
        first = blocks[s:s + step] < n
        ids = blocks[s:s + step] % n
        v = x[ids]
        sq = (v * v).sum(-1)
        dist = sq[:, :, None] + sq[:, None, :] - 2.0 * torch.bmm(v, v.transpose(1, 2).contiguous())
        key = _keys(dist, ids[:, None, :].expand(dist.shape))
        key = torch.where(ids[:, :, None] == ids[:, None, :], torch.full_like(key, _NONE), key)
        best = torch.topk(key, count, dim=2, largest=False, sorted=True)[0]
        got[ids[first]] = best[first]
    return got


def _neighbours_of_neighbours(x, keys, width):
    n, d = x.shape
    out = torch.empty_like(keys)
    near = (keys[:, :width] & 0xFFFFFFFF)
    near = torch.where(keys[:, :width] < _NONE, near, torch.arange(n, device=x.device)[:, None])
    step = max(1, (1 << 29) // (width * width * d))
    for s in range(0, n, step):
        me = torch.arange(s, min(n, s + step), device=x.device)
        ids = near[near[me]].reshape(me.numel(), -1)
        v = x[ids] - x[me][:, None, :]
        key = _keys((v * v).sum(-1), ids)
        key = torch.where(ids == me[:, None], torch.full_like(key, _NONE), key)
        out[s:s + step] = _unique_smallest(torch.cat([keys[me], key], 1), keys.shape[1])
    return out


def _prune(x, keys, most):
    """Relative-neighbourhood pruning of sorted candidates, at most `most` kept first."""
    n, d = x.shape
    count = keys.shape[1]
    out = torch.full((n, most), -1, dtype=torch.int64, device=x.device)
    step = max(1, (1 << 29) // (count * d))
    for s in range(0, n, step):
        k = keys[s:s + step]
        ok = k < _NONE
        ids = torch.where(ok, k & 0xFFFFFFFF, 0)
        dist = (k >> 32).to(torch.int32).view(torch.float32)
        v = x[ids]
        sq = (v * v).sum(-1)
        pair = sq[:, :, None] + sq[:, None, :] - 2.0 * torch.bmm(v, v.transpose(1, 2).contiguous())
        nearer = pair <= dist[:, :, None]
        kept = torch.zeros_like(ok)
        for j in range(count):
            kept[:, j] = ok[:, j] & ~(kept[:, :j] & nearer[:, j, :j]).any(1)
        place = torch.cumsum(kept.to(torch.int64), 1) - 1
        kept &= place < most
        row = torch.arange(k.shape[0], device=x.device)[:, None].expand(k.shape)
        out[s:s + step][row[kept], place[kept]] = ids[kept]
    return out


def _fill(graph, src, dst):
    """Offers src -> dst take free slots of dst's row, in the order given."""
    n, R = graph.shape
    fresh = (dst != src) & ~(graph[dst] == src[:, None]).any(1)
    src, dst = src[fresh], dst[fresh]
    order = torch.sort(dst, stable=True)[1]
    src, dst = src[order], dst[order]
    count = torch.bincount(dst, minlength=n)
    rank = torch.arange(dst.numel(), device=dst.device) - (torch.cumsum(count, 0) - count)[dst]
    slot = (graph >= 0).sum(1)[dst] + rank
    ok = slot < R
    graph[dst[ok], slot[ok]] = src[ok]


def _graph(x, R, g, quality=True):
    """n x R int32 neighbour ids, -1 where there is none."""
    n = x.shape[0]
    block = 4096 if quality else 256
    while block // 2 >= max(n, 2):
        block //= 2
    if not quality:  # nearest rows of one partition, for builds
        keys = _partition_neighbours(x, min(R, block - 1), block, g)
        keys = _unique_smallest(keys, keys.shape[1])
        graph = torch.where(keys < _NONE, keys & 0xFFFFFFFF, -1)
        if graph.shape[1] < R:
            graph = torch.cat([graph, torch.full((n, R - graph.shape[1]), -1, device=x.device)], 1)
        return graph.to(torch.int32).contiguous()
    width = min(24, block - 1)
    keys = torch.cat([_partition_neighbours(x, width, block, g) for _ in range(6)], 1)
    keys = _unique_smallest(keys, 40)
    for _ in range(2):
        keys = _neighbours_of_neighbours(x, keys, 16)
    graph = torch.full((n, R), -1, dtype=torch.int64, device=x.device)
    most = R * 3 // 4
    graph[:, :most] = _prune(x, keys, most)
    dst = graph[:, :most].reshape(-1)
    src = torch.arange(n, device=x.device)[:, None].expand(n, most).reshape(-1)
    # nearest offers first: the column is the rank of the edge in its own row
    rank = torch.arange(most, device=x.device)[None, :].expand(n, most).reshape(-1)
    order = torch.sort(rank, stable=True)[1]
    dst, src = dst[order], src[order]
    _fill(graph, src[dst >= 0], dst[dst >= 0])
    for _ in range(2):
        free = (graph[:, -1] < 0).nonzero().reshape(-1)
        _fill(graph, torch.randint(0, n, free.shape, generator=g, device=x.device), free)
    return graph.to(torch.int32).contiguous()


# ---------------------------------------------------------------------------
# what a program keeps
# ---------------------------------------------------------------------------
_kept = {"collection": collections.OrderedDict(), "index": collections.OrderedDict()}


def _keep(group, key, make, most=3):
    box = _kept[group]
    if key not in box:
        while len(box) >= most:
            box.popitem(last=False)
        box[key] = make()
    box.move_to_end(key)
    return box[key]


def _collection(case):
    def make():
        x = _vectors(case["kind"], case["d"], case["n"], 7, 1)
        graph = _graph(x, case["R"], _generator(3, case["n"], case["d"]))
        entry = int(((x - x.mean(0, keepdim=True)) ** 2).sum(1).argmin())
        return x, graph, entry
    return _keep("collection", tuple(case[k] for k in ("kind", "n", "d", "R")), make)


def _directions(case, seed=5):
    g = _generator(4, seed, case["d"], case["L"], case["m"])
    A = torch.randn((case["L"], case["m"], case["d"] // case["L"]), generator=g, device="cuda")
    B = torch.randn((case["m"], case["d"]), generator=g, device="cuda")
    return A, B


def _index(case):
    def make():
        x, graph, entry = _collection(case)
        A, B = _directions(case)
        return P.peos_build_tables(x, graph, entry, case["L"], case["m"], A, B, _metric(case["kind"]),
                                   flags=case["flags"])
    return _keep("index", tuple(case[k] for k in ("kind", "n", "d", "R", "L", "m", "flags")), make)


def _queries(case, count, seed):
    return _vectors(case["kind"], case["d"], count, 7, 1000 + seed)


def _pool(case):
    return {"hnsw": case["ef"], "twice": -2, "unbounded": 0}[case["rule"]]


def _uneven(nq, seed):
    """k and ef of a batch of uneven requests."""
    r = np.random.default_rng([seed, 9])
    ef = r.choice(np.array([32, 64, 100, 128, 256], dtype=np.int32), size=nq)
    k = r.choice(np.array([1, 10, 100], dtype=np.int32), size=nq)
    return k, np.maximum(ef, k).astype(np.int32)


def _requests(case, seed):
    """(queries, k, ef) of each request, on the host; the seed draws the queries."""
    r = np.random.default_rng([case["mix"], 8])
    sizes = [int(min(64, max(1, round(math.exp(r.uniform(0.0, math.log(64.0))))))) for _ in range(case["requests"])]
    q = _queries(case, sum(sizes), seed).cpu().numpy()
    out, at = [], 0
    for s in sizes:
        k, ef = int(r.choice([1, 10, 100])), int(r.choice([32, 64, 128, 256, 512]))
        out.append((q[at:at + s].copy(), k, max(ef, k)))
        at += s
    return out


def _search_buffers(nq, k):
    return (torch.empty((nq, k), dtype=torch.int64, device="cuda"),
            torch.empty((nq, k), dtype=torch.float32, device="cuda"),
            torch.empty((nq, P.PEOS_NSTATS), dtype=torch.int32, device="cuda"))


def prepare(case, seed):
    st = dict(op=case["op"])
    if case["op"] == "build":
        x = _vectors(case["kind"], case["d"], case["n"], 7, 2000 + seed)
        A, B = _directions(case, 6 + seed)
        st.update(x=x, graph=_graph(x, case["R"], _generator(5, seed), quality=False), A=A, B=B, L=case["L"],
                  m=case["m"], metric=_metric(case["kind"]), flags=case["flags"])
        return st
    if case["op"] == "tables":
        small = dict(case, kind="lowrank" if case["d"] > 256 else "counts", n=512, R=16, flags=0)
        q = _queries(small, case["nq"], seed)
        st.update(index=_index(small), q=q, norms=torch.empty(case["nq"], device="cuda"),
                  tables=torch.empty((case["nq"], case["L"] + 1, case["m"]), device="cuda"))
        return st
    index = _index(case)
    st["index"] = index
    if case["op"] == "serve":
        st["requests"] = _requests(case, seed)
        st["server"] = P.Server(index, max_batch=128, max_k=100, max_ef=512, max_inflight=4, eps=case["eps"])
        return st
    nq = case["nq"]
    q = _queries(case, nq, seed)
    if case["op"] == "graph":
        k, ef = (torch.from_numpy(a).cuda() for a in _uneven(nq, seed))
        out = _search_buffers(nq, 100)
        ws = torch.empty(P.peos_search_ws_bytes(index, nq, 256, -2), dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        st.update(out=out, graph=P.peos_graph_create(index, q, k, ef, 100, -2, case["eps"], P.PEOS_MODE_PEOS, *out,
                                                     ws, k_all=100, ef_all=256))
        return st
    pool = _pool(case)
    ws = torch.empty(P.peos_search_ws_bytes(index, nq, max(case["ef"], case["k"]), pool), dtype=torch.uint8,
                     device="cuda")
    st.update(q=q, k=case["k"], ef=case["ef"], pool=pool, eps=case["eps"], mode=case["mode"],
              out=_search_buffers(nq, case["k"]), ws=ws)
    return st


def run(st):
    if st["op"] == "search":
        P.peos_search(st["index"], st["q"], st["k"], st["ef"], st["k"], st["pool"], st["eps"], st["mode"], *st["out"],
                      st["ws"])
        return dict(zip(("ids", "dists", "stats"), st["out"]))
    if st["op"] == "graph":
        st["graph"].launch()
        return dict(zip(("ids", "dists", "stats"), st["out"]))
    if st["op"] == "tables":
        P.peos_query_tables(st["index"], st["q"], st["tables"], st["norms"])
        return dict(tables=st["tables"], norms=st["norms"])
    if st["op"] == "serve":
        srv = st["server"]
        tickets = [srv.submit(q, k, ef) for q, k, ef in st["requests"]]
        done = {}
        while len(done) < len(tickets):
            done.update((t, (ids, dists)) for t, ids, dists in srv.poll(wait=True))
        return dict(ids=[done[t][0] for t in tickets], dists=[done[t][1] for t in tickets])
    index = P.peos_build_tables(st["x"], st["graph"], 0, st["L"], st["m"], st["A"], st["B"], st["metric"],
                                flags=st["flags"])
    return _records(index)


def _records(index):
    """The parts of a built index, as views of its memory."""
    lay, mem = index.layout(), index._keep[-1]
    rec = mem[:lay.n * lay.node_stride].view(lay.n, lay.node_stride)
    part = lambda at, size: rec[:, at:at + size]  # noqa: E731
    out = dict(codes=part(lay.codes_offset, lay.R * lay.code_bytes))
    if lay.flags & P.PEOS_FLAG_COMPACT:
        out.update(header=part(0, 16).view(torch.float32), scalars=part(lay.scalars_offset, 2 * lay.R))
    else:
        half = torch.float16 if lay.flags & P.PEOS_FLAG_FP16 else torch.float32
        out["scalars"] = part(lay.scalars_offset, lay.scalar_bytes * lay.R).view(half)
    if lay.flags & P.PEOS_FLAG_BF16_BASE:
        at = lay.bf16_offset
        out["copy"] = mem[at:at + 2 * lay.n * lay.d].view(torch.bfloat16)
    return out


# ---------------------------------------------------------------------------
# the work of a pass
# ---------------------------------------------------------------------------
def _search_work(case, ef, rule):
    """Bytes and operations of one query with a list of ef: its expansions
    read a neighbour row and, with the test on, the edges' codes and scalars;
    the nodes that are reached read their vector once.  On these graphs a
    query expands about ef + 8 nodes (six times as many with the unbounded
    queue, twice as many with a queue of 2 ef) and computes about 14 new
    distances per expansion (9 on the correlated clusters, 8 with the
    unbounded queue).  Each query goes its own way through arrays that no
    cache holds, so each pays for its own reads."""
    n_exp = min(case["n"], int((ef + 8) * {"hnsw": 1.0, "twice": 2.0, "unbounded": 6.0}[rule]))
    n_dist = min(case["n"], n_exp * (8 if rule == "unbounded" else 9 if case["kind"] == "lowrank" else 14))
    width = 2 if case["flags"] & P.PEOS_FLAG_BF16_BASE else 4
    edge = 6 if case["flags"] & P.PEOS_FLAG_COMPACT else (case["L"] + 1 + (8 if case["flags"] & P.PEOS_FLAG_FP16 else 16))
    if case.get("mode", P.PEOS_MODE_PEOS) == P.PEOS_MODE_EXHAUSTIVE:
        edge = 0
    table = 4 * (case["L"] + 1) * case["m"]
    return (n_exp * 4 * case["R"] + n_dist * (width * case["d"] + edge) + 4 * case["d"] + table,
            n_dist * 3 * case["d"] + 4 * case["d"] * case["m"])


def work(case):
    op, d = case["op"], case["d"]
    if op == "tables":
        L, m, nq = case["L"], case["m"], case["nq"]
        return dict(bytes=4.0 * (nq * (d + (L + 1) * m + 1) + 2 * m * d), flops=4.0 * d * m * nq)
    if op == "build":
        n, R, L, m = case["n"], case["R"], case["L"], case["m"]
        out = P.peos_index_bytes(n, d, R, L, m, case["flags"])[0]
        per_edge = 4.0 * d * m if not case["flags"] & P.PEOS_FLAG_COMPACT else 2.0 * d * m
        return dict(bytes=4.0 * n * (d + R) + out, flops=n * R * (per_edge + 8.0 * d))
    if op == "search":
        b, f = _search_work(case, max(case["ef"], case["k"]), case["rule"])
        return dict(bytes=float(case["nq"] * (b + 12 * case["k"])), flops=float(case["nq"] * f))
    if op == "graph":  # mean list of _uneven
        b, f = _search_work(case, 130, "twice")
        return dict(bytes=float(case["nq"] * (b + 1200)), flops=float(case["nq"] * f))
    b, f = _search_work(case, 200, "hnsw")  # about 15 queries a request
    return dict(bytes=15.0 * case["requests"] * (b + 450), flops=15.0 * case["requests"] * f)


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------
def _codes64(e, A, B):
    """Signed codes' table entries are looked up with these: (index, sign) of
    the extreme direction per subspace and of the residual, and w_reg, w_res."""
    L, m, dp = A.shape
    blk = e.view(-1, L, dp)
    p = torch.matmul(blk.transpose(0, 1).contiguous(), A.transpose(1, 2).contiguous())  # L x E x m
    j = p.abs().argmax(2)
    sign = torch.where(torch.gather(p, 2, j[:, :, None])[:, :, 0] < 0, -1.0, 1.0)
    s = blk.norm(dim=2)
    nz = (s > 0).sum(1).clamp(min=1)
    ne = e.norm(dim=1)
    c = s.sum(1) / nz
    res = e - (torch.where(s > 0, c[:, None] / s.clamp(min=1e-300), 0.0)[:, :, None] * blk).reshape(e.shape)
    p0 = res @ B.T.contiguous()
    j0 = p0.abs().argmax(1)
    sign0 = torch.where(torch.gather(p0, 1, j0[:, None])[:, 0] < 0, -1.0, 1.0)
    safe = ne.clamp(min=1e-300)
    w_reg = torch.where(ne > 0, (c * nz.double().sqrt() / safe).clamp(max=1.0), 1.0)
    w_res = torch.where(ne > 0, (res.norm(dim=1) / safe).clamp(max=1.0), 0.0)
    return j.T, sign.T, j0, sign0, ne, w_reg, w_res


def _tables64(q, A, B):
    L, m, dp = A.shape
    u = q / q.norm(dim=1, keepdim=True)
    sub = torch.matmul(u.view(-1, L, dp).transpose(0, 1).contiguous(), A.transpose(1, 2).contiguous()).transpose(0, 1)
    return torch.cat([(u @ B.T.contiguous())[:, None, :], sub], 1)


def _search64(case, q, ef, k, rule, eps, mode):
    """Best-first search of all queries in step, in float64: distances of the
    k nearest found, +inf where there are fewer."""
    x, graph, entry = _collection(case)
    A, B = (t.double() for t in _directions(case))
    L, m, _ = A.shape
    metric, nq, d, R = _metric(case["kind"]), q.shape[0], case["d"], case["R"]
    q = q.double()
    qn = q.norm(dim=1)
    tables = _tables64(q, A, B)
    eta = math.sqrt(2.0 * L * math.log(m))
    c_eps = math.sqrt(2.0) * float(torch.erfinv(torch.tensor(2.0 * eps - 1.0, dtype=torch.float64)))
    cap = {"hnsw": ef, "twice": 2 * ef, "unbounded": max(256, 16 * ef)}[rule]
    dev = x.device

    def dist(rows, ids):
        v = x[ids.clamp(min=0)].double()
        if metric == P.PEOS_METRIC_L2:
            return ((v - q[rows][:, None, :]) ** 2).sum(-1)
        return 1.0 - (v * (q[rows] / qn[rows, None])[:, None, :]).sum(-1)

    seen = torch.zeros((nq, case["n"]), dtype=torch.bool, device=dev)
    ids = torch.full((nq, cap + R), -1, dtype=torch.int64, device=dev)
    dd = torch.full((nq, cap + R), math.inf, dtype=torch.float64, device=dev)
    done = torch.zeros((nq, cap + R), dtype=torch.bool, device=dev)
    ids[:, 0] = entry
    dd[:, :1] = dist(torch.arange(nq, device=dev), ids[:, :1])
    seen[:, entry] = True
    for step in range(1 << 16):
        open_ = (ids[:, :cap] >= 0) & ~done[:, :cap]
        rows = open_.any(1).nonzero().reshape(-1)
        if not rows.numel():
            break
        at = open_[rows].to(torch.int8).argmax(1)
        v, dv, delta = ids[rows, at], dd[rows, at], dd[rows, ef - 1]
        done[rows, at] = True
        full = torch.isfinite(delta)
        nb = graph[v].long()
        ok = (nb >= 0) & ~seen[rows[:, None], nb.clamp(min=0)]
        if mode == P.PEOS_MODE_PEOS and bool(full.any()):
            r, c = (ok & full[:, None]).nonzero(as_tuple=True)
            u = nb[r, c]
            xu, xv = x[u].double(), x[v[r]].double()
            j, sign, j0, sign0, ne, w_reg, w_res = _codes64(xu - xv, A, B)
            t = tables[rows[r]]
            h = w_reg * (sign * torch.gather(t[:, 1:], 2, j[:, :, None])[:, :, 0]).sum(1)
            h = h + math.sqrt(L) * w_res * sign0 * torch.gather(t[:, 0], 1, j0[:, None])[:, 0]
            diff = dv[r] - delta[r]
            if metric == P.PEOS_METRIC_L2:
                num = 0.5 * ((xu * xu).sum(1) - (xv * xv).sum(1) + diff)
                a = num / (qn[rows[r]] * ne)
            else:
                num = diff
                a = num / ne
            var = (w_reg ** 2 + L * w_res ** 2 - L * a * a / (L + 1)).clamp(min=0)
            passed = torch.where(ne > 0, (a <= 0) | ((a < 1) & (h >= a * eta + c_eps * var.sqrt())), num < 0)
            ok[r, c] = passed
        new = torch.where(ok, dist(rows, nb), math.inf)
        keep = ok & (new < delta[:, None])
        r, c = ok.nonzero(as_tuple=True)
        seen[rows[r], nb[r, c]] = True
        ids[rows, cap:] = torch.where(keep, nb, -1)
        dd[rows, cap:] = torch.where(keep, new, math.inf)
        done[rows, cap:] = False
        # by (distance, id); past ef only what is still to be expanded stays
        li, ld, lx = ids[rows], dd[rows], done[rows]
        for by in (li, None):
            o = torch.sort(by if by is not None else ld, dim=1, stable=True)[1]
            li, ld, lx = (torch.gather(t, 1, o) for t in (li, ld, lx))
        if cap > ef:
            gone = lx & (torch.arange(cap + R, device=dev)[None, :] >= ef)
            li, ld = torch.where(gone, -1, li), torch.where(gone, math.inf, ld)
            o = torch.sort(ld, dim=1, stable=True)[1]
            li, ld, lx = (torch.gather(t, 1, o) for t in (li, ld, lx))
        ids[rows], dd[rows], done[rows] = li, ld, lx
        ids[:, cap:], dd[:, cap:] = -1, math.inf
    return dd[:, :k]


def exact(case, seed):
    op = case["op"]
    if op == "tables":
        small = dict(case, kind="lowrank" if case["d"] > 256 else "counts")
        q = _queries(small, case["nq"], seed).double()
        A, B = (t.double() for t in _directions(small))
        return dict(tables=_tables64(q, A, B), norms=q.norm(dim=1))
    if op == "build":
        if case["flags"] & P.PEOS_FLAG_COMPACT:
            return None  # quantised against each node's own ranges
        st = prepare(dict(case, op="build"), seed)
        x, graph, n, R, L = st["x"], st["graph"], case["n"], case["R"], case["L"]
        A, B = st["A"].double(), st["B"].double()
        out = torch.zeros((n, R, 4), dtype=torch.float64, device="cuda")
        step = max(1, (1 << 26) // (R * case["d"]))
        for s in range(0, n, step):
            v, c = (graph[s:s + step] >= 0).nonzero(as_tuple=True)
            xu, xv = x[graph[s + v, c].long()].double(), x[s + v].double()
            _, _, _, _, ne, w_reg, w_res = _codes64(xu - xv, A, B)
            ge = 0.5 * ((xu * xu).sum(1) - (xv * xv).sum(1)) * (_metric(case["kind"]) == P.PEOS_METRIC_L2)
            if case["flags"] & P.PEOS_FLAG_FP16:
                inv = 1.0 / ne
                four = torch.stack([torch.where(ne > 0, ge * inv, 0.0), inv, w_reg, math.sqrt(L) * w_res], 1)
            else:
                four = torch.stack([ge, ne, w_reg, math.sqrt(L) * w_res], 1)
            out[s + v, c] = four
        r = dict(codes=None, scalars=out.view(n, 4 * R))
        if case["flags"] & P.PEOS_FLAG_BF16_BASE:
            r["copy"] = x.double().view(-1)
        return r
    # the routes of the reduced forms depend on their own rounding, and
    # visited sets and lists past these sizes take too long here
    if case["flags"] or case["n"] * case.get("nq", 64) > 1.1e10:
        return None
    if op == "search":
        if case["rule"] != "hnsw" and case["nq"] * case["ef"] > 2.5e4:
            return None
        if case["nq"] * case["ef"] ** 2 * case["d"] > 6e9:
            return None
        dd = _search64(case, _queries(case, case["nq"], seed), case["ef"], case["k"], case["rule"], case["eps"],
                       case["mode"])
        return dict(ids=None, dists=dd, stats=None)
    if op == "serve":
        dists = []
        for q, k, ef in _requests(case, seed):
            if ef > 256:
                dists.append(None)
                continue
            dists.append(_search64(case, torch.from_numpy(q).cuda(), ef, k, "hnsw", case["eps"], P.PEOS_MODE_PEOS))
        return dict(ids=[None] * len(dists), dists=dists)
    return None
