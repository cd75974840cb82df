"""The work that users of this library have it do, as measurable cases.

A user's program holds a graph on the GPU and builds its index (exact cosine
or Jaccard, weighted, or approximate), or it holds an index and asks it
(mu, eps) clustering queries: one at a time, in batches, through the server,
or over a parameter grid. Graphs are skewed R-MAT ones (a, b, c, d = .57, .19,
.19, .05; any vertex count: ids of 2^scale past it are dropped) or planted
partitions (stochastic block models), drawn on the GPU. A case's edges are
one fixed draw of its recipe, so that its index has one size; the vertex ids
are shuffled by the seed, and so are weights, random draws and requests.
"""

import math

import torch

import paper_2012_11188_amd as scan

_INDEX_ARRAYS = (("no_ids", scan.ARR_NO_IDS, "<i4", 4), ("no_sim", scan.ARR_NO_SIM, "<f8", 8),
                 ("co_off", scan.ARR_CO_OFF, "<i8", 8), ("co_ids", scan.ARR_CO_IDS, "<i4", 4),
                 ("co_thr", scan.ARR_CO_THR, "<f8", 8))
_SIMS = ("sims", scan.ARR_SIMS, "<f8", 8)


def listed():
    return [
        # The smallest build: 20 blocks of 100 vertices, about 14 neighbours
        # each. Launches and waits count, not bytes.
        {"name": "build-sbm-2000", "path": "build", "graph": "sbm", "n": 2000, "blocks": 20, "degree": 13.7,
         "kind": "cosine", "bits": 32, "keep_sims": False},
        # An ordinary skewed graph, Jaccard, int64 offsets, a vertex count
        # that is no power of two, per-edge similarities kept.
        {"name": "build-rmat-60k", "path": "build", "graph": "rmat", "n": 60000, "edge_factor": 16,
         "kind": "jaccard", "bits": 64, "keep_sims": True},
        # The headline build: scale 20, edge factor 16.
        {"name": "build-rmat-1m", "path": "build", "graph": "rmat", "n": 1 << 20, "edge_factor": 16,
         "kind": "cosine", "bits": 32, "keep_sims": False},
        # The largest build: scale 23, edge factor 32, int64 offsets, hubs of
        # several hundred thousand neighbours.
        {"name": "build-rmat-8m", "path": "build", "graph": "rmat", "n": 1 << 23, "edge_factor": 32,
         "kind": "cosine", "bits": 64, "keep_sims": False},
        # Many graphs of uneven size built in merged launches.
        {"name": "batch-sbm-12", "path": "batch", "graph": "sbm", "graphs": 12, "n_lo": 1000, "n_hi": 1000000,
         "degree_lo": 8.0, "degree_hi": 64.0, "kind": "cosine", "bits": 32},
        # The weighted cosine (full-mantissa weights).
        {"name": "weighted-rmat-1m", "path": "weighted", "graph": "rmat", "n": 1 << 20, "edge_factor": 16,
         "bits": 32},
        # The approximate index: SimHash, and MinHash with int64 offsets.
        {"name": "simhash-rmat-1m", "path": "simhash", "graph": "rmat", "n": 1 << 20, "edge_factor": 16,
         "samples": 256, "bits": 32},
        {"name": "minhash-rmat-1m", "path": "minhash", "graph": "rmat", "n": 1 << 20, "edge_factor": 16,
         "samples": 256, "bits": 64},
        # One query of a small index: a caller that waits for each answer.
        {"name": "query-sbm-2000", "path": "query", "graph": "sbm", "n": 2000, "blocks": 20, "degree": 13.7,
         "mu": 3, "eps": 0.2},
        # Mixed (mu, eps), mu uniform in 2..16, eps on .10, .15, ... .90, answered together.
        {"name": "query-batch-rmat-1m", "path": "query_batch", "graph": "rmat", "n": 1 << 20, "edge_factor": 16,
         "queries": 32},
        # The same mix through the continuous-batching server, results on the device.
        {"name": "serve-rmat-1m", "path": "serve", "graph": "rmat", "n": 1 << 20, "edge_factor": 16,
         "queries": 128, "max_slots": 128, "max_batch": 32},
        # Parameter selection: modularity over the paper's (mu, eps) grid,
        # then the chosen clustering with its hubs and outliers.
        {"name": "select-rmat-100k", "path": "select", "graph": "rmat", "n": 100000, "edge_factor": 16},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(("build", "build", "build", "batch", "weighted", "simhash", "minhash", "query", "query_batch",
                       "serve", "select"))
    case = {"path": path}
    if path == "batch":
        return dict(case, graph="sbm", graphs=rng.randint(2, 12), n_lo=1000, n_hi=_log_uniform(rng, 5000, 1000000),
                    degree_lo=8.0, degree_hi=round(rng.uniform(16.0, 64.0), 1),
                    kind=rng.choice(("cosine", "jaccard")), bits=rng.choice((32, 64)))
    if path in ("build", "query") and rng.random() < 0.3:
        n = _log_uniform(rng, 1000, 400000)
        degree = round(rng.uniform(8.0, 64.0), 1)
        case.update(graph="sbm", n=n, blocks=rng.randint(2, max(2, min(200, int(n / (2 * degree))))), degree=degree)
    else:
        top = {"build": 4000000, "weighted": 1 << 20, "simhash": 1 << 20, "minhash": 1 << 20, "select": 100000}
        n = _log_uniform(rng, 2000, top.get(path, 1 << 20))
        case.update(graph="rmat", n=n, edge_factor=rng.randint(8, 32 if path == "build" else 16))
    if path == "build":
        case.update(kind=rng.choice(("cosine", "jaccard")), bits=rng.choice((32, 64)),
                    keep_sims=rng.choice((False, True)))
    elif path == "weighted":
        case.update(bits=rng.choice((32, 64)))
    elif path in ("simhash", "minhash"):
        case.update(samples=rng.choice((64, 128, 256)), bits=rng.choice((32, 64)))
    elif path == "query":
        case.update(mu=rng.randint(2, 6), eps=rng.randint(2, 12) / 50.0)  # where these graphs have clusters
    elif path == "query_batch":
        case.update(queries=rng.randint(1, 32))
    elif path == "serve":
        batch = rng.choice((1, 8, 32))
        case.update(queries=rng.randint(16, 128), max_slots=4 * batch, max_batch=batch)
    return case


# ---------------------------------------------------------------------------
# Inputs.


_SHUFFLE = 64  # ids are shuffled within runs of this many


def _csr(u, v, n, bits, gen):
    """The simple undirected graph of the pairs (u, v), its ids shuffled by
    gen within short runs (which leaves hubs and blocks where they are): rows
    ascending, both directions, no loops, no repeats."""
    keep = (u != v) & (u < n) & (v < n)
    u, v = u[keep], v[keep]
    del keep
    run = (torch.arange(n, device="cuda") // _SHUFFLE).to(torch.float64)
    label = torch.argsort(run + torch.rand(n, device="cuda", generator=gen, dtype=torch.float64))
    u, v = label[u], label[v]
    key = torch.cat((u * n + v, v * n + u))
    del u, v
    key = torch.sort(key).values
    first = torch.ones_like(key, dtype=torch.bool)
    torch.ne(key[1:], key[:-1], out=first[1:])
    key = key[first]
    del first
    off = torch.searchsorted(key, torch.arange(n + 1, device="cuda", dtype=torch.int64) * n)
    adj = key.remainder_(n).to(torch.int32)
    return off.to(torch.int32 if bits == 32 else torch.int64), adj


def _rmat(n, edge_factor, bits, gen):
    edges = torch.Generator(device="cuda")
    edges.manual_seed(20 + n + edge_factor)
    scale = max(1, (n - 1).bit_length())
    # (pairs with an end past n are dropped)
    count = int(edge_factor * n)
    us, vs = [], []
    while count > 0:
        m = min(count, 1 << 25)
        count -= m
        u = torch.zeros(m, dtype=torch.int64, device="cuda")
        v = torch.zeros(m, dtype=torch.int64, device="cuda")
        for _ in range(scale):
            r = torch.rand(m, device="cuda", generator=edges)
            u.mul_(2).add_(r >= 0.76)
            v.mul_(2).add_(((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
        us.append(u)
        vs.append(v)
    return _csr(torch.cat(us), torch.cat(vs), n, bits, gen)


def _sbm(n, blocks, degree, bits, gen):
    """Planted partition: equal consecutive blocks, p_out = p_in / 50."""
    edges = torch.Generator(device="cuda")
    edges.manual_seed(2000 + n + blocks)
    size = n / blocks
    p_in = min(1.0, degree / ((size - 1) + 0.02 * (n - size)))
    inside, across = int(p_in * n * (size - 1) / 2), int(0.02 * p_in * n * (n - size) / 2)
    u = torch.randint(0, n, (inside + across,), device="cuda", generator=edges)
    lo = torch.floor(torch.floor(u[:inside] / size) * size)
    w = lo + torch.floor(torch.rand(inside, device="cuda", generator=edges, dtype=torch.float64) * size)
    v = torch.cat((w.to(torch.int64).clamp_(max=n - 1),
                   torch.randint(0, n, (across,), device="cuda", generator=edges)))
    return _csr(u, v, n, bits, gen)


def _graph(case, gen):
    bits = case.get("bits", 32)
    if case["graph"] == "rmat":
        return _rmat(case["n"], case["edge_factor"], bits, gen)
    return _sbm(case["n"], case["blocks"], case["degree"], bits, gen)


def _batch_shapes(case):
    """(n, blocks, degree) of each graph: sizes even over the logarithm of
    the range, degrees spread over theirs (golden-ratio steps)."""
    count = case["graphs"]
    shapes = []
    for i in range(count):
        x, y = (i + 0.5) / count, (i * 0.6180339887 + 0.25) % 1.0
        n = int(case["n_lo"] * (case["n_hi"] / case["n_lo"]) ** x)
        degree = case["degree_lo"] + (case["degree_hi"] - case["degree_lo"]) * y
        shapes.append((n, max(2, min(5 + 16 * i, int(n / (2 * degree)))), degree))
    return shapes


def _edge_weights(off, adj, seed):
    """Uniform in [.05, 1), full mantissas, equal for both directions: a hash
    of the edge's two ends."""
    deg = torch.diff(off.to(torch.int64))
    u = torch.repeat_interleave(torch.arange(len(deg), device="cuda"), deg)
    lo, hi = torch.minimum(u, adj.to(torch.int64)), torch.maximum(u, adj.to(torch.int64))
    x = lo * 0x9E3779B97F4A7C1 + hi * 0xC2B2AE3D27D4EB4 + (seed * 0x165667B19E3779F + 12345) % (1 << 62)
    for shift, mult in ((29, 0x3F58476D1CE4E5B9), (32, 0x14D049BB133111EB), (31, 0x2545F4914F6CDD1D)):
        x = (x ^ (x >> shift)) * mult
    unit = ((x >> 11) & ((1 << 53) - 1)).to(torch.float64) / float(1 << 53)
    return 0.05 + 0.95 * unit


def _mix(count, gen):
    """(mu, eps) requests: mu uniform in 2..16, eps on .10, .15, ... .90."""
    mus = torch.randint(2, 17, (count,), generator=gen, device="cuda").tolist()
    eps = [(10 + 5 * k) / 100.0 for k in torch.randint(0, 17, (count,), generator=gen, device="cuda").tolist()]
    return mus, eps


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    state = dict(case)
    path = case["path"]
    if path == "batch":
        state["graphs"] = [_sbm(n, blocks, degree, case["bits"], gen) for n, blocks, degree in _batch_shapes(case)]
        return state
    off, adj = _graph(case, gen)
    if path in ("build", "weighted", "simhash", "minhash"):
        state["off"], state["adj"] = off, adj
        n = off.numel() - 1
        if path == "weighted":
            state["weights"] = _edge_weights(off, adj, seed)
        elif path == "simhash":
            state["gauss"] = torch.randn((n, case["samples"]), generator=gen, device="cuda", dtype=torch.float64)
        elif path == "minhash":
            state["perm"] = torch.randperm(n, generator=gen, device="cuda").to(torch.uint32)
        return state
    # The programs that ask keep the index, not the graph.
    index = scan.scan_build_index(off, adj, scan.COSINE)
    state["index"] = index
    if path in ("query_batch", "serve"):
        state["mus"], state["epss"] = _mix(case["queries"], gen)
    if path == "serve":
        n = case["n"]
        state["server"] = scan.Server(index, case["max_slots"], case["max_batch"], 9 * (n + 64) * case["max_slots"])
        state["results"] = torch.empty((case["queries"], n), dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
    elif path == "select":
        grid = scan.paper_sweep_grid(index.info.dmax)
        state["mus"], state["epss"] = [mu for mu, _ in grid], [eps for _, eps in grid]
    return state


# ---------------------------------------------------------------------------
# One pass.


class _DeviceArray:
    """An index array where it lies on the GPU; keeps its index alive."""

    def __init__(self, index, what, typestr, itemsize):
        ptr, size = scan.scan_index_device_ptr(index, what)
        self.index = index
        self.__cuda_array_interface__ = {"shape": (size // itemsize,), "typestr": typestr, "data": (ptr, False),
                                         "version": 2}


def _arrays(index, sims=False):
    named = _INDEX_ARRAYS + ((_SIMS,) if sims else ())
    return {name: torch.as_tensor(_DeviceArray(index, what, typestr, itemsize), device="cuda")
            for name, what, typestr, itemsize in named}


_KINDS = {"cosine": scan.COSINE, "jaccard": scan.JACCARD}


def run(state):
    path = state["path"]
    if path == "build":
        flags = scan.SCAN_KEEP_SIMS if state["keep_sims"] else 0
        return _arrays(scan.scan_build_index(state["off"], state["adj"], _KINDS[state["kind"]], flags),
                       state["keep_sims"])
    if path == "batch":
        return [_arrays(ix) for ix in scan.scan_build_index_batch(state["graphs"], _KINDS[state["kind"]])]
    if path == "weighted":
        return _arrays(scan.scan_build_index_weighted(state["off"], state["adj"], state["weights"]))
    if path == "simhash":
        return _arrays(scan.scan_build_index_lsh(state["off"], state["adj"], scan.COSINE, state["samples"],
                                                 gauss=state["gauss"]))
    if path == "minhash":
        return _arrays(scan.scan_build_index_lsh(state["off"], state["adj"], scan.JACCARD, state["samples"],
                                                 perm=state["perm"]))
    index = state["index"]
    if path == "query":
        return list(scan.scan_query_ex(index, state["mu"], state["eps"]))
    if path == "query_batch":
        return scan.scan_query_batch(index, state["mus"], state["epss"])
    if path == "serve":
        server, results = state["server"], state["results"]
        tickets, waited = [], 0
        for mu, eps, dst in zip(state["mus"], state["epss"], results):
            while (ticket := server.submit_ex(mu, eps, dst, block=False)) is None:  # the queue is full
                server.wait(tickets[waited])
                waited += 1
            tickets.append(ticket)
        for ticket in tickets[waited:]:
            server.wait(ticket)
        return results
    quality = scan.scan_sweep_modularity(index, state["mus"], state["epss"])
    best = int(quality.argmax())
    memberships = scan.scan_query(index, state["mus"][best], state["epss"][best])
    return {"quality": quality, "memberships": memberships, "roles": scan.scan_query_roles(index, memberships)}


def work(case):
    """Bytes: each input read once, each output written once (graph sizes as
    expected of the recipe). Operations: the fewest id comparisons are not
    known for these paths; SimHash's multiply-adds are counted."""
    if case["path"] == "batch":
        n = sum(s[0] for s in _batch_shapes(case))
        nnz = sum(s[0] * s[2] for s in _batch_shapes(case))
    else:
        n = case["n"]
        nnz = n * (case["degree"] if case["graph"] == "sbm" else 1.85 * case["edge_factor"])
    path, off = case["path"], case.get("bits", 32) // 8
    if path in ("build", "batch", "weighted", "simhash", "minhash"):
        size = off * n + 4 * nnz + 24 * nnz + (8 * nnz if case.get("keep_sims") or path == "weighted" else 0)
        flops = 0.0
        if path == "simhash":
            size += 8.0 * n * case["samples"]
            flops = 2.0 * nnz * case["samples"]
        elif path == "minhash":
            size += 4.0 * n
        return {"bytes": size, "flops": flops}
    if path == "query":
        return {"bytes": 5 * n, "flops": 0.0}
    if path == "select":  # the index, then the grid's scores, the clustering and the roles
        return {"bytes": 24.0 * nnz + 5.0 * n + 8.0 * 1782, "flops": 0.0}
    return {"bytes": 4.0 * n * case["queries"], "flops": 0.0}


# ---------------------------------------------------------------------------
# What the builds return, from the definitions in 64 bits. Ids and offsets are
# whole numbers and have no such value; similarities are given in the order of
# both indexes.

_MOST_PROBES = 12_000_000_000  # common-neighbour tests that take some seconds


def _edges(off, adj):
    deg = torch.diff(off)
    u = torch.repeat_interleave(torch.arange(len(deg), device="cuda"), deg)
    return deg, u, adj.to(torch.int64)


def _common(off, adj, edges, weights=None):
    """For every edge slot in `edges`: the sum over common neighbours x of
    w(u, x) w(v, x) (weights None: their number)."""
    deg, u, v = _edges(off, adj)
    n = len(deg)
    key = u * n + v
    a, b = u[edges], v[edges]
    swap = deg[a] > deg[b]
    short, other = torch.where(swap, b, a), torch.where(swap, a, b)
    del a, b, swap
    out = torch.zeros(len(edges), dtype=torch.float64, device="cuda")
    ends = torch.cumsum(deg[short], 0)
    total = int(ends[-1]) if len(edges) else 0
    if total > _MOST_PROBES:
        return None
    lo = 0
    while lo < len(edges):
        base = int(ends[lo - 1]) if lo else 0
        hi = min(len(edges), max(lo + 1, int(torch.searchsorted(ends, base + (1 << 27)))))
        reps = deg[short[lo:hi]]
        which = torch.repeat_interleave(torch.arange(lo, hi, device="cuda"), reps)
        start = torch.repeat_interleave(torch.cumsum(reps, 0) - reps, reps)
        slot = off[short[which]] + torch.arange(len(which), device="cuda") - start
        want = other[which] * n + v[slot]
        at = torch.searchsorted(key, want).clamp_(max=len(key) - 1)
        hit = key[at] == want
        part = hit.to(torch.float64) if weights is None else torch.where(hit, weights[slot] * weights[at], 0.0)
        out.index_add_(0, which, part)
        del which, start, slot, want, at, hit, part
        lo = hi
    return out


def _mirrored(off, adj, values, edges):
    """Both directions' values from those of the slots with u < v."""
    deg, u, v = _edges(off, adj)
    n = len(deg)
    full = torch.empty(len(adj), dtype=torch.float64, device="cuda")
    full[edges] = values
    full[torch.searchsorted(u * n + v, v[edges] * n + u[edges])] = values
    return full


def _sorted_rows(row, value):
    by_value = torch.sort(value, descending=True, stable=True)
    by_row = torch.sort(row[by_value.indices], stable=True)
    return by_value.values[by_row.indices]


def _orders(off, adj, sims, keep):
    deg, u, _ = _edges(off, adj)
    no_sim = _sorted_rows(u, sims)
    place = torch.arange(len(adj), device="cuda") - off[u]  # mu - 2 of the entry
    out = {"no_ids": None, "no_sim": no_sim, "co_off": None, "co_ids": None, "co_thr": _sorted_rows(place, no_sim)}
    return dict(out, sims=sims) if keep else out


def _exact_sims(off, adj, kind):
    deg, u, v = _edges(off, adj)
    edges = torch.nonzero(u < v).flatten()
    t = _common(off, adj, edges)
    if t is None:
        return None
    c, a, b = t + 2.0, (deg[u[edges]] + 1).double(), (deg[v[edges]] + 1).double()
    return _mirrored(off, adj, c / torch.sqrt(a * b) if kind == "cosine" else c / (a + b - c), edges)


def _exact_weighted(off, adj, w):
    deg, u, v = _edges(off, adj)
    edges = torch.nonzero(u < v).flatten()
    dot = _common(off, adj, edges, w)
    if dot is None:
        return None
    norm = torch.ones(len(deg), dtype=torch.float64, device="cuda").index_add_(0, u, w * w)
    dot += 2.0 * w[edges]  # x = u and x = v: equal weights of both directions
    return _mirrored(off, adj, dot / torch.sqrt(norm[u[edges]] * norm[v[edges]]), edges)


def _exact_simhash(off, adj, gauss, sims):
    deg, u, v = _edges(off, adj)
    k = gauss.shape[1]
    high = torch.nonzero(deg > k).flatten()
    rank = torch.full((len(deg),), -1, dtype=torch.int64, device="cuda")
    rank[high] = torch.arange(len(high), device="cuda")
    dots = gauss[high].clone()
    slots = torch.nonzero(rank[u] >= 0).flatten()
    for part in torch.split(slots, 1 << 22):
        dots.index_add_(0, rank[u[part]], gauss[v[part]])
    bits = dots >= 0
    for part in torch.split(slots, 1 << 22):
        part = part[rank[v[part]] >= 0]
        h = (bits[rank[u[part]]] != bits[rank[v[part]]]).sum(1)
        sims[part] = torch.cos(math.pi * h.double() / k)
    return sims


def _exact_minhash(off, adj, perm, k, sims):
    deg, u, v = _edges(off, adj)
    n = len(deg)
    perm = perm.to(torch.int64)
    high = torch.nonzero(2 * deg > 3 * k).flatten()
    rank = torch.full((n,), -1, dtype=torch.int64, device="cuda")
    rank[high] = torch.arange(len(high), device="cuda")
    sketch = torch.full((max(1, len(high)) * k,), n, dtype=torch.int64, device="cuda")
    slots = torch.nonzero(rank[u] >= 0).flatten()
    who, what = torch.cat((rank[u[slots]], rank[high])), perm[torch.cat((v[slots], high))]
    sketch.scatter_reduce_(0, who * k + what * k // n, what, "amin")
    sketch = sketch.view(-1, k)
    for part in torch.split(slots, 1 << 20):
        part = part[rank[v[part]] >= 0]
        a, b = sketch[rank[u[part]]], sketch[rank[v[part]]]
        empty = ((a == n) & (b == n)).sum(1)
        match = ((a == b) & (a < n)).sum(1)
        sims[part] = match.double() / (k - empty).double()
    return sims


def exact(case, seed):
    path = case["path"]
    if path not in ("build", "batch", "weighted", "simhash", "minhash"):
        return None
    state = prepare(case, seed)
    graphs = state["graphs"] if path == "batch" else [(state["off"], state["adj"])]
    out = []
    for off, adj in graphs:
        off = off.to(torch.int64)
        if len(adj) > 100_000_000:
            return None
        kind = "jaccard" if path == "minhash" else case.get("kind", "cosine")
        sims = _exact_weighted(off, adj, state["weights"]) if path == "weighted" else _exact_sims(off, adj, kind)
        if sims is None:
            return None
        if path == "simhash":
            sims = _exact_simhash(off, adj, state["gauss"], sims)
        elif path == "minhash":
            sims = _exact_minhash(off, adj, state["perm"], state["samples"], sims)
        out.append(_orders(off, adj, sims, bool(case.get("keep_sims"))))
    return out if path == "batch" else out[0]
