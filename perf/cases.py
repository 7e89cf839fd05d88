"""The work that users of this framework have it do, as cases that can be timed.

A case names one call path of the public interface and its sizes.  Two kinds of
input, as in the repository's workloads: R-MAT graphs (the paper's recursive
generator, symmetrised, no self-loops or duplicates; `n` need not be a power of
two) and 4-neighbour grids, the low-diameter and the high-diameter end of what
is traversed.  Graphs, weights, sources and frontiers are made on the GPU from
the seed alone; a state holds what a program keeps between calls: the resident
graph, its workspaces, output arrays and, for batches, the open batch.
"""
import ctypes
import math

import torch

import paper_1504_04804_amd as fg

DEV = "cuda"


def listed():
    return [
        # one traversal of a tiny graph: launch and per-level latency
        {"name": "bfs_small", "kind": "bfs", "graph": "rmat", "n": 1 << 12, "ef": 16},
        # one interactive query on a resident social-type graph, default options
        {"name": "bfs_call", "kind": "bfs", "graph": "rmat", "n": 1 << 20, "ef": 16},
        # one query on a road-like graph of ragged size, asynchronous push as
        # the server runs it
        {"name": "bfs_grid", "kind": "bfs", "graph": "grid", "rows": 1000, "cols": 1537},
        # the benchmark step: 64 direction-optimizing sources one at a time
        # beside one push query on the largest grid, tuned options
        {"name": "bfs_step", "kind": "step", "n": 1 << 22, "ef": 16, "sources": 64,
         "rows": 4096, "cols": 4096},
        # single-source shortest paths, the paper's R-MAT size and a served grid
        {"name": "sssp_rmat", "kind": "sssp", "graph": "rmat", "n": 1 << 22, "ef": 16},
        {"name": "sssp_grid", "kind": "sssp", "graph": "grid", "rows": 1024, "cols": 1024},
        # full serving batches of the two query kinds
        {"name": "msbfs", "kind": "msbfs", "graph": "rmat", "n": 1 << 20, "ef": 16, "lanes": 64},
        {"name": "mssp", "kind": "mssp", "graph": "rmat", "n": 300_007, "ef": 16, "lanes": 64},
        # the other two primitives, at the size they are reported on
        {"name": "pagerank", "kind": "pagerank", "graph": "rmat", "n": 1 << 22, "ef": 16,
         "iters": 20},
        {"name": "components", "kind": "cc", "graph": "rmat", "n": 1 << 22, "ef": 16},
        # one level by the separate operators, as a program with a loop of its own runs it
        {"name": "operators", "kind": "level", "n": 1 << 20, "ef": 16, "share": 0.02},
        # split + package of one partition's output frontier, with parents
        {"name": "package", "kind": "package", "n": 1 << 20, "ef": 16, "parts": 4, "share": 0.9},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _grid(rng, lo, hi):
    cells = _log(rng, lo, hi)
    rows = max(2, int(math.sqrt(cells) * math.exp(rng.uniform(-0.7, 0.7))))
    return {"graph": "grid", "rows": rows, "cols": max(2, cells // rows)}


def draw(rng):
    kind = rng.choice(["bfs", "bfs", "step", "sssp", "sssp", "msbfs", "mssp", "pagerank", "cc",
                       "level", "package"])
    rmat = lambda lo, hi: {"graph": "rmat", "n": _log(rng, lo, hi), "ef": rng.randint(6, 20)}
    c = {"kind": kind}
    if kind == "bfs":
        c.update(rmat(1000, 4 << 20) if rng.random() < 0.6 else _grid(rng, 1000, 9 << 20))
    elif kind == "step":
        c.update(n=_log(rng, 1 << 16, 3 << 20), ef=rng.randint(6, 18), sources=rng.randint(4, 64))
        g = _grid(rng, 1 << 16, 9 << 20)
        c.update(rows=g["rows"], cols=g["cols"])
    elif kind == "sssp":
        c.update(rmat(1000, 3 << 20) if rng.random() < 0.6 else _grid(rng, 1000, 1 << 20))
    elif kind == "msbfs":
        c.update(rmat(1000, 1 << 20) if rng.random() < 0.6 else _grid(rng, 1000, 1 << 18))
        c["lanes"] = rng.randint(1, 64)
    elif kind == "mssp":
        c.update(rmat(1000, 300_000) if rng.random() < 0.6 else _grid(rng, 1000, 1 << 16))
        c["lanes"] = rng.randint(1, 64)
    elif kind == "pagerank":
        c.update(rmat(1000, 4 << 20) if rng.random() < 0.8 else _grid(rng, 1000, 4 << 20))
        c["iters"] = rng.randint(5, 20)
    elif kind == "cc":
        c.update(rmat(1000, 4 << 20) if rng.random() < 0.6 else _grid(rng, 1000, 9 << 20))
    elif kind == "level":
        c.update(n=_log(rng, 1000, 2 << 20), ef=rng.randint(6, 18),
                 share=round(math.exp(rng.uniform(math.log(0.001), math.log(0.2))), 4))
    else:
        c.update(n=_log(rng, 1000, 1 << 20), ef=rng.randint(6, 16), parts=rng.randint(2, 8),
                 share=round(rng.uniform(0.05, 1.0), 3))
    return c


# ------------------------------------------------------------------ inputs

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 7919 + 17)


def _rmat_csr(n, ef, gen):
    """Undirected simple R-MAT graph (0.57, 0.19, 0.19, 0.05): offsets, columns."""
    scale = max(1, (n - 1).bit_length())
    u = torch.zeros(n * ef, dtype=torch.int64, device=DEV)
    v = torch.zeros_like(u)
    for _ in range(scale):
        r = torch.rand(n * ef, device=DEV, generator=gen)
        u.mul_(2).add_(r >= 0.76)
        v.mul_(2).add_(((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
    u.remainder_(n)
    v.remainder_(n)
    keep = u != v
    u, v = u[keep], v[keep]
    key = torch.unique(torch.cat([u * n + v, v * n + u]))
    row = torch.div(key, n, rounding_mode="floor")
    col = (key - row * n).to(torch.int32)
    off = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    off[1:] = torch.cumsum(torch.bincount(row, minlength=n), 0)
    return off.to(torch.int32), col


def _grid_csr(rows, cols):
    """4-neighbour grid, id = r * cols + c, rows ascending."""
    n = rows * cols
    v = torch.arange(n, device=DEV)
    r, c = torch.div(v, cols, rounding_mode="floor"), v % cols
    has = torch.stack([r > 0, c > 0, c < cols - 1, r < rows - 1], 1)
    nbr = v[:, None] + torch.tensor([-cols, -1, 1, cols], device=DEV)
    off = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    off[1:] = torch.cumsum(has.sum(1), 0)
    return off.to(torch.int32), nbr[has].to(torch.int32)


def _rows_of(off, m):
    n = off.numel() - 1
    deg = (off[1:] - off[:-1]).to(torch.int64)
    return torch.repeat_interleave(torch.arange(n, device=DEV), deg, output_size=m)


def _weights(off, col, seed):
    """Symmetric integer weights in [1, 64], a hash of the edge and the seed."""
    u, v = _rows_of(off, col.numel()), col.to(torch.int64)
    h = torch.minimum(u, v) * 0x9E3779B1 + torch.maximum(u, v) * 0x85EBCA77 + seed * 0xC2B2AE3D
    h = (h ^ (h >> 29)) * 0xBF58476D
    return (1 + ((h ^ (h >> 32)) & 63)).to(torch.int32)


def _csr(case, seed):
    if case.get("graph", "rmat") == "rmat":
        return _rmat_csr(case["n"], case["ef"], _gen(seed))
    off, col = _grid_csr(case["rows"], case["cols"])
    if case["kind"] in ("cc", "pagerank"):
        # on a whole grid these depend on nothing else: a quarter of its edges goes
        n, keep = off.numel() - 1, _weights(off, col, seed) <= 48
        deg = torch.bincount(_rows_of(off, col.numel())[keep], minlength=n)
        off = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
        off[1:] = torch.cumsum(deg, 0)
        off, col = off.to(torch.int32), col[keep].contiguous()
    return off, col


def _sources(off, k, seed):
    cand = torch.nonzero(off[1:] > off[:-1]).flatten()
    at = torch.randperm(cand.numel(), device=DEV, generator=_gen(seed + 1))[:k]
    return cand[at].to(torch.int32)


def _out(n, dtype=torch.int32):
    return torch.empty(n, dtype=dtype, device=DEV)


def _bits(mask):
    """Bitmask words (int64, bit v % 64 of word v / 64) of a boolean vertex mask."""
    n = mask.numel()
    w = torch.zeros((n + 63) // 64 * 64, dtype=torch.int64, device=DEV)
    w[:n] = mask
    shift = torch.arange(64, device=DEV)
    return (w.view(-1, 64) << shift).sum(1)


class _State:
    pass


def prepare(case, seed):
    s = _State()
    s.case = case
    kind = case["kind"]
    if kind == "package":
        return _prepare_package(s, case, seed)
    off, col = _csr(case, seed)
    n = off.numel() - 1
    w = _weights(off, col, seed) if kind in ("sssp", "mssp") else None
    s.g = g = fg.Graph(off, col, w, validate=False)
    if kind == "bfs":
        s.src = int(_sources(off, 1, seed)[0])
        s.opts = fg.bfs_opts() if case["graph"] == "rmat" else \
            fg.bfs_opts(mode=fg.FG_MODE_PUSH, async_levels=64, team_blocks=64)
        s.depth, s.parent, s.stats = _out(n), _out(n), fg.new_stats()
        g.workspace(fg.FG_PRIM_BFS)
    elif kind == "step":
        s.srcs = _sources(off, case["sources"], seed)
        s.opts = fg.bfs_opts(do_a=(1, 100000), big_degree=32, team_blocks=24, grid_blocks=152)
        s.depth, s.parent = _out(len(s.srcs) * n), _out(len(s.srcs) * n)
        s.stats = fg.new_stats_many(len(s.srcs))
        goff, gcol = _grid_csr(case["rows"], case["cols"])
        s.g2 = fg.Graph(goff, gcol, validate=False)
        s.opts2 = fg.bfs_opts(mode=fg.FG_MODE_PUSH, async_levels=128, team_blocks=64,
                              big_degree=32)
        s.depth2, s.parent2, s.stats2 = _out(s.g2.n), _out(s.g2.n), fg.new_stats()
        g.workspace(fg.FG_PRIM_BFS)
        s.g2.workspace(fg.FG_PRIM_BFS)
    elif kind == "sssp":
        s.src = int(_sources(off, 1, seed)[0])
        s.opts = fg.sssp_opts()
        s.dist, s.parent, s.stats = _out(n), _out(n), fg.new_stats()
        g.workspace(fg.FG_PRIM_SSSP)
    elif kind in ("msbfs", "mssp"):
        s.srcs = _sources(off, case["lanes"], seed).tolist()
        s.batch = (fg.MsBatch if kind == "msbfs" else fg.MsspBatch)(g, case["lanes"])
        s.rows = torch.empty((len(s.srcs), n), dtype=torch.int32, device=DEV)
    elif kind == "pagerank":
        s.rank, s.stats = _out(n, torch.float64), fg.new_stats()
        g.workspace(fg.FG_PRIM_PR)
    elif kind == "cc":
        s.label, s.comps = _out(n), torch.zeros(1, dtype=torch.int64, device=DEV)
        g.workspace(fg.FG_PRIM_CC)
    elif kind == "level":
        k = max(1, int(case["share"] * n))
        s.front = _sources(off, k, seed)
        deg = (off[1:] - off[:-1])[s.front.long()]
        s.total = int(deg.sum())
        mask = torch.zeros(n, dtype=torch.bool, device=DEV)
        mask[s.front.long()] = True
        s.seen = _bits(mask)
        s.visited, s.visited_b = s.seen.clone(), s.seen.clone()
        s.next = torch.empty_like(s.seen)
        s.start = torch.where(mask, 0, -1).to(torch.int32)
        s.depth, s.depth_b = s.start.clone(), s.start.clone()
        s.parent, s.parent_b = s.start.clone(), s.start.clone()
        s.cap = 2 * n * case["ef"]
        s.dst = torch.full((s.cap,), -7, dtype=torch.int32, device=DEV)
        s.src = s.dst.clone()
        s.edges = torch.zeros(1, dtype=torch.int64, device=DEV)
        s.q, s.len = _out(n), torch.zeros(1, dtype=torch.int32, device=DEV)
        s.q_b, s.len_b = _out(n), torch.zeros(1, dtype=torch.int32, device=DEV)
        s.read = torch.zeros(1, dtype=torch.int64, device=DEV)
        s.list, s.list_len = torch.full((n,), -1, dtype=torch.int32, device=DEV), \
            torch.zeros(1, dtype=torch.int32, device=DEV)
        s.ws = g.workspace(fg.FG_PRIM_BFS_UNFUSED)
    return s


def _prepare_package(s, case, seed):
    n, parts = case["n"], case["parts"]
    gen = _gen(seed + 2)
    off, col = _rmat_csr(n, case["ef"], _gen(seed))
    owner = torch.randint(parts, (n,), device=DEV, generator=gen).to(torch.uint8)
    s.share = sh = fg.Share(off.cpu().numpy(), col.cpu().numpy(), owner.cpu().numpy(), parts, 0)
    k = max(1, int(case["share"] * sh.n_total))
    s.front = torch.randperm(sh.n_total, device=DEV, generator=gen)[:k].to(torch.int32)
    s.depth = torch.randint(1, 8, (sh.n_total,), device=DEV, generator=gen).to(torch.int32)
    s.parent = torch.randint(sh.n_total, (sh.n_total,), device=DEV, generator=gen).to(torch.int32)
    full = lambda m: torch.full((m,), -7, dtype=torch.int32, device=DEV)
    s.ids, s.dep, s.par, s.local = full(parts * n), full(parts * n), full(parts * n), full(n)
    s.counts, s.local_count = full(parts), full(1)
    s.bufs = fg.PeerBufs(s.ids.data_ptr(), s.dep.data_ptr(), s.par.data_ptr(),
                         s.counts.data_ptr(), s.local.data_ptr(), s.local_count.data_ptr(), n)
    s.ws = sh.workspace(k)
    return s


# -------------------------------------------------------------------- a pass

def _ptr(t):
    return ctypes.c_void_p(t.data_ptr())


def _stream():
    return ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)


def run(s):
    kind = s.case["kind"]
    if kind == "bfs":
        # every reached vertex's parent is asked for, as users do.  Which of
        # several valid parents a direction-optimizing run keeps differs from
        # run to run, so it is an output here only where it is determined:
        # the asynchronous push (the smallest id)
        fg.bfs_into(s.g, s.src, s.depth, s.parent, s.opts, stats=s.stats)
        return (s.depth, s.parent) if s.case["graph"] == "grid" else (s.depth,)
    if kind == "step":
        fg.bfs_corun_into(s.g, s.srcs, s.depth, s.parent, s.opts, None, s.stats, s.g2, 0,
                          s.depth2, s.parent2, s.opts2, stats2=s.stats2, out_stride=s.g.n)
        return s.depth, s.depth2, s.parent2
    if kind == "sssp":
        fg.sssp_into(s.g, s.src, s.dist, s.parent, s.opts, stats=s.stats)
        return s.dist, s.parent
    if kind in ("msbfs", "mssp"):
        for lane, src in enumerate(s.srcs):
            s.batch.admit(lane, src)
        s.batch.step(1 << 20)
        done, _ = s.batch.poll()
        for lane in range(len(s.srcs)):
            s.batch.read(lane, s.rows[lane])
        return done == s.batch.admitted, s.rows
    if kind == "pagerank":
        fg.pagerank_into(s.g, s.rank, 0.85, 0.0, s.case["iters"], stats=s.stats)
        return s.rank
    if kind == "cc":
        fg.cc_into(s.g, s.label, s.comps)
        return s.label, s.comps
    if kind == "level":
        return _run_level(s)
    st = fg.lib().fg_package(s.share.handle, _ptr(s.front), s.front.numel(), None, _ptr(s.depth),
                             _ptr(s.parent), ctypes.byref(s.bufs), _ptr(s.ws), s.ws.numel(),
                             _stream())
    if st != fg.FG_OK:
        raise RuntimeError(fg.last_error())
    return s.ids, s.dep, s.par, s.counts, s.local, s.local_count


def _run_level(s):
    """Forward: advance + filter from the frontier; backward: the pull step
    from the same frontier and the list of what it found."""
    g = s.g
    s.visited.copy_(s.seen)
    s.depth.copy_(s.start)
    s.visited_b.copy_(s.seen)
    s.depth_b.copy_(s.start)
    st = fg.lib().fg_advance(g.handle, _ptr(s.front), s.front.numel(), None, _ptr(s.dst),
                             _ptr(s.src), s.cap, _ptr(s.edges), _ptr(s.ws), s.ws.numel(),
                             _stream())
    if st != fg.FG_OK:
        raise RuntimeError(fg.last_error())
    fg.filter_(g, s.dst, s.src, s.total, s.visited, 0, s.depth, s.parent, s.q, s.len,
               len_dev=s.edges)
    fg.pull_step(g, s.seen, s.visited_b, s.next, 0, s.depth_b, s.parent_b, s.q_b, s.len_b, s.read)
    fg.bitmap_to_queue(g, s.next, s.list, s.list_len, s.ws)
    # the filter's queue order and its choice of parent differ from run to
    # run, and so does the pull step's queue order: left out
    return (s.dst, s.src, s.edges, s.visited, s.depth, s.len, s.visited_b, s.next, s.depth_b,
            s.parent_b, s.len_b, s.read, s.list, s.list_len)


# ------------------------------------------------------- what a pass must move

def work(case):
    """Bytes each input read once and each output written once; a traversal's
    input is the part of the graph that any correct one reads: the offsets and
    one entry per vertex where a vertex may stop at its first hit, all entries
    where every edge counts."""
    def size(c):
        if c.get("graph", "rmat") == "rmat":
            return c["n"], 2 * c["n"] * c["ef"] * 0.95
        n = c["rows"] * c["cols"]
        return n, 4 * n
    kind = case["kind"]
    n, m = size({**case, "graph": "rmat"} if kind == "step" else case)
    flops = 0
    if kind == "bfs":
        b = 4 * n + 8 * n + (4 * n if case["graph"] == "rmat" else 4 * m)
    elif kind == "step":
        n2 = case["rows"] * case["cols"]
        b = case["sources"] * 16 * n + 12 * n2 + 16 * n2
    elif kind == "sssp":
        b = 4 * n + 8 * m + 8 * n
    elif kind == "msbfs":
        b = 4 * n + 4 * m + 4 * n * case["lanes"]
    elif kind == "mssp":
        b = 4 * n + 8 * m + 4 * n * case["lanes"]
    elif kind == "pagerank":
        b = case["iters"] * (4 * m + 4 * n + 16 * n)
        flops = 2 * m * case["iters"]
    elif kind == "cc":
        b = 4 * n + 4 * n + 4 * n
    elif kind == "level":
        k = case["share"] * n
        e = k * m / n
        b = 12 * k + 12 * e + 16 * e + 8 * n + 8 * n + 20 * n
    else:
        k = case["share"] * n
        b = 12 * k + 12 * k + 4 * k
    return {"bytes": b, "flops": flops}


# --------------------------------------------------------------- exact results

def exact(case, seed):
    """The floating outputs (PageRank) by a power iteration in 64 bits over
    the edge list; the other paths return whole numbers."""
    if case["kind"] != "pagerank":
        return None
    off, col = _csr(case, seed)
    n = off.numel() - 1
    col, ends = col.to(torch.int64), off.to(torch.int64)
    deg = (off[1:] - off[:-1]).to(torch.float64)
    rank = torch.full((n,), 1.0 / n, dtype=torch.float64, device=DEV)
    for _ in range(case["iters"]):
        give = torch.where(deg > 0, rank / deg.clamp(min=1), 0.0)
        got = torch.segment_reduce(give[col], "sum", offsets=ends)
        rank = (1 - 0.85) / n + 0.85 * got
    return rank
