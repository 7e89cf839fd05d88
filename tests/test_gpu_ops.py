"""Parity of the standalone operators (advance, filter, pull step, queue /
bitmap conversions) with serial expectations computed from the oracle."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import announce, gpu, need_gpu, to_np

pytestmark = gpu


@pytest.fixture(scope="module")
def fg():
    need_gpu()
    import paper_1504_04804_amd as fg
    fg.lib()
    return fg


def serial_advance(off, col, frontier):
    dst = [col[off[u]:off[u + 1]] for u in frontier]
    src = [np.full(off[u + 1] - off[u], u, np.int32) for u in frontier]
    if not dst:
        return np.zeros(0, np.int32), np.zeros(0, np.int32)
    return np.concatenate(dst), np.concatenate(src)


@pytest.mark.parametrize("scale", [10, 14])
def test_advance_exact_layout(fg, scale):
    off, col = synth.rmat_csr(scale)
    g = fg.Graph(off, col)
    rng = np.random.default_rng(scale)
    n = len(off) - 1
    for size in (0, 1, 63, 64, 65, 1000, n):
        fr = rng.choice(n, size=size, replace=False).astype(np.int32)
        if size and size < n:
            fr[0] = 0  # include the hub
        announce(f"advance scale={scale} size={size}")
        q = torch.from_numpy(fr).cuda() if size else torch.zeros(1, dtype=torch.int32, device="cuda")
        dst, src, tot = fg.advance(g, q[:size] if size else q[:0])
        wd, ws = serial_advance(off, col, fr)
        T = int(to_np(tot)[0])
        assert T == len(wd)
        assert np.array_equal(to_np(dst)[:T], wd)
        assert np.array_equal(to_np(src)[:T], ws)


def test_advance_capacity_overflow(fg):
    off, col = synth.rmat_csr(10)
    g = fg.Graph(off, col)
    q = torch.tensor([0, 1, 2], dtype=torch.int32, device="cuda")
    dst, src, tot = fg.advance(g, q, capacity=10)
    wd, _ = serial_advance(off, col, [0, 1, 2])
    assert int(to_np(tot)[0]) == len(wd)  # the size that would be needed
    assert np.array_equal(to_np(dst)[:10], wd[:10])


def test_filter_heavy_duplicates(fg):
    n = 5000
    off, col = synth.rmat_csr(12)
    g = fg.Graph(off, col)
    rng = np.random.default_rng(1)
    dst = rng.integers(0, 50, size=100000).astype(np.int32)  # heavy duplication
    src = rng.integers(0, n, size=100000).astype(np.int32)
    visited = torch.zeros((4096 + 31) // 32, dtype=torch.int32, device="cuda")
    pre = [3, 7, 49]
    vis_np = np.zeros(len(visited), np.uint32)
    for v in pre:
        vis_np[v >> 5] |= np.uint32(1 << (v & 31))
    visited.copy_(torch.from_numpy(vis_np.view(np.int32)))
    depth = torch.full((4096,), -1, dtype=torch.int32, device="cuda")
    parent = torch.full((4096,), -1, dtype=torch.int32, device="cuda")
    out_q = torch.empty(4096, dtype=torch.int32, device="cuda")
    out_len = torch.zeros(1, dtype=torch.int32, device="cuda")
    announce("filter duplicates")
    fg.filter_(g, torch.from_numpy(dst).cuda(), torch.from_numpy(src).cuda(), len(dst), visited,
               4, depth, parent, out_q, out_len)
    k = int(to_np(out_len)[0])
    got = to_np(out_q)[:k]
    want = sorted(set(dst.tolist()) - set(pre))
    assert sorted(got.tolist()) == want  # each vertex once
    d = to_np(depth)
    p = to_np(parent)
    assert (d[want] == 5).all() and (d[pre] == -1).all()
    for v in want:  # parent is one of the edges that reached v
        assert p[v] in set(src[dst == v].tolist())
    vis = to_np(visited).view(np.uint32)
    for v in want + pre:
        assert vis[v >> 5] >> (v & 31) & 1


def test_pull_step_matches_level(fg, orc):
    off, col = synth.rmat_csr(13)
    n = len(off) - 1
    g = fg.Graph(off, col)
    depth_ref, _, cnt, _ = orc.bfs(off, col, 0)
    nw = (n + 63) // 64
    for k in range(len(cnt)):
        # state at the start of iteration k: visited = depth <= k, frontier = depth == k
        vis = np.zeros(nw, np.uint64)
        fb = np.zeros(nw, np.uint64)
        for v in np.flatnonzero((depth_ref >= 0) & (depth_ref <= k)):
            vis[v >> 6] |= np.uint64(1) << np.uint64(v & 63)
        for v in np.flatnonzero(depth_ref == k):
            fb[v >> 6] |= np.uint64(1) << np.uint64(v & 63)
        T = lambda a: torch.from_numpy(a.view(np.int64)).cuda()
        visited, fbits = T(vis.copy()), T(fb)
        nxt = torch.full((nw,), -1, dtype=torch.int64, device="cuda")
        depth = torch.full((n,), -1, dtype=torch.int32, device="cuda")
        parent = torch.full((n,), -1, dtype=torch.int32, device="cuda")
        out_q = torch.empty(n, dtype=torch.int32, device="cuda")
        out_len = torch.zeros(1, dtype=torch.int32, device="cuda")
        insp = torch.zeros(1, dtype=torch.int64, device="cuda")
        announce(f"pull step k={k}")
        fg.pull_step(g, fbits, visited, nxt, k, depth, parent, out_q, out_len, insp)
        want_new = np.flatnonzero(depth_ref == k + 1)
        got = to_np(out_q)[:int(to_np(out_len)[0])]
        assert sorted(got.tolist()) == want_new.tolist()
        d = to_np(depth)
        p = to_np(parent)
        assert np.array_equal(np.flatnonzero(d == k + 1), want_new)
        for v in want_new:  # early exit: first neighbour in CSR order at depth k
            row = col[off[v]:off[v + 1]]
            assert p[v] == row[np.argmax(depth_ref[row] == k)]
        dirs = np.ones(k + 1, np.int8)
        assert int(to_np(insp)[0]) == orc.edges_inspected(off, col, depth_ref, dirs)[k]
        nb = to_np(nxt).view(np.uint64)
        want_nb = np.zeros(nw, np.uint64)
        for v in want_new:
            want_nb[v >> 6] |= np.uint64(1) << np.uint64(v & 63)
        assert np.array_equal(nb, want_nb)
        assert np.array_equal(to_np(visited).view(np.uint64), vis | want_nb)


def test_queue_bitmap_roundtrip(fg):
    off, col = synth.rmat_csr(12)
    n = len(off) - 1
    g = fg.Graph(off, col)
    rng = np.random.default_rng(5)
    for size in (0, 1, 64, 777, n):
        q = np.sort(rng.choice(n, size=size, replace=False)).astype(np.int32)
        bits = torch.zeros((n + 63) // 64, dtype=torch.int64, device="cuda")
        qt = torch.from_numpy(q).cuda() if size else torch.zeros(0, dtype=torch.int32, device="cuda")
        fg.queue_to_bitmap(g, qt, size, bits)
        out = torch.empty(n, dtype=torch.int32, device="cuda")
        out_len = torch.zeros(1, dtype=torch.int32, device="cuda")
        fg.bitmap_to_queue(g, bits, out, out_len)
        k = int(to_np(out_len)[0])
        assert k == size
        assert np.array_equal(to_np(out)[:k], q)  # ascending order


def test_graph_validation_errors(fg):
    off, col = synth.from_edge_pairs(4, [(0, 1), (1, 2)])
    bad_col = col.copy()
    bad_col[0] = 7
    with pytest.raises(fg.FGError) as e:
        fg.Graph(off, bad_col)
    assert e.value.status == fg.FG_EINVAL
    bad_off = off.copy()
    bad_off[2] = 0
    with pytest.raises(fg.FGError):
        fg.Graph(bad_off, col)
    # directed graph claimed symmetric
    doff = np.array([0, 1, 1, 1, 1], np.int32)
    dcol = np.array([1], np.int32)
    with pytest.raises(fg.FGError):
        fg.Graph(doff, dcol, symmetric=True)
    g = fg.Graph(doff, dcol, symmetric=False)
    with pytest.raises(fg.FGError) as e:
        fg.bfs(g, 0, mode=fg.FG_MODE_DO)
    assert e.value.status == fg.FG_EUNSUPPORTED
    d, p, st = fg.bfs(g, 0, mode=fg.FG_MODE_PUSH)  # push works on directed graphs
    assert to_np(d).tolist() == [0, 1, -1, -1]
    with pytest.raises(fg.FGError) as e:
        fg.bfs(g, 4, mode=fg.FG_MODE_PUSH)
    assert e.value.status == fg.FG_EINVAL
    ws = torch.empty(16, dtype=torch.uint8, device="cuda")
    depth = torch.empty(4, dtype=torch.int32, device="cuda")
    with pytest.raises(fg.FGError) as e:
        fg.bfs_into(g, 0, depth, None, fg.bfs_opts(mode=1), ws=ws)
    assert e.value.status == fg.FG_ENOMEM


@pytest.mark.parametrize("edges", [1, 8191, 8192, 8193, 12_800_000])
def test_filter_tile_edges(fg, edges):
    """Lengths at the filter's tile borders and past three tiles per workgroup
    with every edge a winner (staged entries written out inside the loop)."""
    n = max(64, edges)
    g = fg.Graph(torch.zeros(n + 1, dtype=torch.int32, device="cuda"),
                 torch.zeros(0, dtype=torch.int32, device="cuda"), validate=False)
    announce(f"filter tile edges={edges}")
    gen = torch.Generator(device="cuda").manual_seed(edges)
    dst = torch.randperm(n, device="cuda", generator=gen)[:edges].to(torch.int32)
    dst[edges // 2] = dst[0]  # one duplicate
    src = torch.arange(edges, device="cuda", dtype=torch.int32)
    visited = torch.zeros((n + 63) // 64 * 2, dtype=torch.int32, device="cuda")
    depth = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    parent = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    out_q = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    out_len = torch.zeros(1, dtype=torch.int32, device="cuda")
    fg.filter_(g, dst, src, edges, visited, 2, depth, parent, out_q, out_len)
    k = int(to_np(out_len)[0])
    want = torch.unique(dst)
    assert torch.equal(torch.sort(out_q[:k]).values, want) and bool((out_q[k:] == -1).all())
    assert torch.equal(torch.nonzero(depth == 3).flatten().int(), want)
    assert torch.equal(dst[parent[want.long()].long()], want)
    bits = (visited[torch.arange(n, device="cuda") >> 5] >> (torch.arange(n, device="cuda") & 31)) & 1
    assert torch.equal(torch.nonzero(bits).flatten().int(), want)


@pytest.mark.parametrize("hit", ["none", "first", "last", "random"])
def test_pull_step_row_lengths(fg, hit):
    """Rows around the lengths where the pull step changes how it scans (4, 32,
    256 past the first four), their only frontier neighbour nowhere, first,
    last or anywhere: parent, next bits and the early-exit count."""
    rng = np.random.default_rng(7)
    degs = [1, 2, 3, 4, 5, 7, 8, 9, 31, 32, 33, 35, 36, 37, 63, 64, 65, 67, 68, 69, 259, 260, 261,
            515, 516, 517, 2000] * 5
    H, P = len(degs), 2500
    pairs = []
    for v, d in enumerate(degs):
        pairs += [(v, H + int(x)) for x in rng.choice(P, size=d, replace=False)]
    off, col = synth.from_edge_pairs(H + P, pairs)
    n = len(off) - 1
    front = np.zeros(n, bool)
    if hit == "random":
        front[H + rng.choice(P, size=25, replace=False)] = True
    seen = np.zeros(n, bool)
    seen[H:] = True  # only the long rows' own vertices are candidates
    exp_p = np.full(n, -1, np.int64)
    insp = 0
    if hit in ("first", "last"):
        for v in range(H):
            front[col[off[v] if hit == "first" else off[v + 1] - 1]] = True
    for v in range(H):
        at = np.flatnonzero(front[col[off[v]:off[v + 1]]])
        if len(at):
            exp_p[v] = col[off[v] + at[0]]
            insp += int(at[0]) + 1
        else:
            insp += int(off[v + 1] - off[v])
    nw = (n + 63) // 64
    def words(mask):
        m = np.zeros(nw * 64, np.uint64)
        m[:n] = mask
        return torch.from_numpy((m.reshape(nw, 64) << np.arange(64, dtype=np.uint64)).sum(1)
                                .astype(np.uint64).view(np.int64)).cuda()
    g = fg.Graph(off, col)
    visited, fbits = words(seen), words(front)
    nxt = torch.full((nw,), -1, dtype=torch.int64, device="cuda")
    depth = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    parent = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    out_q = torch.empty(n, dtype=torch.int32, device="cuda")
    out_len = torch.zeros(1, dtype=torch.int32, device="cuda")
    cnt = torch.full((1,), 99, dtype=torch.int64, device="cuda")
    announce(f"pull step row lengths hit={hit}")
    fg.pull_step(g, fbits, visited, nxt, 4, depth, parent, out_q, out_len, cnt)
    new = exp_p >= 0
    assert np.array_equal(to_np(parent), exp_p)
    assert np.array_equal(to_np(depth), np.where(new, 5, -1))
    assert int(to_np(cnt)[0]) == insp
    assert sorted(to_np(out_q)[:int(to_np(out_len)[0])].tolist()) == np.flatnonzero(new).tolist()
    assert torch.equal(nxt, words(new)) and torch.equal(visited, words(seen | new))


@pytest.mark.parametrize("n", [16384 * 2048, 16384 * 2048 + 1, 16384 * 2048 + 70_000])
def test_bitmap_to_queue_many_tiles(fg, n):
    """Both sides of the size at which the tile sums get a kernel of their own."""
    g = fg.Graph(torch.zeros(n + 1, dtype=torch.int32, device="cuda"),
                 torch.zeros(0, dtype=torch.int32, device="cuda"), validate=False)
    gen = torch.Generator(device="cuda").manual_seed(3)
    q = torch.unique(torch.randint(n, (200_000,), device="cuda", generator=gen))
    q = torch.unique(torch.cat([q, torch.tensor([0, 63, 64, n - 1], device="cuda")]))
    bits = torch.zeros((n + 63) // 64, dtype=torch.int64, device="cuda")
    bits.index_put_((q >> 6,), torch.ones_like(q) << (q & 63), accumulate=True)
    out = torch.empty(n, dtype=torch.int32, device="cuda")
    out_len = torch.zeros(1, dtype=torch.int32, device="cuda")
    announce(f"bitmap to queue n={n}")
    fg.bitmap_to_queue(g, bits, out, out_len, ws=g.workspace(fg.FG_PRIM_BFS_UNFUSED))
    assert int(to_np(out_len)[0]) == q.numel()
    assert torch.equal(out[:q.numel()], q.to(torch.int32))


@pytest.mark.parametrize("length", [1024 * 2048, 1024 * 2048 + 1])
def test_advance_many_tiles(fg, length):
    """The same border for the advance's scan over the frontier's degrees."""
    off, col = synth.grid_csr(1500, 1500)
    g = fg.Graph(off, col, validate=False)
    gen = torch.Generator(device="cuda").manual_seed(length)
    q = torch.randperm(g.n, device="cuda", generator=gen)[:length].to(torch.int32)
    announce(f"advance many tiles length={length}")
    dst, src, tot = fg.advance(g, q)
    o = torch.from_numpy(off).cuda().long()
    deg = (o[1:] - o[:-1])[q.long()]
    T = int(deg.sum())
    assert int(to_np(tot)[0]) == T
    wsrc = torch.repeat_interleave(q, deg)
    first = torch.repeat_interleave(torch.cumsum(deg, 0) - deg, deg)
    at = o[wsrc.long()] + torch.arange(T, device="cuda") - first
    assert torch.equal(src[:T], wsrc)
    assert torch.equal(dst[:T], torch.from_numpy(col).cuda()[at])


def _time_us(f, reps=20):
    f()
    a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    a.record()
    for _ in range(reps):
        f()
    b.record()
    torch.cuda.synchronize()
    return a.elapsed_time(b) / reps * 1000


@pytest.mark.parametrize("step,k", [(131072, 512), (4096, 16384), (65536 + 32, 1000),
                                    (32 * 37, 50000)])
def test_filter_of_spread_words(fg, step, k):
    """Edges whose vertices lie in words far apart (a wide grid's column) are
    filtered as well as the same number in neighbouring words, and take about
    as long (the table's slots, of which a word has one, are 4096)."""
    n = 1 << 26
    g = fg.Graph(np.zeros(n + 1, np.int32), np.zeros(0, np.int32))
    vis = torch.zeros(n // 64, dtype=torch.int64, device="cuda")
    dep = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    par, q = torch.zeros_like(dep), torch.zeros_like(dep)
    ln = torch.zeros(1, dtype=torch.int32, device="cuda")
    us = {}
    for st in (32, step):
        v = (torch.arange(k, device="cuda") * st % n).to(torch.int32)
        src = v + 1

        def run():
            vis.zero_()
            fg.filter_(g, v, src, k, vis, 4, dep, par, q, ln)
        announce(f"filter of {k} edges, {st} vertices apart")
        dep.fill_(-1)
        us[st] = _time_us(run)
        assert int(ln) == k and np.array_equal(np.sort(to_np(q[:k])), np.sort(to_np(v)))
        assert int((dep[v.long()] == 5).sum()) == k == int((dep >= 0).sum())
        assert torch.equal(par[v.long()], src)
    assert us[step] < 5 * us[32], us  # with a round per word of a slot 20 to 100 times
    g.close()


@pytest.mark.parametrize("n", [1, 64, 5000, 300000, (1 << 21) + 77])
def test_bitmap_to_queue_densities(fg, n):
    """Sparse words are listed by a lane each, full ones by their wave; both
    kinds in one bitmap, and none."""
    g = fg.Graph(np.zeros(n + 1, np.int32), np.zeros(0, np.int32))
    rng = np.random.default_rng(n)
    q = torch.zeros(n, dtype=torch.int32, device="cuda")
    ln = torch.zeros(1, dtype=torch.int32, device="cuda")
    for dens in (0.0, 0.001, 0.05, 0.2, 0.26, 0.5, 1.0, None):
        p = rng.choice([0.0, 0.02, 0.9], size=n // 4096 + 1).repeat(4096)[:n] if dens is None else dens
        want = np.flatnonzero(rng.random(n) < p)
        bits = np.zeros((n + 63) // 64 * 64, np.uint8)
        bits[want] = 1
        words = np.packbits(bits, bitorder="little").view(np.int64)
        announce(f"bitmap_to_queue n={n} density {dens}")
        fg.bitmap_to_queue(g, torch.from_numpy(words.copy()).cuda(), q, ln)
        assert int(ln) == len(want) and np.array_equal(to_np(q[:len(want)]), want)
    g.close()
