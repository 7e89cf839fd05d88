"""Parity of the HIP SSSP path with the oracle's Dijkstra: distances and the
canonical (smallest-id tight) parents must match bit-exactly."""
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


def check(fg, orc, g, off, col, w, src, **kw):
    announce(f"sssp n={len(off)-1} m={len(col)} src={src} {kw}")
    dist, parent, st = fg.sssp(g, src, **kw)
    d = to_np(dist).astype(np.uint32)
    p = to_np(parent)
    wd, wp = orc.dijkstra(off, col, w, src)
    assert st.status == 0
    assert np.array_equal(d, wd), f"dist mismatch at {np.flatnonzero(d != wd)[:10]}"
    assert np.array_equal(p, wp), f"parent mismatch at {np.flatnonzero(p != wp)[:10]}"
    assert orc.check_sssp(off, col, w, src, d, p) is None
    assert st.reached == int((wd != 0xFFFFFFFF).sum())
    return st


@pytest.mark.parametrize("scale", [10, 12, 16])
def test_rmat_weighted(fg, orc, scale):
    off, col = synth.rmat_csr(scale)
    w = synth.weights(off, col)
    g = fg.Graph(off, col, weights=w)
    for s in [0] + list(synth.sources(off, 3, seed=scale)):
        check(fg, orc, g, off, col, w, int(s))
    check(fg, orc, g, off, col, w, 0, small_frontier=1, small_edges=1)
    check(fg, orc, g, off, col, w, 0, big_degree=2)
    # near-far steps: tiny (many splits, large piles split by the whole
    # grid), below and above the largest weight, and no threshold at all
    for delta in (1, 7, 64, 500, fg.SSSP_NO_THRESHOLD):
        check(fg, orc, g, off, col, w, 0, delta=delta)
    check(fg, orc, g, off, col, w, 0, delta=3, small_frontier=1, small_edges=1)


@pytest.mark.parametrize("delta", [0, 1, 33, 600, 0xFFFFFFFF])
def test_grid_near_far(fg, orc, delta):
    off, col = synth.grid_csr(300, 300)
    w = synth.weights(off, col)
    g = fg.Graph(off, col, weights=w)
    for s in (0, 300 * 150 + 150, 300 * 300 - 1):
        st = check(fg, orc, g, off, col, w, s, delta=delta)
        if delta == 1:
            assert st.iterations > 500  # about one split per distance value


@pytest.mark.parametrize("team,team_e,delta", [(2, 0, 0), (5, 0, 1), (32, 0, 0), (64, 0, 600),
                                               (32, 40, 0), (-1, 0, 0), (3, 0, 0xFFFFFFFF)])
def test_team_mode(fg, orc, team, team_e, delta):
    # small_frontier=1 sends every frontier of more than one vertex to the
    # team (or the full grid when its mean degree is too high)
    off, col = synth.grid_csr(200, 220)
    w = synth.weights(off, col)
    g = fg.Graph(off, col, weights=w)
    for s in (0, 200 * 110 + 37):
        check(fg, orc, g, off, col, w, s, small_frontier=1, small_edges=1, team_blocks=team,
              team_edges=team_e, delta=delta)
    off, col = synth.rmat_csr(13)
    w = synth.weights(off, col)
    g = fg.Graph(off, col, weights=w)
    check(fg, orc, g, off, col, w, 0, small_frontier=1, small_edges=1, team_blocks=team,
          team_edges=team_e, delta=delta)
    check(fg, orc, g, off, col, w, 77, team_blocks=team, team_edges=team_e, delta=delta)


def test_team_handoffs_repeated(fg, orc):
    # back-to-back launches with the team forced on R-MAT and the solo
    # threshold varied, so episodes hand off to each other in quick
    # succession; every run must finish with Dijkstra's distances
    off, col = synth.rmat_csr(14)
    w = synth.weights(off, col)
    g = fg.Graph(off, col, weights=w)
    srcs = [int(s) for s in synth.sources(off, 4, seed=7)]
    want = {s: orc.dijkstra(off, col, w, s)[0] for s in srcs}
    announce("sssp team hand-offs: 60 runs on rmat14")
    for r in range(60):
        s = srcs[r % 4]
        dist, _, st = fg.sssp(g, s, team_blocks=32, small_frontier=(r % 3) * 300 + 1)
        assert st.status == 0, f"run {r}: status {st.status}"
        assert np.array_equal(to_np(dist).astype(np.uint32), want[s]), f"run {r} src {s}"


def test_near_far_gaps(fg, orc):
    # weights far above the step: each split first finds no vertex below the
    # new threshold and jumps to the smallest distance in the pile
    n = 50
    off, col = synth.from_edge_pairs(n, [(i, i + 1) for i in range(n - 1)] + [(0, 25)])
    w = np.full(len(col), 1000, np.uint32)
    g = fg.Graph(off, col, weights=w)
    for delta in (1, 999, 1000, 1001):
        check(fg, orc, g, off, col, w, 0, delta=delta)
        check(fg, orc, g, off, col, w, 0, delta=delta, small_frontier=1, small_edges=1)


def test_closed_forms(fg, orc):
    n = 200
    off, col = synth.from_edge_pairs(n, [(i, i + 1) for i in range(n - 1)])
    wt = np.arange(1, n, dtype=np.uint32)
    w = np.array([wt[min(u, col[k])] for u in range(n) for k in range(off[u], off[u + 1])], np.uint32)
    g = fg.Graph(off, col, weights=w)
    st = check(fg, orc, g, off, col, w, 0)
    R, C = 40, 50
    off, col = synth.grid_csr(R, C)
    w = np.full(len(col), 7, np.uint32)
    g = fg.Graph(off, col, weights=w)
    for delta in (0, 1, 7, 50, fg.SSSP_NO_THRESHOLD):
        dist, parent, st = fg.sssp(g, 0, delta=delta)
        d = to_np(dist)
        assert d.tolist() == [7 * (r + c) for r in range(R) for c in range(C)]
    check(fg, orc, g, off, col, w, R * C // 2 + 7)


def test_zero_weights_and_isolated(fg, orc):
    off, col = synth.rmat_csr(11)
    w = synth.weights(off, col) % 3  # many zero weights (symmetric)
    g = fg.Graph(off, col, weights=w)
    for s in (0, 17):
        check(fg, orc, g, off, col, w, s)
    off, col = synth.from_edge_pairs(6, [(0, 1), (1, 2)])
    w = np.ones(len(col), np.uint32)
    g = fg.Graph(off, col, weights=w)
    check(fg, orc, g, off, col, w, 5)  # isolated source


def test_directed_graph(fg, orc):
    rng = np.random.default_rng(3)
    n = 3000
    eu = rng.integers(0, n, 20000)
    ev = rng.integers(0, n, 20000)
    keep = eu != ev
    pairs = np.unique(np.stack([eu[keep], ev[keep]], 1), axis=0)
    order = np.lexsort((pairs[:, 1], pairs[:, 0]))
    pairs = pairs[order]
    off = np.zeros(n + 1, np.int32)
    np.add.at(off, pairs[:, 0] + 1, 1)
    off = np.cumsum(off).astype(np.int32)
    col = pairs[:, 1].astype(np.int32)
    w = rng.integers(1, 65, len(col)).astype(np.uint32)
    g = fg.Graph(off, col, weights=w, symmetric=False)
    for s in (0, 1, 2):
        check(fg, orc, g, off, col, w, s)


def test_overflow_reported(fg):
    off, col = synth.from_edge_pairs(3, [(0, 1), (1, 2)])
    w = np.full(len(col), 0x90000000, np.uint32)
    g = fg.Graph(off, col, weights=w)
    dist, parent, st = fg.sssp(g, 0)
    assert st.status == fg.FG_EOVERFLOW


def test_sssp_needs_weights(fg):
    off, col = synth.from_edge_pairs(3, [(0, 1)])
    g = fg.Graph(off, col)
    with pytest.raises(fg.FGError) as e:
        fg.sssp(g, 0)
    assert e.value.status == fg.FG_EINVAL


@pytest.mark.slow
def test_config_rmat22_sssp_sampled(fg, orc):
    off, col = synth.rmat_csr(22)
    w = synth.weights(off, col)
    g = fg.Graph(off, col, weights=w)
    for s in synth.sources(off, 64)[:2]:
        check(fg, orc, g, off, col, w, int(s))


@pytest.mark.parametrize("rows,cols,delta,wmax", [
    (1, 2, 0, 64), (1, 5000, 0, 64), (60, 50, 0, 64), (128, 128, 0, 64),
    (129, 128, 0, 64), (300, 250, 0, 64), (300, 250, 5, 64), (300, 250, 0xFFFFFFFF, 64),
    (257, 260, 0, 0), (257, 260, 40, 1), (260, 270, 300, 3), (700, 900, 0, 64)])
def test_async_team(fg, orc, rows, cols, delta, wmax):
    """The default path of low-degree graphs: one to sixteen members; tiny and
    no thresholds (near vertices that find no room in LDS); zero weights (a
    neighbour that a vertex was reached from may still be its predecessor)."""
    off, col = synth.grid_csr(rows, cols)
    w = synth.weights(off, col) if wmax == 64 else synth.weights(off, col) % np.uint32(wmax + 1)
    g = fg.Graph(off, col, weights=w)
    n = rows * cols
    for s in (0, n // 2 + cols // 3 if n > 2 else 0, n - 1):
        st = check(fg, orc, g, off, col, w, s, delta=delta)
        assert st.grid_blocks <= 64 or n > 16384  # from sixteen members on the team may hand over
        st = check(fg, orc, g, off, col, w, s, delta=delta)  # the workspace is left ready
    d, p, st = fg.sssp(g, 0, parents=False, delta=delta)
    assert np.array_equal(to_np(d), orc.dijkstra(off, col, w, 0)[0])


def test_async_team_long_rows_and_handover(fg, orc):
    """Rows past the four entries carried in the queue, a directed graph, and
    a vertex whose neighbours do not fit the members' queues (the
    level-synchronous kernel takes over), then a plain query again."""
    rng = np.random.default_rng(3)
    n = 9000
    eu = np.concatenate([np.arange(n - 1), rng.integers(0, n, 2 * n)]).astype(np.int32)
    ev = np.concatenate([np.arange(1, n), rng.integers(0, n, 2 * n)]).astype(np.int32)
    off, col = orc.csr_from_edges(n, eu, ev)
    assert len(col) <= 8 * n and np.diff(off).max() > 8
    w = synth.weights(off, col)
    g = fg.Graph(off, col, weights=w)
    for s in (0, 17, n - 1):
        assert check(fg, orc, g, off, col, w, s).grid_blocks == 8
    keep = rng.random(len(col)) < 0.7  # directed: rows lose entries at random
    deg = np.add.reduceat(np.append(keep, False).astype(np.int64), off[:-1]) * (np.diff(off) > 0)
    doff = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    dcol, dw = col[keep], w[keep]
    gd = fg.Graph(doff, dcol, weights=dw, symmetric=False)
    for s in (0, 4000):
        check(fg, orc, gd, doff, dcol, dw, s)
    # wide fronts on sixteen and on 64 members: handed over to the whole grid
    for size in (60_000, 400_000):
        eu, ev = rng.integers(0, size, (2, 2 * size)).astype(np.int32)
        off, col = orc.csr_from_edges(size, eu, ev)
        w = synth.weights(off, col)
        g = fg.Graph(off, col, weights=w)
        for delta in (0, 20, 0xFFFFFFFF):
            for s in (0, 5):
                st = check(fg, orc, g, off, col, w, int(col[off[s]]) if off[s + 1] > off[s] else s,
                           delta=delta)
                assert st.grid_blocks in (256, 16, 64)
    assert st.grid_blocks == 256


def test_async_team_near_vertices_without_room(fg, orc):
    """Hubs (below the degree at which the team is not tried) whose neighbours
    do not fit the members' queues: they wait in the far pile."""
    hubs, per = 60, 250
    n = hubs * per + hubs
    leaves = np.arange(hubs, n, dtype=np.int32)
    eu = np.concatenate([leaves % hubs, np.zeros(hubs - 1)]).astype(np.int32)
    ev = np.concatenate([leaves, np.arange(1, hubs)]).astype(np.int32)
    off, col = orc.csr_from_edges(n, eu, ev)
    assert np.diff(off).max() > 256
    w = synth.weights(off, col) % np.uint32(3)
    g = fg.Graph(off, col, weights=w)
    for s in (0, 1, n - 1):
        check(fg, orc, g, off, col, w, s)
    # the same below the border: a path of hubs
    eu = np.concatenate([leaves % hubs, np.arange(hubs - 1)]).astype(np.int32)
    ev = np.concatenate([leaves, np.arange(1, hubs)]).astype(np.int32)
    off, col = orc.csr_from_edges(n, eu, ev)
    assert 250 < np.diff(off).max() <= 256
    for mod in (1, 3, 65):
        w = synth.weights(off, col) % np.uint32(mod)
        g = fg.Graph(off, col, weights=w)
        for s in (0, 1, n - 1):
            assert check(fg, orc, g, off, col, w, s, delta=0xFFFFFFFF).grid_blocks <= 8
            check(fg, orc, g, off, col, w, s)


@pytest.mark.parametrize("blocks", [1, 65, 200])
def test_explicit_width(fg, orc, blocks):
    """grid_blocks is the launch's width also where the default is narrower."""
    off, col = synth.rmat_csr(13)
    w = synth.weights(off, col)
    g = fg.Graph(off, col, weights=w)
    assert check(fg, orc, g, off, col, w, 3).grid_blocks == 64
    assert check(fg, orc, g, off, col, w, 3, grid_blocks=blocks).grid_blocks == blocks


@pytest.mark.parametrize("rows,cols", [(1, 40), (40, 50), (150, 140), (700, 900)])
def test_iteration_times(fg, rows, cols):
    """Every traced iteration has its own end: none before the one before it,
    the first well before the last, and together the run."""
    off, col = synth.grid_csr(rows, cols)
    g = fg.Graph(off, col, weights=synth.weights(off, col))
    announce(f"sssp iteration times {rows}x{cols}")
    st = fg.sssp(g, 0)[2]
    k = min(st.iterations, 64)
    us = st.iteration_us()
    assert len(us) == k > 20 and all(u >= 0 for u in us)
    assert sum(u > 0 for u in us) > k // 2 and max(us) < sum(us) / 2
    g.close()


@pytest.mark.parametrize("kw", [dict(), dict(team_blocks=-1), dict(team_blocks=8), dict(big_degree=2)])
@pytest.mark.parametrize("deg,last,over", [(1, 0x7FFFFFFF, False), (1, 0x80000000, True),
                                           (3, 0x7FFFFFFE, False), (3, 0x80000000, True),
                                           (7, 0x80000000, True)])
def test_way_back_past_the_largest_distance(fg, orc, kw, deg, last, over):
    """A vertex whose way back sums to 2^32 - 2 is fine and to more is reported,
    by every path alike, whatever the length of its row: 0 - 1, then 1 - 2 of
    weight `last` and 2's other neighbours 3, 4, ... (past every distance that
    fits where that way back is)."""
    pairs = [(0, 1), (1, 2)] + [(2, 3 + i) for i in range(deg - 1)]
    off, col = synth.from_edge_pairs(3 + deg, pairs)
    rows = np.repeat(np.arange(3 + deg), np.diff(off))
    w = np.ones(len(col), np.uint32)
    w[(rows == 0) | (col == 0)] = 0
    w[((rows == 1) & (col == 2)) | ((rows == 2) & (col == 1))] = last
    g = fg.Graph(off, col, weights=w)
    announce(f"sssp way back deg={deg} last={last:#x} {kw}")
    for delta in (0, 1, 0xFFFFFFFF):
        d, p, st = fg.sssp(g, 0, delta=delta, **kw)
        assert st.status == (fg.FG_EOVERFLOW if over else 0), (delta, st.status)
        d = to_np(d).astype(np.uint32)
        assert d[:3].tolist() == [0, 0, last] and (d[3:2 + deg] == last + 1).all()
    b = fg.MsspBatch(g, 2)
    b.admit(1, 0)
    b.step(100)
    if over:
        with pytest.raises(fg.FGError) as e:
            b.poll()
        assert e.value.status == fg.FG_EOVERFLOW
    else:
        assert b.poll()[0] & 2
    g.close()


@pytest.mark.parametrize("n,deg", [(16000, 100), (60000, 40)])
def test_default_delta_where_rows_are_alike(fg, orc, n, deg):
    """Uniform random graphs take small steps by default: no more relaxations,
    to a few percent (their order is not fixed), than 24 x mean weight / mean degree."""
    off, col = _random_graph(orc, n, n * deg // 2, deg)
    w = synth.weights(off, col)
    g = fg.Graph(off, col, weights=w)
    announce(f"sssp default delta n={n} deg={deg}")
    step = round(24 * float(w.mean()) * n / len(col))
    least = min(check(fg, orc, g, off, col, w, 0, delta=step).edges_inspected for _ in range(3))
    st = check(fg, orc, g, off, col, w, 0)
    coarse = check(fg, orc, g, off, col, w, 0, delta=256 * step // 24)
    assert st.edges_inspected <= 1.05 * least < coarse.edges_inspected
    g.close()


def _random_graph(orc, n, edges, seed):
    eu, ev = np.random.default_rng(seed).integers(0, n, (2, edges)).astype(np.int32)
    return orc.csr_from_edges(n, eu, ev)


def _tree(orc, n, children):
    return orc.csr_from_edges(n, np.arange(1, n, dtype=np.int32),
                              (np.arange(n - 1) // children).astype(np.int32))


@pytest.mark.parametrize("kind,n,arg,blocks", [
    ("random", 4000, 12000, 4), ("random", 9000, 27000, 8), ("random", 16000, 60000, 256),
    ("tree", 16000, 200, 8), ("tree", 250000, 200, 256), ("tree", 60000, 3, None),
    ("random", 60000, 60000, 256)])
def test_wide_fronts_of_low_degree_graphs(fg, orc, kind, n, arg, blocks):
    """Fronts of a large part of the graph: queues of vertices alone, even
    shares, leaves that are not queued at all; not slower than the whole grid
    from the start."""
    off, col = _random_graph(orc, n, arg, n) if kind == "random" else _tree(orc, n, arg)
    w = synth.weights(off, col)
    g = fg.Graph(off, col, weights=w)
    srcs = [int(s) for s in synth.sources(off, 3, seed=n)] + [0]
    for s in srcs:
        st = check(fg, orc, g, off, col, w, s)
        assert blocks is None or st.grid_blocks == blocks
    dist, parent = (torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(2))
    us = []
    for opts in (fg.sssp_opts(), fg.sssp_opts(team_blocks=32)):
        fg.sssp_into(g, srcs[0], dist, parent, opts)
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(10):
            fg.sssp_into(g, srcs[0], dist, parent, opts)
        b.record()
        torch.cuda.synchronize()
        us.append(a.elapsed_time(b) * 100)
    assert us[0] < 1.5 * us[1], us
    g.close()


@pytest.mark.parametrize("deg", [1, 4, 5, 40, 256])
@pytest.mark.parametrize("wmax", [0, 1, 64])
def test_queues_of_vertices_alone(fg, orc, deg, wmax):
    """A front past the entries that carry their rows (512 per member) and past
    those that do not, zero weights (equal distances still lower a predecessor)
    and directed rows."""
    hubs = 900
    n = hubs * deg + hubs + 1
    kids = np.arange(1 + hubs, n, dtype=np.int32)
    ring = np.arange(1, 1 + hubs, dtype=np.int32)
    eu = np.concatenate([ring[:-1], 1 + (kids - 1 - hubs) // deg, kids[:-1][kids[:-1] % 3 == 0]])
    ev = np.concatenate([ring[1:], kids, kids[:-1][kids[:-1] % 3 == 0] + 1])
    # the hubs hang on a tree of four children each, so they are met together
    eu = np.concatenate([eu, ring]).astype(np.int32)
    ev = np.concatenate([ev, (ring - 1) // 4]).astype(np.int32)
    off, col = orc.csr_from_edges(n, eu, ev)
    w = synth.weights(off, col) % np.uint32(wmax + 1)
    for sym in (True, False):
        g = fg.Graph(off, col, weights=w, symmetric=sym)
        for delta in (0, 3, 0xFFFFFFFF):
            for s in (0, 450, n - 1):
                check(fg, orc, g, off, col, w, s, delta=delta)
        g.close()
