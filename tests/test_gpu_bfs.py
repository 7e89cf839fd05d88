"""Parity of the HIP BFS path with the serial oracle.

Depths are compared bit-exactly; parents are validated as a BFS tree (they
may legally differ); the per-iteration frontier sizes must equal the
oracle's level histogram; in direction-optimizing mode the direction trace
must equal the oracle's prediction from the level histogram (Sec. VI-A) and
the CSR entries read per iteration must equal the oracle's count for the
early-exit pull (which pins the early exit itself).
"""
import numpy as np
import pytest
import torch

import synth
from gpu_util import announce, gpu, need_gpu, to_np

pytestmark = gpu

MODES = {"do": 0, "push": 1, "unfused": 2}


@pytest.fixture(scope="module")
def fg():
    need_gpu()
    import paper_1504_04804_amd as fg
    fg.lib()
    return fg


def check_bfs(fg, orc, g, off, col, src, mode, do_a=(1, 100), do_b=(1, 10), **kw):
    announce(f"bfs n={len(off)-1} m={len(col)} src={src} mode={mode} {kw}")
    depth, parent, st = fg.bfs(g, src, mode=MODES[mode], do_a=do_a, do_b=do_b, **kw)
    d = to_np(depth)
    p = to_np(parent)
    want, _, cnt, mc = orc.bfs(off, col, src)
    assert st.status == 0
    assert np.array_equal(d, want), f"depth mismatch at {np.flatnonzero(d != want)[:10]}"
    err = orc.check_bfs(off, col, src, d, p)
    assert err is None, err
    L = len(cnt)
    assert st.iterations == L
    assert st.reached == cnt.sum()
    dirs, front, insp = st.trace()
    k = min(L, fg.FG_TRACE_MAX)
    assert front == cnt[:k].tolist()
    if mode == "do":
        want_dirs = orc.do_schedule(cnt, len(off) - 1, len(col), do_a, do_b)
        assert dirs == want_dirs[:k].tolist()
    else:
        want_dirs = np.zeros(L, np.int8)
        assert dirs == [0] * k
    want_insp = orc.edges_inspected(off, col, want, want_dirs)
    assert insp == want_insp[:k].tolist()
    if L <= fg.FG_TRACE_MAX:
        assert st.edges_inspected == want_insp.sum()
    return st


@pytest.fixture(scope="module")
def rmat12(fg):
    off, col = synth.rmat_csr(12)
    return off, col, fg.Graph(off, col)


@pytest.mark.parametrize("mode", ["do", "push", "unfused"])
def test_rmat12_from_vertex0(fg, orc, rmat12, mode):
    off, col, g = rmat12
    check_bfs(fg, orc, g, off, col, 0, mode)


@pytest.mark.parametrize("mode", ["do", "push"])
def test_rmat12_random_sources(fg, orc, rmat12, mode):
    off, col, g = rmat12
    for s in synth.sources(off, 6, seed=77):
        check_bfs(fg, orc, g, off, col, int(s), mode)


def test_rmat12_forced_paths(fg, orc, rmat12):
    """Full-grid iterations only, tiny big-degree cut (phase B on), and an
    always-pull / never-pull schedule: results must not change."""
    off, col, g = rmat12
    for s in (0, 5, 100):
        check_bfs(fg, orc, g, off, col, s, "do", small_frontier=1, small_edges=1)
        check_bfs(fg, orc, g, off, col, s, "push", small_frontier=1, small_edges=1, big_degree=2)
        check_bfs(fg, orc, g, off, col, s, "do", do_a=(0, 1), do_b=(0, 1))
        check_bfs(fg, orc, g, off, col, s, "do", do_a=(0, 1), do_b=(10**6, 1))
        check_bfs(fg, orc, g, off, col, s, "do", do_a=(10**6, 1))


def test_closed_form_graphs(fg, orc):
    # path, grid, star, isolated source, disconnected union, single vertex
    cases = []
    n = 300
    cases.append(("path", synth.from_edge_pairs(n, [(i, i + 1) for i in range(n - 1)]), [0, 150, 299]))
    cases.append(("grid", synth.grid_csr(33, 47), [0, 16 * 47 + 23, 33 * 47 - 1]))
    cases.append(("star", synth.from_edge_pairs(2000, [(0, i) for i in range(1, 2000)]), [0, 7]))
    cases.append(("iso", synth.from_edge_pairs(10, [(0, 1), (1, 2)]), [9, 0]))
    cases.append(("two", synth.from_edge_pairs(8, [(0, 1), (1, 2), (4, 5), (5, 6), (6, 7)]), [6, 1]))
    cases.append(("single", (np.zeros(2, np.int32), np.zeros(0, np.int32)), [0]))
    for name, (off, col), srcs in cases:
        g = fg.Graph(off, col)
        for s in srcs:
            for mode in ("do", "push"):
                check_bfs(fg, orc, g, off, col, s, mode)


@pytest.mark.parametrize("scale", [14, 16])
def test_rmat_medium(fg, orc, scale):
    off, col = synth.rmat_csr(scale)
    g = fg.Graph(off, col)
    for s in synth.sources(off, 3, seed=scale):
        for mode in ("do", "push"):
            check_bfs(fg, orc, g, off, col, int(s), mode)
    check_bfs(fg, orc, g, off, col, 0, "do", big_degree=64, small_frontier=1)


def test_grid_high_diameter(fg, orc):
    off, col = synth.grid_csr(256, 256)
    g = fg.Graph(off, col)
    for s in (0, 128 * 256 + 128):
        check_bfs(fg, orc, g, off, col, s, "push")
    check_bfs(fg, orc, g, off, col, 0, "push", small_frontier=1, small_edges=1)
    # full-grid levels only, every vertex cut into descriptors (phase B on
    # every level), the same workspace reused across the runs
    for src in (0, 255, 128 * 256 + 128):
        check_bfs(fg, orc, g, off, col, src, "push", small_frontier=1, small_edges=1,
                  team_blocks=-1, big_degree=2)
    # team levels whose shares drift apart (the frontier grows at its ends)
    check_bfs(fg, orc, g, off, col, 0, "push", small_edges=1, team_blocks=8)
    check_bfs(fg, orc, g, off, col, 128 * 256 + 128, "push", small_edges=1, team_blocks=64)


def test_lds_queue_modes(fg, orc, rmat12):
    """Levels run by one workgroup or a team from LDS queues: team widths
    from 2 to the whole grid, and a hub whose 3000 neighbours exceed one
    workgroup's LDS queue, so the overflow goes to the global queue."""
    n = 6001
    edges = [(0, i) for i in range(1, 3001)] + [(i, i + 3000) for i in range(1, 3001)]
    off, col = synth.from_edge_pairs(n, edges)
    g = fg.Graph(off, col)
    for mode in ("do", "push"):
        check_bfs(fg, orc, g, off, col, 0, mode)
        check_bfs(fg, orc, g, off, col, 0, mode, small_edges=1, team_blocks=2)
        check_bfs(fg, orc, g, off, col, 0, mode, small_edges=1, team_blocks=7, team_edges=1 << 20)
        check_bfs(fg, orc, g, off, col, 4000, mode, small_frontier=1, team_blocks=3)
    # 100 vertices of degree 51 (mean degree low enough for LDS levels)
    # discover 5000 leaves: more than one workgroup's LDS queue holds
    edges = [(0, i) for i in range(1, 101)]
    edges += [(i, 101 + 50 * (i - 1) + j) for i in range(1, 101) for j in range(50)]
    off, col = synth.from_edge_pairs(5101, edges)
    g = fg.Graph(off, col)
    for mode in ("do", "push"):
        check_bfs(fg, orc, g, off, col, 0, mode, small_edges=1 << 18)
        check_bfs(fg, orc, g, off, col, 0, mode, small_edges=1, team_blocks=2)
        check_bfs(fg, orc, g, off, col, 0, mode, small_edges=1, team_blocks=3, team_edges=1 << 18)
    off, col, g = rmat12
    for team in (-1, 2, 5, 64, 10**6):
        for s in (0, 5):
            check_bfs(fg, orc, g, off, col, s, "push", team_blocks=team)
            check_bfs(fg, orc, g, off, col, s, "push", team_blocks=team, small_edges=1,
                      team_edges=1 << 30)
            check_bfs(fg, orc, g, off, col, s, "do", team_blocks=team, small_edges=1,
                      team_edges=1 << 30)


def test_repeat_determinism(fg, orc, rmat12):
    """Atomic races must not change depths: 50 repeats, identical depths."""
    off, col, g = rmat12
    want = orc.bfs(off, col, 3)[0]
    for _ in range(50):
        d, p, st = fg.bfs(g, 3, mode=0)
        assert np.array_equal(to_np(d), want)


@pytest.mark.slow
def test_config_rmat22_dobfs_sampled(fg, orc):
    """Full-size RMAT scale 22 DOBFS in the benchmark's launch configuration."""
    off, col = synth.rmat_csr(22)
    g = fg.Graph(off, col)
    for s in synth.sources(off, 64)[:4]:
        check_bfs(fg, orc, g, off, col, int(s), "do")


@pytest.mark.slow
def test_config_grid4096_push(fg, orc):
    off, col = synth.grid_csr(4096, 4096)
    g = fg.Graph(off, col)
    announce("grid 4096x4096 push from 0")
    depth, parent, st = fg.bfs(g, 0, mode=1)
    d = to_np(depth)
    r = np.arange(4096, dtype=np.int32)
    assert np.array_equal(d.reshape(4096, 4096), r[:, None] + r[None, :])
    assert st.iterations == 8191
    assert orc.check_bfs(off, col, 0, d, to_np(parent)) is None


def test_workspace_alignment_checked(fg, orc):
    """A workspace whose start is not 256-byte aligned is refused with
    FG_EINVAL before anything runs (every primitive carves its workspace
    into 256-byte aligned pieces); the aligned one still works."""
    off, col = synth.rmat_csr(8)
    g = fg.Graph(off, col)
    need = g.workspace_bytes(fg.FG_PRIM_BFS)
    big = torch.zeros(need + 512, dtype=torch.uint8, device="cuda")
    depth = torch.empty(g.n, dtype=torch.int32, device="cuda")
    for shift in (16, 128):
        with pytest.raises(fg.FGError) as e:
            fg.bfs_into(g, 0, depth, None, fg.bfs_opts(), ws=big[shift:shift + need])
        assert e.value.status == fg.FG_EINVAL
        srcs = torch.zeros(2, dtype=torch.int32, device="cuda")
        with pytest.raises(fg.FGError) as e:
            fg.bfs_many_into(g, srcs, depth, None, fg.bfs_opts(), ws=big[shift:shift + need])
        assert e.value.status == fg.FG_EINVAL
        with pytest.raises(fg.FGError) as e:
            fg.cc_into(g, torch.empty(g.n, dtype=torch.int32, device="cuda"),
                       ws=big[shift:shift + 64])
        assert e.value.status == fg.FG_EINVAL
    fg.bfs_into(g, 0, depth, None, fg.bfs_opts(), ws=big[256:256 + need])
    assert np.array_equal(to_np(depth), orc.bfs(off, col, 0)[0])
    g.close()


def _hubs(orc, n, edges, degs, seed):
    """Random graph of n vertices with rows of about the given lengths."""
    rng = np.random.default_rng(seed)
    u = [rng.integers(0, n, edges).astype(np.int32)]
    v = [rng.integers(0, n, edges).astype(np.int32)]
    for i, d in enumerate(degs):
        hub = (i * 37 + 5) % n
        to = rng.permutation(n)[:d].astype(np.int32)
        u.append(np.full(len(to), hub, np.int32))
        v.append(to)
    return orc.csr_from_edges(n, np.concatenate(u), np.concatenate(v))


# one workgroup up to 32768 vertices (direction-optimizing) and up to 20480
# vertices and 2^18 entries (push, and a direction rule above 1); both sides
# of each bound, rows at and past the length that all waves share (256), rows
# that a pull reads past its 4th and 16th entry
@pytest.mark.parametrize("n,edges,degs", [
    (1, 0, []), (2, 1, []), (33, 20, []), (64, 300, []), (1025, 900, [255, 256, 257, 1000]),
    (5000, 40000, [4999, 3000, 700]), (20480, 30000, [300]), (20481, 30000, [300]),
    (16384, 127000, []), (16384, 135000, []), (32767, 40000, [20000]), (32768, 400000, [32767]),
    (32769, 40000, []), (9000, 4000, [9, 17, 64, 80, 81] * 20)])
def test_one_workgroup(fg, orc, n, edges, degs):
    off, col = _hubs(orc, n, edges, degs, seed=n + edges)
    g = fg.Graph(off, col)
    m = len(col)
    for src in sorted({0, 5 % n, n - 1}):
        st = check_bfs(fg, orc, g, off, col, src, "do")
        assert (st.grid_blocks == 1) == (n <= 32768 and m <= 1 << 21)
        st = check_bfs(fg, orc, g, off, col, src, "push")
        assert (st.grid_blocks == 1) == (n <= 20480 and m <= 1 << 18)
        st = check_bfs(fg, orc, g, off, col, src, "do", do_a=(1000, 1), do_b=(1, 10))
        assert (st.grid_blocks == 1) == (n <= 32768 and m <= 1 << 18)
        # pulls and pushes in turn
        check_bfs(fg, orc, g, off, col, src, "do", do_a=(1, 100000), do_b=(10, 1))
        st = check_bfs(fg, orc, g, off, col, src, "do", team_blocks=2)
        assert st.grid_blocks > 1
    depth, parent, st = fg.bfs(g, 0, mode=MODES["push"], parents=False)
    assert parent is None and np.array_equal(to_np(depth), orc.bfs(off, col, 0)[0])
    depth, parent, st = fg.bfs(g, 0, parents=False)
    assert parent is None and np.array_equal(to_np(depth), orc.bfs(off, col, 0)[0])
    g.close()


def test_one_workgroup_long_diameter(fg, orc):
    """More levels than the record traces, on both kinds of visited set."""
    for rows, cols in ((1, 20480), (3, 6000), (2, 16384)):
        off, col = synth.grid_csr(rows, cols)
        g = fg.Graph(off, col)
        for mode in ("do", "push"):
            st = check_bfs(fg, orc, g, off, col, cols // 3, mode)
            assert (st.grid_blocks == 1) == (mode == "do" or g.n <= 20480)
            if mode == "push":
                assert st.edges_inspected == len(col)
        g.close()


# the pull's two ways through a wave's words (a lane per bit, candidates laid
# over the lanes) on one workgroup, whose waves find too many to list, on a few
# and on all; pulls and pushes in turn, so that a listed frontier, an unlisted
# one and an empty one are each taken over by a push
@pytest.mark.parametrize("n,edges,degs", [
    (64, 200, [50]), (4097, 9000, [900, 30, 18]), (40001, 60000, [20000]),
    (40000, 15000, [39999]), (131072, 1300000, [300, 200]), (262143, 250000, [100000, 64])])
@pytest.mark.parametrize("blocks", [1, 7, 0])
def test_pull_words(fg, orc, n, edges, degs, blocks):
    off, col = _hubs(orc, n, edges, degs, seed=n + 1)
    g = fg.Graph(off, col)
    kw = dict(grid_blocks=blocks) if blocks else dict(team_blocks=2)
    for src in sorted({0, 5 % n, 42 % n, n - 1}):
        for do_b in ((1, 10), (1, 1), (1000, 1)):
            check_bfs(fg, orc, g, off, col, src, "do", do_a=(1, 100000), do_b=do_b, **kw)
    g.close()


# pushes of short frontiers of long rows, whose chunks every workgroup lists
# itself: up to 1024 vertices of mean degree big_degree (any degree up to 64
# vertices), and the descriptors just past each bound; consecutive levels take
# turns between the two, so each finds the other's counters
@pytest.mark.parametrize("width,deg", [(64, 3), (65, 63), (65, 64), (900, 70), (1023, 300),
                                       (1024, 64), (1025, 64), (1025, 300), (5000, 66)])
@pytest.mark.parametrize("blocks", [1, 7, 0])
def test_push_chunks(fg, orc, width, deg, blocks):
    # source -> `width` vertices, each with deg - 1 neighbours of its own range
    # of 6000, then chains behind those back to one vertex
    n = 1 + width + 6000 + 500
    rng = np.random.default_rng(width * deg)
    a = np.arange(1, 1 + width)
    u = [np.zeros(width, np.int64), np.repeat(a, deg - 1)]
    v = [a, 1 + width + rng.integers(0, 6000, width * (deg - 1))]
    u.append(1 + width + rng.integers(0, 6000, 500))
    v.append(1 + width + 6000 + np.arange(500))
    off, col = orc.csr_from_edges(n, np.concatenate(u).astype(np.int32),
                                  np.concatenate(v).astype(np.int32))
    g = fg.Graph(off, col)
    kw = dict(grid_blocks=blocks) if blocks else dict(blocks_per_cu=1)
    for src in (0, n - 1, 1 + width):
        check_bfs(fg, orc, g, off, col, src, "push", team_blocks=-1, small_edges=1, **kw)
        check_bfs(fg, orc, g, off, col, src, "do", big_degree=33, **kw)
    g.close()


@pytest.mark.parametrize("n,m,bfs,sssp", [(16384, 200000, 1, 64), (16385, 200000, 1, 128),
                                          (131072, 900000, 64, 128), (131073, 900000, 64, None),
                                          (524288, 1500000, 64, None), (524289, 1500000, 128, None)])
def test_default_width(fg, orc, n, m, bfs, sssp):
    """The launch is as wide as the size asks for unless an option says
    otherwise (mean degree above 8 for the shortest paths)."""
    off, col = _hubs(orc, n, m, [700, 40], seed=n)
    g = fg.Graph(off, col, synth.weights(off, col))
    full = fg.bfs(g, 5, do_a=(1001, 1000))[2].grid_blocks
    st = check_bfs(fg, orc, g, off, col, 5, "do")
    assert st.grid_blocks == min(bfs, full) if bfs > 1 else st.grid_blocks == 1
    assert check_bfs(fg, orc, g, off, col, 5, "do", grid_blocks=200).grid_blocks == 200
    assert fg.sssp(g, 5)[2].grid_blocks == (sssp or full)
    g.close()


@pytest.mark.parametrize("deg", [65, 1022, 1023, 1024, 1025, 2500])
def test_one_hub_levels(fg, orc, deg):
    """A frontier of one long row: up to 1024 entries workgroup 0 takes it
    alone, whatever the mean degree, past that the whole grid does."""
    n = 40000
    u = np.concatenate([np.zeros(1), np.full(deg, 1), np.full(deg, n - 1), np.arange(2, 30000)])
    v = np.concatenate([np.ones(1), 2 + 3 * np.arange(deg), 5 + 7 * np.arange(deg),
                        np.arange(3, 30001)])
    off, col = orc.csr_from_edges(n, u.astype(np.int32), v.astype(np.int32))
    g = fg.Graph(off, col)
    for src in (0, 1, n - 1):
        for mode in ("do", "push"):
            check_bfs(fg, orc, g, off, col, src, mode)
        check_bfs(fg, orc, g, off, col, src, "do", do_a=(1, 100000), small_edges=deg - 1)
    g.close()


def test_default_width_by_entries(fg, orc):
    """Where rows are alike the launch is as wide as the entries ask for;
    where most are in hubs' rows (R-MAT) BFS goes by the vertices alone."""
    rng = np.random.default_rng(8)
    for n, edges, bfs, sssp in ((131072, 1900000, 128, None), (131072, 2400000, None, None),
                                (16000, 1400000, 64, None)):
        off, col = orc.csr_from_edges(n, *rng.integers(0, n, (2, edges)).astype(np.int32))
        g = fg.Graph(off, col, synth.weights(off, col))
        full = fg.bfs(g, 5, do_a=(1001, 1000))[2].grid_blocks
        assert check_bfs(fg, orc, g, off, col, 5, "do", team_blocks=2).grid_blocks == (bfs or full)
        assert fg.sssp(g, 5)[2].grid_blocks == (sssp or full)
        g.close()
    off, col = synth.rmat_csr(17)
    assert len(col) > 3 << 20
    g = fg.Graph(off, col, synth.weights(off, col))
    src = int(synth.sources(off, 1)[0])
    assert check_bfs(fg, orc, g, off, col, src, "do").grid_blocks == 64
    assert fg.sssp(g, src)[2].grid_blocks == 128
    g.close()


@pytest.mark.parametrize("n,edges,solo", [(20480, 215000, True), (20480, 225000, False),
                                          (32768, 655360, False), (8192, 800000, False)])
def test_one_workgroup_where_rows_are_alike(fg, orc, n, edges, solo):
    """On uniform random graphs a pull reads a large part of the entries, so
    one workgroup takes fewer of them than where hubs end it early."""
    rng = np.random.default_rng(n + edges)
    off, col = orc.csr_from_edges(n, *rng.integers(0, n, (2, edges)).astype(np.int32))
    assert (len(col) + 4 * n <= 1 << 19) == solo
    g = fg.Graph(off, col)
    for src in (0, n - 1):
        assert (check_bfs(fg, orc, g, off, col, src, "do").grid_blocks == 1) == solo
    g.close()


@pytest.mark.parametrize("k", [5, 6, 13, 14, 37, 38, 101, 102, 149, 300])
def test_one_workgroup_beside_dense_components(fg, orc, k):
    """Rows that a pull reads to their end (cliques that the source does not
    reach) and rows with their first reached entry anywhere, at the borders of
    the steps that read them: 4, then 8 up to 36, then 64 entries at a time."""
    i, j = np.triu_indices(k, 1)
    n0, nc = 2000, 1 if k == 300 else 6
    rng = np.random.default_rng(k)
    # the source's component: long rows whose reached entries are few and last
    u = [rng.integers(0, n0, 4 * n0), np.arange(40).repeat(k)]
    v = [rng.integers(0, n0, 4 * n0), n0 - 1 - rng.integers(0, n0 // 2, 40 * k)]
    for c in range(nc):
        u.append(n0 + c * k + i)
        v.append(n0 + c * k + j)
    n = n0 + nc * k
    off, col = orc.csr_from_edges(n, np.concatenate(u).astype(np.int32),
                                  np.concatenate(v).astype(np.int32))
    g = fg.Graph(off, col)
    for src in (n0 - 1, n0 // 2, 0):
        for da in ((1, 100), (1, 100000)):
            st = check_bfs(fg, orc, g, off, col, src, "do", do_a=da, do_b=(1, 1000))
            assert st.grid_blocks == 1
    g.close()
