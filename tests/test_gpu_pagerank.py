"""PageRank (fg_pagerank) against the oracle's double-precision power
iteration (O13), through the C ABI.

Tolerance.  Both sides evaluate the same formula in IEEE double; they
differ only in the order of the additions of a row's sum (the kernel sums
short rows in segments of a wave step, longer rows in strided partial sums
combined as a tree; the oracle in CSR order).  Summing k positive terms in any order is within
gamma_{k-1} = (k-1)u / (1 - (k-1)u) of the exact sum (u = 2^-53), and the
contributions, the update and the division add a few roundings more, so
after K iterations every rank agrees to the relative error
    K * (2 gamma_{D-1} + 8u),   D the largest degree,
which these tests assert elementwise (about 1e-9 for R-MAT 22 after 20
iterations; far tighter on grids).  Iteration counts under the
threshold-ratio stop must be equal.
"""
import numpy as np
import pytest
import torch

import synth
import workloads
from gpu_util import announce, gpu, need_gpu, to_np

pytestmark = gpu

U = 2.0 ** -53


def bound(off, iters):
    D = int(np.diff(off).max()) if len(off) > 1 else 0
    k = max(D - 1, 0)
    gamma = k * U / (1 - k * U)
    return max(iters, 1) * (2 * gamma + 8 * U)


@pytest.fixture(scope="module")
def fg():
    need_gpu()
    import paper_1504_04804_amd as fg
    fg.lib()
    return fg


def check(fg, orc, off, col, what, damping=0.85, tol=0.0, max_iter=20):
    announce(f"pagerank {what} n={len(off) - 1} d={damping} tol={tol} max_iter={max_iter}")
    g = fg.Graph(off, col, symmetric=True, validate=False)
    rank, st = fg.pagerank(g, damping, tol, max_iter)
    got = to_np(rank)
    g.close()
    want, it = orc.pagerank(off, col, damping, tol, max_iter)
    assert st.status == 0
    assert st.iterations == it, (what, st.iterations, it)
    rel = np.abs(got - want) / np.maximum(np.abs(want), 1e-300)
    b = bound(off, it)
    assert rel.max() <= b, (what, float(rel.max()), b)
    return got, st


def test_small_graphs(fg, orc):
    for s in (6, 10, 12, 16):
        off, col = synth.rmat_csr(s)
        check(fg, orc, off, col, f"rmat{s}")
    for r, c in ((1, 2), (9, 13), (100, 70)):
        off, col = synth.grid_csr(r, c)
        check(fg, orc, off, col, f"grid{r}x{c}")


def test_long_rows_and_iterations(fg, orc):
    """R-MAT 18 has rows past the workgroup cut (4096 entries) as well as
    wave-summed and lane-summed rows."""
    off, col = synth.rmat_csr(18)
    assert int(np.diff(off).max()) >= 4096
    for d, it in ((0.85, 1), (0.85, 30), (0.5, 10), (0.0, 3), (1.0, 5)):
        check(fg, orc, off, col, f"rmat18 d={d}", damping=d, max_iter=it)
    check(fg, orc, off, col, "rmat18 no iterations", max_iter=0)


def test_threshold_stop(fg, orc):
    off, col = synth.rmat_csr(14)
    for tol in (1e-2, 1e-4, 1e-6):
        _, st = check(fg, orc, off, col, f"rmat14 tol={tol}", tol=tol, max_iter=200)
        assert 1 <= st.iterations < 200
    off, col = synth.grid_csr(40, 40)
    check(fg, orc, off, col, "grid tol", tol=1e-5, max_iter=500)


def test_regular_graph_uniform_and_trace(fg):
    # every vertex of a cycle keeps 1/n; the trace records the vertices above
    # the threshold (none after the first iteration) and m entries read
    n = 1000
    a = np.arange(n, dtype=np.int32)
    import oracle
    off, col = oracle.oracle().csr_from_edges(n, a, (a + 1) % n)
    g = fg.Graph(off, col)
    rank, st = fg.pagerank(g, 0.85, 1e-12, 50)
    r = to_np(rank)
    assert np.allclose(r, 1.0 / n, rtol=1e-14, atol=0)
    assert st.iterations == 1
    assert st.trace()[1][0] == 0 and st.trace()[2][0] == len(col)
    g.close()


def test_argument_errors(fg):
    off, col = synth.grid_csr(3, 3)
    g = fg.Graph(off, col)
    rank = torch.empty(g.n, dtype=torch.float64, device="cuda")
    for kw, code in ((dict(damping=1.5), fg.FG_EINVAL), (dict(tol=-1.0), fg.FG_EINVAL),
                     (dict(max_iter=-1), fg.FG_EINVAL)):
        with pytest.raises(fg.FGError) as e:
            fg.pagerank_into(g, rank, **kw)
        assert e.value.status == code
    with pytest.raises(fg.FGError) as e:
        fg.pagerank_into(g, rank, ws=torch.zeros(16, dtype=torch.uint8, device="cuda"))
    assert e.value.status == fg.FG_ENOMEM
    g.close()
    gd = fg.Graph(np.array([0, 1, 1], np.int32), np.array([1], np.int32), symmetric=False)
    with pytest.raises(fg.FGError) as e:
        fg.pagerank_into(gd, torch.empty(2, dtype=torch.float64, device="cuda"))
    assert e.value.status == fg.FG_EUNSUPPORTED
    gd.close()


@pytest.mark.slow
def test_workload_rmat22(fg, orc):
    off, col, _ = workloads.graph("rmat22")
    check(fg, orc, off, col, "rmat22", max_iter=20)


@pytest.mark.parametrize("pad", range(8))
def test_planned_form_row_classes(fg, orc, pad):
    """Rows at the lengths where the planned form changes how it sums them (a
    lane, 8, 16, 64 lanes, segments of 2048 entries), numbers at every place
    of the last group of eight, no vertex without edges; the ranks of two
    calls are the same bits."""
    degs = [1, 2, 7, 8, 9, 62, 63, 64, 65, 255, 256, 257, 1023, 1024, 1025, 2047, 2048, 2049,
            4095, 4096, 4097, 6200]
    H, P = len(degs), 7000 + pad
    rng = np.random.default_rng(pad)
    eu = np.concatenate([np.full(d, h) for h, d in enumerate(degs)] + [np.arange(P)])
    ev = np.concatenate([rng.choice(P, size=d, replace=False) + H for d in degs]
                        + [(np.arange(P) + 1) % P])
    eu[-P:] += H
    ev[-P:] += H
    off, col = orc.csr_from_edges(H + P, eu.astype(np.int32), ev.astype(np.int32))
    assert (np.diff(off) > 0).all()
    a, _ = check(fg, orc, off, col, f"row classes pad={pad}", max_iter=2 + pad)
    b, _ = check(fg, orc, off, col, f"row classes pad={pad} again", max_iter=2 + pad)
    assert np.array_equal(a, b)


@pytest.mark.parametrize("n", [2, 64, 4095, 4096, 4097, 8193])
def test_planned_form_numbering_tiles(fg, orc, n):
    # sparse random graphs (many empty rows) at the tile sizes of the numbering
    rng = np.random.default_rng(n)
    eu = rng.integers(0, n, n).astype(np.int32)
    ev = rng.integers(0, n, n).astype(np.int32)
    off, col = orc.csr_from_edges(n, eu, ev)
    check(fg, orc, off, col, f"tiles n={n}", max_iter=6)
    check(fg, orc, off, col, f"tiles n={n} tol", tol=1e-3, max_iter=50)


def test_workspace_without_room_for_the_plan(fg, orc):
    """A workspace of the direct form's size is still taken."""
    off, col = synth.rmat_csr(13)
    n = len(off) - 1
    up = lambda x: (x + 255) // 256 * 256
    ws = torch.zeros(2 * up(8 * n) + up(4 * n) + 256, dtype=torch.uint8, device="cuda")
    g = fg.Graph(off, col)
    assert ws.numel() < g.workspace_bytes(fg.FG_PRIM_PR)
    rank = torch.empty(n, dtype=torch.float64, device="cuda")
    announce("pagerank small workspace")
    fg.pagerank_into(g, rank, 0.85, 0.0, 10, ws=ws)
    want, it = orc.pagerank(off, col, 0.85, 0.0, 10)
    got = to_np(rank)
    assert (np.abs(got - want) / want).max() <= bound(off, it)
    g.close()


@pytest.mark.parametrize("cut", [0, 1])
def test_one_launch_for_runs_that_may_stop(fg, orc, cut):
    """With a tolerance the iterations run in one launch, or, from a workspace
    without its barrier, in one or two launches each: the same ranks, counts
    and trace, repeatedly and from a workspace of any contents."""
    for what, (off, col) in (("rmat13", synth.rmat_csr(13)), ("grid", synth.grid_csr(90, 77)),
                             ("none", (np.zeros(6, np.int32), np.zeros(0, np.int32)))):
        g = fg.Graph(off, col)
        need = g.workspace_bytes(fg.FG_PRIM_PR)
        ws = torch.full((need - cut,), 0x5a, dtype=torch.uint8, device="cuda")
        rank = torch.empty(g.n, dtype=torch.float64, device="cuda")
        for tol, most in ((1e-1, 1000), (1e-5, 200), (1e-5, 3), (1e-300, 70)):
            want, it = orc.pagerank(off, col, 0.85, tol, most)
            for _ in range(2):
                stats = fg.new_stats()
                announce(f"pagerank loop {what} tol={tol} max_iter={most} cut={cut}")
                fg.pagerank_into(g, rank, 0.85, tol, most, ws=ws, stats=stats)
                st = fg.read_stats(stats)
                assert st.status == 0 and st.iterations == it
                assert st.edges_inspected == it * len(col)
                k = min(it, 64)
                front = st.trace()[1]
                assert all(f > 0 for f in front[:k - 1]) and (it == most or front[k - 1] == 0 or it > 64)
                got = to_np(rank)
                assert (np.abs(got - want) / want).max() <= bound(off, it)
        g.close()


def test_iterations_left_after_the_stop_cost_nothing(fg):
    off, col = synth.rmat_csr(14)
    g = fg.Graph(off, col)
    rank = torch.empty(g.n, dtype=torch.float64, device="cuda")
    us = {}
    for most in (20, 2000):
        fg.pagerank_into(g, rank, 0.85, 0.1, most)
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        announce(f"pagerank of at most {most} iterations")
        a.record()
        for _ in range(5):
            fg.pagerank_into(g, rank, 0.85, 0.1, most)
        b.record()
        torch.cuda.synchronize()
        us[most] = a.elapsed_time(b) * 200
    assert us[2000] < 3 * us[20], us  # with a launch or two for each some 30 times
    g.close()


@pytest.mark.parametrize("tol", [0.0, 1e-3])
def test_captured(fg, tol):
    """Replays of a captured call, with other work between them."""
    off, col = synth.rmat_csr(12)
    g = fg.Graph(off, col)
    rank = torch.empty(g.n, dtype=torch.float64, device="cuda")
    g.workspace(fg.FG_PRIM_PR)
    fg.pagerank_into(g, rank, 0.85, tol, 30)
    want = to_np(rank).copy()
    graph = torch.cuda.CUDAGraph()
    announce(f"pagerank captured tol={tol}")
    with torch.cuda.graph(graph):
        fg.pagerank_into(g, rank, 0.85, tol, 30)
    for _ in range(4):
        rank.fill_(-1.0)
        torch.cuda.synchronize()
        graph.replay()
        assert np.array_equal(to_np(rank), want)
        fg.pagerank(g, 0.5, 1e-2, 20)
    g.close()
