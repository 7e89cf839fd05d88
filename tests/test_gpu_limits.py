"""Rows at the end of the largest column array a graph may have (2^31 - 1
entries): a place formed past such a row's end does not fit int32.  Depths,
distances, ranks and entry counts by closed form, through the C ABI."""
import numpy as np
import pytest
import torch

from gpu_util import announce, gpu, need_gpu, to_np

pytestmark = gpu

N, M = 4096, (1 << 31) - 1
BULK = 1024  # 256 vertices from here on hold most entries
FIRST = 100  # the last row's neighbours are FIRST, FIRST + 1, ...


@pytest.fixture(scope="module")
def env():
    need_gpu()
    if torch.cuda.get_device_properties(0).total_memory < 100 << 30:
        pytest.skip("needs 100 GB of device memory")
    import paper_1504_04804_amd as fg
    fg.lib()
    col = torch.full((M,), 5, dtype=torch.int32, device="cuda")
    w = torch.ones(M, dtype=torch.int32, device="cuda")
    yield fg, col, w
    del col, w
    torch.cuda.empty_cache()


@pytest.mark.parametrize("hit", [False, True])
@pytest.mark.parametrize("L", [1, 2, 3, 30, 62, 130, 300, 700])
def test_rows_that_end_at_the_largest_entry(env, L, hit):
    """Vertex 5 has one entry, to 6; the last vertex has L, none of them 5
    unless `hit`, then the last; 256 vertices hold all others, every one 5."""
    fg, col, w = env
    last = N - 1
    many = M - L - 1
    off = np.full(N + 1, many + 1, np.int64)
    off[:6] = 0
    off[6:BULK] = 1
    off[BULK:BULK + 257] = 1 + many * np.arange(257) // 256
    off[N] = M
    col.fill_(5)
    col[0] = 6
    col[M - L:] = torch.arange(FIRST, FIRST + L, dtype=torch.int32, device="cuda")
    if hit:
        col[M - 1] = 5
    row = list(range(FIRST, FIRST + L - 1)) + [5 if hit else FIRST + L - 1]
    announce(f"largest entry: last row of {L}, hit {hit}")
    g = fg.Graph(torch.from_numpy(off.astype(np.int32)), col, w, validate=False)
    bulk = list(range(BULK, BULK + 256))

    # pushes out of the last row
    want = np.full(N, -1, np.int32)
    want[last] = 0
    want[row] = 1
    if hit:
        want[6] = 2
    modes = [dict(mode=fg.FG_MODE_PUSH), dict(mode=fg.FG_MODE_PUSH, team_blocks=-1, small_edges=1),
             dict(mode=fg.FG_MODE_PUSH, team_blocks=-1, small_edges=1, big_degree=2)]
    for kw in modes:
        d, _, st = fg.bfs(g, last, **kw)
        assert st.status == 0 and np.array_equal(to_np(d), want), kw
    announce("... msbfs")
    b = fg.MsBatch(g, 3, fg.msbfs_opts(pull_div=1))  # pushes throughout
    for lane in range(3):
        b.admit(lane, last)
    b.step(10)
    assert b.poll()[0] == 7
    assert all(np.array_equal(to_np(b.read(lane)), want) for lane in range(3))
    b.close()
    announce("... mssp, sssp")
    uw = want.astype(np.int64) % (1 << 32)
    for opts in (fg.mssp_opts(delta=100), fg.mssp_opts(delta=100, dense_lanes=1),
                 fg.mssp_opts(delta=100, dense_lanes=1, big_degree=4096)):
        b = fg.MsspBatch(g, 8, opts)
        for lane in range(8):
            b.admit(lane, last)
        b.step(20)
        assert b.poll()[0] == 255
        assert all(np.array_equal(to_np(b.read(lane)).astype(np.uint32), uw) for lane in (0, 7))
        b.close()
    for kw in (dict(), dict(big_degree=2, team_blocks=-1, small_edges=1)):
        d, _, st = fg.sssp(g, last, **kw)
        assert st.status == 0 and np.array_equal(to_np(d).astype(np.uint32), uw)

    announce("... bfs and msbfs pulls")
    # pulls into it: from 5 (one entry, to 6), then every vertex looks for 5 or 6
    want = np.full(N, -1, np.int32)
    want[5], want[6], want[bulk] = 0, 1, 2
    if hit:
        want[last] = 2
    d, _, st = fg.bfs(g, 5, do_a=(1, 1000000), do_b=(1, 1000000))
    at = [5, 6, last] + bulk
    assert st.trace()[0][:2] == [0, 1] and np.array_equal(to_np(d)[at], want[at])
    assert st.trace()[2][1] == 256 + L  # the bulk stops at its first entries
    b = fg.MsBatch(g, 2, fg.msbfs_opts(pull_div=1 << 30, push_div=1 << 30))
    b.admit(1, 5)
    b.step(10)
    assert b.poll()[0] & 2
    got = to_np(b.read(1))
    assert got[5] == 0 and got[last] == (1 if hit else -1)  # pulls from the start
    b.close()
    announce("... pull step")
    seen = torch.zeros(N // 64, dtype=torch.int64, device="cuda")
    seen[0] = 1 << 5
    vis = seen.clone()
    vis[BULK // 64:BULK // 64 + 4] = -1
    nxt, dep, par = torch.zeros_like(seen), *torch.zeros((2, N), dtype=torch.int32, device="cuda")
    q, ln = torch.zeros(N, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32,
                                                                          device="cuda")
    read = torch.zeros(1, dtype=torch.int64, device="cuda")
    fg.pull_step(g, seen, vis, nxt, 0, dep, par, q, ln, read)
    assert int(ln) == hit and int(read) == L
    if hit:
        assert int(q[0]) == last and int(dep[last]) == 1 and int(par[last]) == 5

    announce("... pagerank")
    # ranks: direct (one iteration) and planned
    deg = np.diff(off).astype(np.float64)
    rank = np.full(N, 1.0 / N)
    for it in range(1, 5):
        c = np.divide(rank, deg, out=np.zeros(N), where=deg > 0)
        rank = np.full(N, 0.15 / N)
        rank[bulk] += 0.85 * deg[bulk] * c[5]
        rank[5] += 0.85 * c[6]
        rank[last] += 0.85 * c[row].sum()
        if it in (1, 4):
            r = torch.empty(N, dtype=torch.float64, device="cuda")
            fg.pagerank_into(g, r, 0.85, 0.0, it)
            # a sum of 2^23 equal terms, in any order: 2^23 roundings of 2^-53
            assert np.allclose(to_np(r), rank, rtol=2.0 ** -29, atol=0)
    g.close()
