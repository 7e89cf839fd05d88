"""Parity of the 64-lane batched BFS: every lane's depths equal the oracle's
BFS from that lane's source (and fg_bfs's), alone or in the mix, including
lanes admitted mid-flight and lanes reused after release."""
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


def check_lanes(fg, orc, b, off, col, srcs):
    for lane, s in srcs.items():
        got = to_np(b.read(lane))
        want = orc.bfs(off, col, int(s))[0]
        assert np.array_equal(got, want), f"lane {lane} src {s}: {np.flatnonzero(got != want)[:8]}"


@pytest.mark.parametrize("opts", [dict(), dict(pull_div=1), dict(pull_div=1 << 30, push_div=1 << 30),
                                  dict(big_degree=4)])
def test_rmat12_64_lanes(fg, orc, opts):
    off, col = synth.rmat_csr(12)
    g = fg.Graph(off, col)
    srcs = {i: int(s) for i, s in enumerate(synth.sources(off, 64, seed=11))}
    announce(f"msbfs rmat12 64 lanes {opts}")
    b = fg.MsBatch(g, 64, fg.msbfs_opts(**opts))
    for lane, s in srcs.items():
        b.admit(lane, s)
    b.run(k_iters=4)
    check_lanes(fg, orc, b, off, col, srcs)


def test_few_lanes_duplicates_isolated(fg, orc):
    off, col = synth.from_edge_pairs(300, [(i, i + 1) for i in range(250)] + [(0, 260)])
    g = fg.Graph(off, col)
    srcs = {0: 5, 1: 5, 2: 299, 3: 120, 7: 0}
    b = fg.MsBatch(g, 8)
    for lane, s in srcs.items():
        b.admit(lane, s)
    b.run(k_iters=64)
    check_lanes(fg, orc, b, off, col, srcs)


def test_continuous_admission_and_reuse(fg, orc):
    off, col = synth.rmat_csr(13)
    g = fg.Graph(off, col)
    src = synth.sources(off, 96, seed=5)
    b = fg.MsBatch(g, 64)
    first = {i: int(src[i]) for i in range(32)}
    for lane, s in first.items():
        b.admit(lane, s)
    b.step(2)                       # mid-flight
    second = {32 + i: int(src[32 + i]) for i in range(32)}
    for lane, s in second.items():
        b.admit(lane, s)
    b.run(k_iters=3)
    check_lanes(fg, orc, b, off, col, {**first, **second})
    # reuse lanes 3, 40, 63 for new queries while the others stay done
    again = {3: int(src[64]), 40: int(src[65]), 63: int(src[66])}
    for lane in again:
        b.release(lane)
    for lane, s in again.items():
        b.admit(lane, s)
    b.run(k_iters=5)
    check_lanes(fg, orc, b, off, col, again)
    check_lanes(fg, orc, b, off, col, {5: first[5], 50: second[50]})  # untouched lanes


def test_alone_equals_in_the_mix(fg, orc):
    off, col = synth.rmat_csr(12)
    g = fg.Graph(off, col)
    srcs = [int(s) for s in synth.sources(off, 64, seed=2)]
    b = fg.MsBatch(g, 64)
    for lane, s in enumerate(srcs):
        b.admit(lane, s)
    b.run()
    alone = fg.MsBatch(g, 1)
    for lane in (0, 17, 63):
        single, _, _ = fg.bfs(g, srcs[lane], mode=fg.FG_MODE_DO)
        mix = to_np(b.read(lane))
        alone.admit(0, srcs[lane])
        alone.run()
        assert np.array_equal(mix, to_np(single))
        assert np.array_equal(mix, to_np(alone.read(0)))


def test_grid_64_sources_closed_form(fg):
    R = C = 96
    off, col = synth.grid_csr(R, C)
    g = fg.Graph(off, col)
    rng = np.random.default_rng(4)
    srcs = rng.choice(R * C, 64, replace=False)
    b = fg.MsBatch(g, 64)
    for lane, s in enumerate(srcs):
        b.admit(lane, int(s))
    b.run(k_iters=32)
    rr, cc = np.divmod(np.arange(R * C), C)
    for lane, s in enumerate(srcs):
        r0, c0 = divmod(int(s), C)
        assert np.array_equal(to_np(b.read(lane)), np.abs(rr - r0) + np.abs(cc - c0))


@pytest.mark.parametrize("team,team_e,lanes", [(32, 0, 1), (32, 0, 8), (2, 0, 5), (7, 0, 64),
                                               (64, 0, 3), (32, 300, 8), (-1, 0, 8), (0, 0, 4),
                                               (1, 0, 2)])
def test_team_levels(fg, orc, team, team_e, lanes):
    # grid levels run as a team; k_iters=3 ends episodes in mid-flight and
    # the next step resumes them; lanes are admitted between steps
    R, C = 150, 170
    off, col = synth.grid_csr(R, C)
    g = fg.Graph(off, col)
    rng = np.random.default_rng(abs(team) * 100 + lanes)
    srcs = {int(l): int(s) for l, s in zip(rng.choice(64, lanes, replace=False),
                                           rng.choice(R * C, lanes, replace=False))}
    announce(f"msbfs team={team} team_e={team_e} lanes={lanes}")
    b = fg.MsBatch(g, 64, fg.msbfs_opts(team_blocks=team, team_edges=team_e))
    items = list(srcs.items())
    half = len(items) // 2
    for lane, s in items[:half]:
        b.admit(lane, s)
    if half:
        b.step(3)
    for lane, s in items[half:]:
        b.admit(lane, s)
    b.run(k_iters=3)
    check_lanes(fg, orc, b, off, col, srcs)
    # R-MAT with pull off: push levels of every shape, hubs included
    off, col = synth.rmat_csr(13)
    g = fg.Graph(off, col)
    srcs = {i: int(s) for i, s in enumerate(synth.sources(off, lanes, seed=abs(team) + 50))}
    b = fg.MsBatch(g, 64, fg.msbfs_opts(team_blocks=team, team_edges=team_e, pull_div=1))
    for lane, s in srcs.items():
        b.admit(lane, s)
    b.run(k_iters=5)
    check_lanes(fg, orc, b, off, col, srcs)


def test_team_back_to_back_handoffs(fg, orc):
    # One-lane batches on R-MAT with the team requested: a team episode that
    # leaves because the frontier's degree grew is re-entered and handed back
    # at once, so two hand-offs follow each other within microseconds.  Every
    # step must finish (no wait reaching its limit) with the oracle's depths.
    off, col = synth.rmat_csr(16)
    g = fg.Graph(off, col)
    srcs = [int(s) for s in synth.sources(off, 64, seed=99)]
    want = {s: orc.bfs(off, col, s)[0] for s in srcs[:8]}
    announce("msbfs team hand-offs: 150 one-lane batches on rmat16")
    b = fg.MsBatch(g, 64, fg.msbfs_opts(team_blocks=1))
    for r in range(150):
        if r:
            b.release(0)
        s = srcs[r % 8]
        b.admit(0, s)
        b.step(1 << 30)
        done, _ = b.poll()  # raises FGError (FG_EDEVICE) if a wait hit its limit
        assert done & 1
        if r < 8 or r % 16 == 0:
            assert np.array_equal(to_np(b.read(0)), want[s]), f"batch {r} src {s}"


def test_msbfs_argument_errors(fg):
    off, col = synth.from_edge_pairs(4, [(0, 1)])
    g = fg.Graph(off, col)
    b = fg.MsBatch(g, 4)
    for bad in ((4, 0), (-1, 0), (0, 4), (0, -1)):
        with pytest.raises(fg.FGError):
            b.admit(*bad)
    b.admit(1, 0)
    with pytest.raises(fg.FGError):
        b.admit(1, 2)  # already pending


@pytest.mark.slow
def test_config_rmat23_64_sources(fg, orc):
    off, col = synth.rmat_csr(23)
    g = fg.Graph(off, col)
    srcs = [int(s) for s in synth.sources(off, 64, seed=23)]
    b = fg.MsBatch(g, 64)
    for lane, s in enumerate(srcs):
        b.admit(lane, s)
    b.run(k_iters=8)
    check_lanes(fg, orc, b, off, col, {lane: srcs[lane] for lane in (0, 31, 63)})


@pytest.mark.slow
def test_config_grid2048_64_sources(fg):
    R = 2048
    off, col = synth.grid_csr(R, R)
    g = fg.Graph(off, col)
    rng = np.random.default_rng(7)
    srcs = rng.choice(R * R, 64, replace=False)
    b = fg.MsBatch(g, 64)
    for lane, s in enumerate(srcs):
        b.admit(lane, int(s))
    b.run(k_iters=512)
    rr, cc = np.divmod(np.arange(R * R, dtype=np.int64), R)
    for lane in range(0, 64, 9):
        r0, c0 = divmod(int(srcs[lane]), R)
        assert np.array_equal(to_np(b.read(lane)), np.abs(rr - r0) + np.abs(cc - c0))


# pull rows at the edges of their classes: the head's four entries, sixteen
# more (two per lane of eight), up to 64, and the listed ones past that, on one
# workgroup (whose waves' lists of long rows fill up on the way) and on all
@pytest.mark.parametrize("n,deg,blocks", [(9000, 70, 1), (4099, 64, 0), (4099, 65, 3), (3001, 20, 0),
                                          (3001, 21, 0), (3001, 5, 2), (3001, 4, 0), (1, 0, 0),
                                          (70001, 24, 0)])
def test_pull_row_classes(fg, orc, n, deg, blocks):
    # vertex v's neighbours: v +- 1, +- k (mod n), so that most rows have
    # exactly `deg` entries, and one vertex of 300
    off_v = np.arange(n, dtype=np.int64)
    steps = [1 + i * max(1, n // (4 * deg + 4)) for i in range(deg // 2)]
    u = np.concatenate([off_v] * len(steps) + [np.zeros(0, np.int64)])
    v = np.concatenate([(off_v + s) % n for s in steps] + [np.zeros(0, np.int64)])
    if n > 1000:
        u = np.concatenate([u, np.full(300, 17)])
        v = np.concatenate([v, np.arange(300) * (n // 300)])
    off, col = orc.csr_from_edges(n, u.astype(np.int32), v.astype(np.int32))
    g = fg.Graph(off, col)
    rng = np.random.default_rng(deg)
    srcs = {i: int(s) for i, s in enumerate(rng.integers(0, n, 13))}
    announce(f"msbfs pull rows n={n} deg={deg} blocks={blocks}")
    for pull_div in (1, 1 << 20):
        b = fg.MsBatch(g, 13, fg.msbfs_opts(grid_blocks=blocks, pull_div=pull_div,
                                            push_div=1 << 20))
        for rep in range(2):  # the second time over reused lanes
            for lane, s in srcs.items():
                b.admit(lane, s)
            b.run(k_iters=3 + rep)
            check_lanes(fg, orc, b, off, col, srcs)
            srcs = {lane: (s + 1) % n for lane, s in srcs.items()}
        # into a row that is not aligned as the lane's
        out = torch.full((n + 3,), -5, dtype=torch.int32, device="cuda")
        for o in range(4):
            b.read(3, out[o:o + n] if o + n <= n + 3 else out[:n])
            torch.cuda.synchronize()
            o = o if o + n <= n + 3 else 0
            assert np.array_equal(to_np(out[o:o + n]), to_np(b.read(3)))
        b.close()
    g.close()


def test_read_into_pinned_host_memory(fg, orc):
    """A lane's row goes wherever the copy could put it: device memory by a
    kernel, host memory by the runtime; no error is left behind."""
    off, col = synth.rmat_csr(10)
    g = fg.Graph(off, col)
    b = fg.MsBatch(g, 4)
    b.admit(2, 7)
    b.run()
    host = torch.full((g.n,), -9, dtype=torch.int32, pin_memory=True)
    b.read(2, host)
    torch.cuda.synchronize()
    assert np.array_equal(host.numpy(), orc.bfs(off, col, 7)[0])
    check_lanes(fg, orc, b, off, col, {2: 7})
    fg.bfs(g, 3)
    b.close()
    g.close()


def _pull_work(off, col, srcs):
    """Entries read and vertex visits of a batch that only pulls, by the
    counting rule: the first four entries, then up to the early exit, four at a
    time in rows of up to 32, all of a row of up to 64."""
    n = len(off) - 1
    seen, front = [0] * n, [0] * n
    for lane, s in enumerate(srcs):
        seen[s] |= 1 << lane
        front[s] |= 1 << lane
    live = (1 << len(srcs)) - 1
    edges = verts = 0
    while live:
        new = [0] * n
        verts += n
        for v in range(n):
            row = col[off[v]:off[v + 1]]
            want = live & ~seen[v]
            if not want or not len(row):
                continue
            got = 0
            for at in range(0, len(row) if len(row) <= 32 else 4, 4):
                edges += len(row[at:at + 4])
                for u in row[at:at + 4]:
                    got |= front[u] & want
                if got == want:
                    break
            if len(row) > 32 and got != want:
                edges += len(row) - 4
                for u in row[4:]:
                    got |= front[u] & want
            new[v] = got
        live = 0
        for v in range(n):
            seen[v] |= new[v]
            live |= new[v]
        front = new
    return edges, verts


@pytest.mark.parametrize("lanes", [1, 3, 64])
@pytest.mark.parametrize("most", [6, 22, 34, 64])
def test_pull_counts(fg, orc, lanes, most):
    """fg_msbfs_counts of a batch that only pulls, rows of every length up to
    the one that is cut into chunks."""
    n = 700
    rng = np.random.default_rng(most)
    deg = rng.integers(0, most // 2, n)
    u = np.repeat(np.arange(n), deg)
    off, col = orc.csr_from_edges(n, u.astype(np.int32), rng.integers(0, n, len(u)).astype(np.int32))
    assert np.diff(off).max() <= 64
    g = fg.Graph(off, col)
    srcs = [int(s) for s in rng.choice(n, lanes)]
    b = fg.MsBatch(g, lanes, fg.msbfs_opts(pull_div=1 << 30, push_div=1 << 30))
    announce(f"msbfs pull counts lanes={lanes} rows up to {np.diff(off).max()}")
    for lane, s in enumerate(srcs):
        b.admit(lane, s)
    b.run(k_iters=3)
    for lane, s in enumerate(srcs):
        assert np.array_equal(to_np(b.read(lane)), orc.bfs(off, col, s)[0])
    assert b.counts() == _pull_work(off.tolist(), col.tolist(), srcs)
    b.close()
