"""Connected components (fg_cc, hooking + pointer jumping) against the
oracle's component-minimum labels (O12), bit-exact, through the C ABI:
sparse random graphs with many components, R-MAT (many isolated
vertices), grids, degenerate graphs, and the workload graphs R-MAT 22 and
the 4096 x 4096 grid."""
import numpy as np
import pytest
import torch

import synth
import workloads
from gpu_util import announce, gpu, need_gpu, to_np

pytestmark = gpu


@pytest.fixture(scope="module")
def fg():
    need_gpu()
    import paper_1504_04804_amd as fg
    fg.lib()
    return fg


def er_graph(n, p, seed):
    rng = np.random.default_rng(seed)
    k = int(rng.binomial(n * (n - 1) // 2, p))
    eu = rng.integers(0, n, k).astype(np.int32)
    ev = rng.integers(0, n, k).astype(np.int32)
    return eu, ev


def check(fg, orc, off, col, what):
    announce(f"cc {what} n={len(off) - 1} m={len(col)}")
    g = fg.Graph(off, col, symmetric=True, validate=True)
    for rep in range(2):  # twice on the same graph: no state kept between calls
        label, comps = fg.cc(g)
        want, wc = orc.cc(off, col)
        got = to_np(label)
        assert np.array_equal(got, want), (what, rep, np.flatnonzero(got != want)[:8])
        assert comps == wc
    g.close()


@pytest.mark.parametrize("seed", range(6))
def test_sparse_random_many_components(fg, orc, seed):
    rng = np.random.default_rng(seed)
    n = int(rng.integers(1000, 200000))
    for avg in (0.3, 0.9, 1.1, 3.0):
        eu, ev = er_graph(n, avg / n, seed * 10 + int(avg * 10))
        off, col = orc.csr_from_edges(n, eu, ev)
        check(fg, orc, off, col, f"er seed={seed} avg={avg}")


def test_rmat_and_grids(fg, orc):
    for s in (8, 12, 16, 18):
        off, col = synth.rmat_csr(s)
        check(fg, orc, off, col, f"rmat{s}")
    for r, c in ((1, 1), (1, 700), (33, 65), (512, 512)):
        off, col = synth.grid_csr(r, c)
        check(fg, orc, off, col, f"grid{r}x{c}")


def test_degenerate(fg, orc):
    # no edges; one vertex; a path written in descending order; a star whose
    # centre has the largest id; two components interleaved by parity
    off, col = orc.csr_from_edges(9, np.zeros(0, np.int32), np.zeros(0, np.int32))
    check(fg, orc, off, col, "empty")
    off, col = orc.csr_from_edges(1, np.zeros(0, np.int32), np.zeros(0, np.int32))
    check(fg, orc, off, col, "single")
    n = 5000
    eu = np.arange(n - 1, 0, -1, dtype=np.int32)
    off, col = orc.csr_from_edges(n, eu, eu - 1)
    check(fg, orc, off, col, "path")
    leaves = np.arange(0, 9999, dtype=np.int32)
    off, col = orc.csr_from_edges(10000, leaves, np.full_like(leaves, 9999))
    check(fg, orc, off, col, "star")
    a = np.arange(0, 20000 - 2, dtype=np.int32)
    off, col = orc.csr_from_edges(20000, a, a + 2)
    check(fg, orc, off, col, "parity")


@pytest.mark.parametrize("deg", [3, 64, 1023, 1024, 1025, 1026, 9000])
def test_components_joined_by_long_rows_alone(fg, orc, deg):
    """Hubs outside the giant component whose only edge into it is past the
    first two entries of both its rows, so the hub's own row has to hook it:
    rows around the length at which they get a pass of their own."""
    hubs, G = 5, 60_000
    leaves = hubs * (deg - 1)
    chain = np.arange(leaves, leaves + G - 1, dtype=np.int32)
    eu, ev = [chain], [chain + 1]
    for h in range(hubs):
        hub = leaves + G + h
        mine = np.arange(h * (deg - 1), (h + 1) * (deg - 1), dtype=np.int32)
        eu += [np.full(deg, hub, np.int32)]
        ev += [np.append(mine, np.int32(leaves + 100 + 7 * h))]
    off, col = orc.csr_from_edges(leaves + G + hubs, np.concatenate(eu), np.concatenate(ev))
    check(fg, orc, off, col, f"joined by rows of {deg}")


def test_directed_graph_rejected(fg):
    off = np.array([0, 1, 1], np.int32)
    col = np.array([1], np.int32)
    g = fg.Graph(off, col, symmetric=False, validate=True)
    label = torch.empty(2, dtype=torch.int32, device="cuda")
    with pytest.raises(fg.FGError) as e:
        fg.cc_into(g, label)
    assert e.value.status == fg.FG_EUNSUPPORTED
    g.close()


@pytest.mark.slow
@pytest.mark.parametrize("name", ["rmat22", "grid4096"])
def test_workload_graphs(fg, orc, name):
    off, col, _ = workloads.graph(name)
    announce(f"cc {name}")
    g = fg.Graph(off, col, symmetric=True, validate=False)
    label, comps = fg.cc(g)
    got = to_np(label)
    g.close()
    want, wc = orc.cc(off, col)
    assert np.array_equal(got, want)
    assert comps == wc


def _cliques(sizes):
    """CSR of disjoint cliques."""
    deg = np.repeat(np.asarray(sizes) - 1, sizes)
    off = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    col, lo = [], 0
    for k in sizes:
        x = np.tile(np.arange(lo, lo + k, dtype=np.int32), (k, 1))
        col.append(x[~np.eye(k, dtype=bool)])
        lo += k
    return off, np.concatenate(col)


def test_large_components_of_medium_rows(fg, orc):
    """Rows of some hundred entries outside the giant component cost about
    what longer ones do (per entry), wherever the border between the passes
    lies."""
    us = {}
    for k in (60, 66, 100, 300, 1000, 1500):
        off, col = _cliques([k] * (1500 // k * 2))
        g = fg.Graph(off, col, validate=False)
        label = torch.empty(g.n, dtype=torch.int32, device="cuda")
        comps = torch.zeros(1, dtype=torch.int64, device="cuda")
        announce(f"cc cliques of {k}")
        fg.cc_into(g, label, comps)
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(10):
            fg.cc_into(g, label, comps)
        b.record()
        want, wc = orc.cc(off, col)
        assert np.array_equal(to_np(label), want) and int(comps) == wc
        us[k] = a.elapsed_time(b) * 100
        g.close()
    assert max(us.values()) < 4 * us[1500], us  # by one wave per 64 rows 26 times


@pytest.mark.parametrize("deg", [63, 65, 66, 67, 200])
def test_joined_by_rows_at_the_border(fg, orc, deg):
    test_components_joined_by_long_rows_alone(fg, orc, deg)


def test_count_into_host_memory(fg, orc):
    """The number of components into pinned host memory and into unaligned
    device memory: copied there behind the kernels."""
    off, col = synth.rmat_csr(12)
    g = fg.Graph(off, col)
    want, wc = orc.cc(off, col)
    label = torch.empty(g.n, dtype=torch.int32, device="cuda")
    host = torch.full((1,), -9, dtype=torch.int64, pin_memory=True)
    dev = torch.zeros(24, dtype=torch.uint8, device="cuda")[4:12]
    announce("cc count into pinned host memory")
    for out in (host, dev):
        for _ in range(2):
            fg.cc_into(g, label, out)
            assert np.array_equal(to_np(label), want)
            assert int(out.cpu().numpy().view(np.int64)[0]) == wc
    g.close()
