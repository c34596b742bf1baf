"""GPU: a compute that runs out of memory, at each of its allocations in turn,
leaves the handle usable: the next compute on it, without the limit, gives the
oracle's results.

The limit is narrowed down to every place where one more block is had (the
allocator's blocks are multiples of 512 bytes), told apart by the peak of
the bytes in use and by the bytes that the handle holds after the failure."""
import numpy as np
import pytest

from oracle import native
from paper_2105_00110_amd import graphgen as gg
from tests.test_gpu_tiles import _dense_core

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

STEP = 512
# above 16384 vertices the scans take scratch of their own
FORMS = {
    "mid": (lambda: gg.ba(20_000, 4, seed=11), {"algorithm": 2}),
    # beside the core's matrix the later arrays are what does not fit
    "mid_core": (lambda: _dense_core(20_000, 2048, 0.35, 12, 20_000), {"algorithm": 2}),
    # the symmetric adjacency that the low pivot aggregates over; as one small
    # graph by one workgroup it sorts for it
    "low": (lambda: gg.ba(20_000, 4, seed=11), {"algorithm": 1}),
    # AUTO: the middle pivot, and the slot merge where it does not fit
    "short_rows": (lambda: gg.disjoint_cliques(80, 100), None),
    "low_small": (lambda: gg.clique(170), {"algorithm": 1}),
}


@pytest.mark.parametrize("name", sorted(FORMS))
def test_compute_again_after_each_failed_allocation(tclib, name):
    graph, tuning = FORMS[name]
    src, dst, n = graph()
    ref = native.o2_paper(src, dst, n)

    def probe(steps):
        """Computes with room for steps * STEP bytes; how far it got."""
        tclib.tc_set_memory_limit(0)
        g = tclib.Graph.from_edges(src, dst, n)
        tclib.tc_trim_memory()
        before = tclib.tc_memory_stats(reset_peaks=True)["in_use"]
        tclib.tc_set_memory_limit(before + steps * STEP)
        failed = False
        try:
            g.compute(tuning)
        except tclib.TCError as e:
            assert e.status == tclib.TC_ERR_BUDGET
            failed = True
        tclib.tc_set_memory_limit(0)
        got = (failed, tclib.tc_memory_stats()["peak_in_use"] - before, g.device_bytes())
        if failed:
            g.compute(tuning)
        r = g.results()
        np.testing.assert_array_equal(r["support"], ref.sup)
        np.testing.assert_array_equal(r["num"], ref.num)
        g.close()
        return got

    try:
        g = tclib.Graph.from_edges(src, dst, n)
        hi = g.compute_bytes(tuning) // STEP + 1
        g.close()
        ends = {0: probe(0), hi: probe(hi)}
        assert ends[0][0] and not ends[hi][0]
        todo, places = [(0, hi)], 0
        while todo:
            a, b = todo.pop()
            if ends[a] == ends[b]:
                continue
            if b == a + 1:
                places += 1
                print("[case] memory limits", name, "place", places, "at", b * STEP, ends[b], flush=True)
                continue
            m = (a + b) // 2
            ends[m] = probe(m)
            todo += [(a, m), (m, b)]
        assert places >= 8, places
    finally:
        tclib.tc_set_memory_limit(0)
        tclib.tc_trim_memory()


# between 200 and 600 thousand edges AUTO may take the middle pivot; what
# tc_compute_bytes asks for there stays the low pivot's bound, and holds: with the
# cache emptied after the build, every block of the count is new
PROMISED = {
    "clique_660": lambda: gg.clique(660),
    "clique_1090": lambda: gg.clique(1090),
    "core": lambda: _dense_core(2048, 2048, 0.28, 13, 0),
    "flat_rows": lambda: gg.ba(3000, 150, seed=1),
    "rmat_15": lambda: gg.rmat(15, 16, seed=1),
    "rmat_16": lambda: gg.rmat(16, 8, seed=1),
}


@pytest.mark.parametrize("name", sorted(PROMISED))
def test_compute_bytes_of_mid_sized_graphs(tclib, name):
    src, dst, n = PROMISED[name]()
    g = tclib.Graph.from_edges(src, dst, n)
    assert 200_000 <= g.m < 600_000
    tclib.tc_trim_memory()
    need = g.compute_bytes()
    assert need == g.compute_bytes({"algorithm": tclib.TC_ALGO_LOW_PIVOT})
    before = tclib.tc_memory_stats(reset_peaks=True)["held"]
    g.compute()
    grown = tclib.tc_memory_stats()["peak_held"] - before
    ws = g.work_stats()
    print("[case] compute bytes", name, "edges", g.m, "longest row", ws["max_dplus"], "algorithm",
          ws["algorithm"], "bound", need, "growth", grown, flush=True)
    assert ws["algorithm"] == tclib.TC_ALGO_MID_PIVOT
    assert grown <= need
    g.close()


def _sparse_with_cliques(n, m, size):
    """A sparse random graph with a clique on its first vertices: many vertices per
    edge, and rows that the slot merge does not take."""
    rng = np.random.default_rng(21)
    s, d, _ = gg.clique(size)
    a, b = rng.integers(0, n, (2, m)).astype(np.int32)
    return np.concatenate([s, a]), np.concatenate([d, b]), n


# whatever the low pivot fits into is enough for AUTO, also where the middle pivot's
# count fits and its aggregation does not
@pytest.mark.parametrize("name", ["sparse", "dense"])
def test_auto_fits_where_the_low_pivot_does(tclib, name):
    src, dst, n = _sparse_with_cliques(200_000, 210_000, 220) if name == "sparse" else gg.clique(700)
    ref = native.o2_paper(src, dst, n)

    def fits(steps, tuning):
        tclib.tc_set_memory_limit(0)
        g = tclib.Graph.from_edges(src, dst, n)
        assert 200_000 <= g.m < 600_000
        tclib.tc_trim_memory()
        tclib.tc_set_memory_limit(tclib.tc_memory_stats()["in_use"] + steps * 4096)
        try:
            g.compute(tuning)
            tclib.tc_set_memory_limit(0)
            np.testing.assert_array_equal(g.results()["num"], ref.num)
            return g.work_stats()["algorithm"]
        except tclib.TCError as e:
            assert e.status == tclib.TC_ERR_BUDGET
            return 0
        finally:
            tclib.tc_set_memory_limit(0)
            g.close()

    low = {"algorithm": tclib.TC_ALGO_LOW_PIVOT}
    try:
        g = tclib.Graph.from_edges(src, dst, n)
        hi = g.compute_bytes() // 4096 + 1
        g.close()
        a, b = 0, hi  # the least room for the low pivot
        assert fits(hi, low)
        while a + 1 < b:
            m = (a + b) // 2
            a, b = (a, m) if fits(m, low) else (m, b)
        used = [fits(b + (hi - b) * i // 60, None) for i in range(61)]
        print("[case] least room", b * 4096, "of", hi * 4096, "forms", used, flush=True)
        assert all(used), used
        assert used[-1] == tclib.TC_ALGO_MID_PIVOT
    finally:
        tclib.tc_set_memory_limit(0)
        tclib.tc_trim_memory()


def test_top_k_of_few_vertices_under_a_limit(tclib):
    # room for a sort of 40 vertices (under 10 KB), not for the selection's
    # histograms (64 KB)
    src, dst, n = gg.clique(40)
    ref = native.o2_paper(src, dst, n)
    g = tclib.Graph.from_edges(src, dst, n)
    g.compute()
    try:
        tclib.tc_trim_memory()
        tclib.tc_set_memory_limit(tclib.tc_memory_stats()["in_use"] + (32 << 10))
        verts, vals = g.top_k(10)
    finally:
        tclib.tc_set_memory_limit(0)
    np.testing.assert_array_equal(verts, np.arange(10))
    np.testing.assert_array_equal(vals.view(np.uint64), ref.tc[:10].view(np.uint64))
    g.close()


def test_estimate_holds_for_many_isolated_vertices(tclib):
    # a triangle among 24 million vertices: what counts is the bytes per vertex
    n = 24_000_000
    src, dst = np.array([5, 1000, n - 1], np.int32), np.array([1000, n - 1, 5], np.int32)
    est = tclib.tc_estimate_device_bytes(src.shape[0], n)
    try:
        tclib.tc_trim_memory()
        before = tclib.tc_memory_stats(reset_peaks=True)["in_use"]
        tclib.tc_set_memory_limit(tclib.tc_memory_stats()["held"] + est)
        g = tclib.Graph.from_edges(src, dst, n)
        g.compute()
        used = tclib.tc_memory_stats()["peak_in_use"] - before
        verts, _ = g.top_k(3)
        g.close()
    finally:
        tclib.tc_set_memory_limit(0)
        tclib.tc_trim_memory()
    print("[case] estimate", est, "used", used, flush=True)
    assert list(verts) == [5, 1000, n - 1]
    assert used <= est


# all ids distinct, a power of two of them and not: keys, the sort's other buffer and
# its counts, the ids; what the lookup needs beside the map lies in those
@pytest.mark.parametrize("pairs", [1, 2, 1 << 16, 100_000])
def test_relabel_within_the_sorts_memory(tclib, pairs):
    ids = np.random.default_rng(3).permutation(8 * pairs)[:2 * pairs].astype(np.int64) << 20
    src, dst = torch.from_numpy(ids[:pairs]).cuda(), torch.from_numpy(ids[pairs:]).cuda()
    s32, d32 = (torch.empty(pairs, dtype=torch.int32, device="cuda") for _ in range(2))
    tclib.tc_trim_memory()
    before = tclib.tc_memory_stats(reset_peaks=True)["in_use"]
    n = tclib.tc_relabel_ids(src.data_ptr(), dst.data_ptr(), pairs, s32.data_ptr(), d32.data_ptr(), None,
                             tclib.TC_MEM_DEVICE, None)
    used = tclib.tc_memory_stats()["peak_in_use"] - before
    want = np.sort(ids)
    assert n == 2 * pairs
    np.testing.assert_array_equal(s32.cpu().numpy(), np.searchsorted(want, ids[:pairs]))
    np.testing.assert_array_equal(d32.cpu().numpy(), np.searchsorted(want, ids[pairs:]))
    # three arrays of 8 bytes an id, 1 KB of counts per 2048 ids and two more, blocks
    # rounded up to 512 bytes (2 MiB from 1 MiB on)
    n2 = 2 * pairs
    def block(b):
        unit = 512 if b < 1 << 20 else 2 << 20
        return (b + unit - 1) // unit * unit

    rounded = [8 * n2] * 3 + [1024 * (n2 // 2048 + 2), 4 * (n2 // 4096 + 1), 4, 16]
    print("[case] relabel", pairs, "used", used, flush=True)
    assert used <= sum(block(b) for b in rounded)
