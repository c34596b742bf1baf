"""GPU parity at the edges of tiles, classes and dispatch rules.

Each test takes one kernel (or one rule that picks a kernel) at the sizes
where it can go wrong: a tile exactly full, one more, the first and last row
of a class, long runs of empty rows.  Expected values come from the CPU
oracle; all integers are equal and the quotient bit-identical.
"""
import numpy as np
import pytest

from oracle import native
from paper_2105_00110_amd import graphgen as gg
from tests.test_gpu_fused import check_all, run_fused
from tests.test_gpu_parity import _csr, _say, assert_parity, run_gpu

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _star(n, center, leaves):
    leaves = np.asarray(leaves, np.int32)
    return np.full(leaves.shape[0], center, np.int32), leaves, n


CSR_TILE = 4096  # row ends plus entries per workgroup
CSR_CASES = {
    # n + entries at a tile, one short and one past it (upper triangle only)
    "full_tile": lambda: _star(CSR_TILE - 100, 7, np.arange(8, 108)),
    "one_short": lambda: _star(CSR_TILE - 100, 7, np.arange(8, 107)),
    "one_past": lambda: _star(CSR_TILE - 100, 7, np.arange(8, 109)),
    # a row over several tiles whose neighbours lie below and above it
    "hub": lambda: _star(3 * CSR_TILE, 5000, np.setdiff1d(np.arange(3 * CSR_TILE), [5000])),
    # whole tiles of empty rows before, between and after the edges
    "empty_runs": lambda: (np.array([9000, 9000, 9001, 20000, 20000, 20001], np.int32),
                           np.array([9001, 9002, 9002, 20001, 29000, 29000], np.int32), 40000),
    "no_edges": lambda: (np.zeros(0, np.int32), np.zeros(0, np.int32), 2 * CSR_TILE),
    "skewed": lambda: gg.rmat(13, 16, seed=8),
}


@pytest.mark.parametrize("name", sorted(CSR_CASES))
def test_simple_sorted_csr_tiles(tclib, name):
    src, dst, n = CSR_CASES[name]()
    ref = native.o2_paper(src, dst, n)
    sym = _csr(np.concatenate([ref.eu, ref.ev]), np.concatenate([ref.ev, ref.eu]), n)
    for form, (rp, col) in (("symmetric", sym), ("upper", _csr(ref.eu, ref.ev, n))):
        _say("simple sorted CSR tiles", name, form, "n", n, "entries", col.shape[0])
        g = tclib.Graph.from_csr(torch.as_tensor(rp).cuda(), torch.as_tensor(col).cuda(), n,
                                 assume_simple_sorted=True)
        st = g.compute()
        res = g.results()
        res["eu"], res["ev"] = g.edges()
        res["status"], res["m"] = st, g.m
        g.close()
        assert_parity(res, ref)


ID_TILE = 4096  # sorted ids per workgroup of the deduplication
RELABEL_CASES = {
    "one_id": lambda rng: np.full(2 * 70, 123456789, np.int64),
    "full_tile": lambda rng: rng.permutation(ID_TILE).astype(np.int64) * 3,
    "past_tile": lambda rng: rng.permutation(ID_TILE + 2).astype(np.int64) * 3,
    "two_tiles_repeats": lambda rng: rng.integers(5, 9, 2 * ID_TILE),
    # the whole range of an id, and all but one id in a single bucket
    "extremes": lambda rng: np.concatenate([np.array([0, 2**63 - 1], np.int64),
                                            rng.integers(0, 2**63 - 1, 998)]),
    "clustered": lambda rng: np.concatenate([np.array([2**62], np.int64),
                                             rng.integers(0, 5000, 9999)]),
}


@pytest.mark.parametrize("name", sorted(RELABEL_CASES))
def test_relabel_tiles_and_ranges(tclib, name):
    ids = RELABEL_CASES[name](np.random.default_rng(11))
    src, dst = ids[::2].copy(), ids[1::2].copy()
    _say("relabel tiles", name, "pairs", src.shape[0])
    s32, d32, got, n = tclib.relabel(src, dst)
    want = np.unique(ids)
    assert n == want.shape[0]
    np.testing.assert_array_equal(got, want)
    np.testing.assert_array_equal(s32, np.searchsorted(want, src))
    np.testing.assert_array_equal(d32, np.searchsorted(want, dst))


def _rank(tcv, k):
    """The oracle's ranking: value descending, then smaller id."""
    order = np.lexsort((np.arange(tcv.shape[0]), -tcv))[:k]
    return order.astype(np.int32), tcv[order]


TOPK_GRAPHS = {
    "rmat_s14": lambda: gg.rmat(14, 16, seed=5),
    # many equal values: 1200 copies of K5 (6000 ties), and 500 (2500)
    "ties_above_cap": lambda: gg.disjoint_cliques(1200, 5),
    "ties_below_cap": lambda: gg.disjoint_cliques(500, 5),
    "all_zero": lambda: (np.arange(0, 9999, dtype=np.int32), np.arange(1, 10000, dtype=np.int32),
                         10000),
    "one_vertex_more": lambda: gg.ba(4097, 4, seed=3),
    "tiny": lambda: gg.clique(3),
}


@pytest.mark.parametrize("name", sorted(TOPK_GRAPHS))
def test_top_k_selection(tclib, name):
    src, dst, n = TOPK_GRAPHS[name]()
    ref = native.o2_paper(src, dst, n)
    g = tclib.Graph.from_edges(src, dst, n)
    g.compute()
    for k in (1, 2, 10, 1000, 1024, 1025, n):  # selection up to 1024, sort above
        k = min(k, n)
        _say("top k", name, "k", k, "n", n)
        verts, vals = g.top_k(k)
        want_v, want = _rank(ref.tc, k)
        np.testing.assert_array_equal(verts, want_v)
        np.testing.assert_array_equal(vals.view(np.uint64), want.view(np.uint64))
    g.close()


# ids per sort: the last size whose tile counts the scatter sums itself, one
# tile more, and both sides of the big tiles
@pytest.mark.parametrize("count", [2048, 128 * 2048, 128 * 2048 + 2, (1 << 22) - 2, 1 << 22])
def test_sort_tile_forms(tclib, count):
    ids = np.random.default_rng(13).integers(0, 1 << 34, count)
    src, dst = ids[::2].copy(), ids[1::2].copy()
    _say("sort tile forms", count)
    s32, d32, got, n = tclib.relabel(src, dst)
    want = np.unique(ids)
    assert n == want.shape[0]
    np.testing.assert_array_equal(got, want)
    np.testing.assert_array_equal(s32, np.searchsorted(want, src))
    np.testing.assert_array_equal(d32, np.searchsorted(want, dst))


# vertices per scan: one round and two of the single workgroup, then tiles
@pytest.mark.parametrize("n", [8192, 8193, 16384, 16385, 5 * 4096 + 1])
def test_scan_forms(tclib, n):
    src, dst, _ = gg.er(n, 12.0 / n, seed=n)
    # a triangle on the last vertices: their rows end every scan
    src = np.concatenate([src, np.array([n - 1, n - 2, n - 3], np.int32)])
    dst = np.concatenate([dst, np.array([n - 2, n - 3, n - 1], np.int32)])
    _say("scan forms, n", n)
    assert_parity(run_gpu(tclib, src, dst, n), native.o2_paper(src, dst, n))


def _hub_and_clique(n):
    """A star on the last vertex plus K_6 on the lowest ids: the hub is the top
    rank, the others fill the ranks below."""
    s, d, _ = gg.clique(6)
    return (np.concatenate([s, np.full(n - 1, n - 1, np.int32)]),
            np.concatenate([d, np.arange(n - 1, dtype=np.int32)]), n)


# the slot merge: rows at its window of 8 entries, the ranks kept in LDS (2048)
# and just more, the longest row that takes it (128) and one more
SLOT_GRAPHS = {
    **{f"K{k}": (lambda k=k: gg.clique(k)) for k in (2, 8, 9, 10, 17, 18, 129, 130)},
    "top_ranks": lambda: _hub_and_clique(2048),
    "top_ranks_past": lambda: _hub_and_clique(2049),
    "triangle_free": lambda: gg.single_triangle_with_pendants((0, 4000, 1)),
    "ba_cliques": lambda: gg.ba(6000, 12, seed=9),
}


@pytest.mark.parametrize("name", sorted(SLOT_GRAPHS))
def test_slot_merge_edges(tclib, name):
    src, dst, n = SLOT_GRAPHS[name]()
    _say("slot merge", name, "n", n)
    assert_parity(run_gpu(tclib, src, dst, n), native.o2_paper(src, dst, n))
    # the same handle after the middle pivot, and the algebraic numerator
    g = tclib.Graph.from_edges(src, dst, n)
    g.compute({"algorithm": tclib.TC_ALGO_MID_PIVOT})
    a = g.results()
    g.compute()
    b = g.results()
    for k in ("tri", "support", "triG", "num"):
        np.testing.assert_array_equal(a[k], b[k])
    np.testing.assert_array_equal(g.numerator_algebraic(), b["num"])
    g.close()


# short rows whose edges have many triangles (as many as half their entries) cost
# the merge an atomic add each: the middle pivot takes them, the merge the others
@pytest.mark.parametrize("name,mid", [("cliques", True), ("batch_rmat", True), ("flat", False),
                                      ("few_cliques", False)])
def test_slot_merge_or_middle_pivot(tclib, name, mid):
    if name == "batch_rmat":
        graphs = [gg.rmat(12, 16, seed=40 + i % 4) for i in range(40)]
        po = np.cumsum([0] + [len(x[0]) for x in graphs])
        vo = np.cumsum([0] + [x[2] for x in graphs])
        src, dst = (np.concatenate([x[k] for x in graphs]).astype(np.int32) for k in (0, 1))
        g = tclib.Graph.batch(src, dst, po, vo)
        off = np.repeat(vo[:-1], np.diff(po)).astype(np.int32)
        src, dst, n = src + off, dst + off, int(vo[-1])
    else:
        src, dst, n = {"cliques": lambda: gg.disjoint_cliques(400, 100),
                       "flat": lambda: gg.ba(100_000, 16, seed=2),
                       "few_cliques": lambda: gg.disjoint_cliques(30, 100)}[name]()
        g = tclib.Graph.from_edges(src, dst, n)
    _say("slot merge or middle pivot", name)
    g.compute()
    r, ws = g.results(), g.work_stats()
    g.close()
    assert ws["max_dplus"] <= 128
    assert ws["algorithm"] == (tclib.TC_ALGO_MID_PIVOT if mid else tclib.TC_ALGO_LOW_PIVOT)
    ref = native.o2_paper(src, dst, n)
    for k, want in (("support", ref.sup), ("tri", ref.tri), ("num", ref.num)):
        np.testing.assert_array_equal(r[k], want)


def _wide(graph, n):
    """The graph with isolated vertices up to n: past the sizes of one workgroup."""
    src, dst, _ = graph
    return src, dst, n


def _long_rows(lows):
    """`lows` vertices with 127 or 128 higher neighbours each, out of 128 hubs of
    which three are linked: rows that end at and across the runs of a workgroup,
    with a triangle here and there."""
    keep = np.ones((lows, 128), bool)
    keep[::3, 5] = False
    v, h = np.nonzero(keep)
    hubs = np.array([[9, 70], [70, 127], [9, 127]])
    return (np.concatenate([128 + v, hubs[:, 0]]).astype(np.int32),
            np.concatenate([h, hubs[:, 1]]).astype(np.int32), 128 + max(lows, 4500))


# as above, on builds that take the slot merge's own kernels: rows at its window,
# the longest row, and graphs of as many vertices as the sums keep in LDS (8192)
# and one more; runs of 256 slots a workgroup and of 2048
SLOT_KERNEL_GRAPHS = {
    **{f"K{k}": (lambda k=k: _wide(gg.clique(k), 5000)) for k in (3, 8, 9, 10, 17, 18, 129)},
    "window": lambda: _hub_and_clique(8192),
    "window_past": lambda: _hub_and_clique(8193),
    "triangle_free": lambda: _wide(gg.single_triangle_with_pendants((0, 4000, 1)), 6000),
    "long_rows": lambda: _long_rows(700),
    "long_rows_long_runs": lambda: _long_rows(64_000),
}


@pytest.mark.parametrize("name", sorted(SLOT_KERNEL_GRAPHS))
def test_slot_merge_kernels(tclib, name):
    src, dst, n = SLOT_KERNEL_GRAPHS[name]()
    _say("slot merge kernels", name, "n", n)
    assert n > 4096  # not one workgroup's
    ref = native.o2_paper(src, dst, n)
    assert_parity(run_gpu(tclib, src, dst, n), ref)
    g = tclib.Graph.from_edges(src, dst, n)
    g.compute()
    ws = g.work_stats()
    g.close()
    assert ws["max_dplus"] <= 128 and ws["algorithm"] == tclib.TC_ALGO_LOW_PIVOT
    if name.startswith("long"):
        assert ws["max_dplus"] == 128


def test_slot_merge_batch(tclib):
    # graphs that end inside wavefronts, with and without triangles
    graphs = [gg.clique(3 + i % 9) if i % 3 else (np.arange(5, dtype=np.int32),
                                                 np.arange(1, 6, dtype=np.int32), 7 + i % 60)
              for i in range(90)]
    po = np.cumsum([0] + [len(g[0]) for g in graphs])
    vo = np.cumsum([0] + [g[2] for g in graphs])
    g = tclib.Graph.batch(np.concatenate([x[0] for x in graphs]),
                          np.concatenate([x[1] for x in graphs]), po, vo)
    _say("slot merge batch", len(graphs))
    g.compute()
    r, eoff = g.results(), g.edge_offsets()
    for i, (s, d, n) in enumerate(graphs):
        ref = native.o2_paper(s, d, n)
        np.testing.assert_array_equal(r["support"][eoff[i]:eoff[i + 1]], ref.sup)
        np.testing.assert_array_equal(r["tri"][vo[i]:vo[i + 1]], ref.tri)
        np.testing.assert_array_equal(r["num"][vo[i]:vo[i + 1]], ref.num)
        np.testing.assert_array_equal(r["tc"][vo[i]:vo[i + 1]].view(np.uint64), ref.tc.view(np.uint64))
        assert int(r["triG"][i]) == ref.triG
    g.close()


# ranks by graph: (graph, degree) keys of 32 bits at most, graphs without
# vertices between others, a graph above the sums' LDS window of 8192 ranks,
# runs of slots that end inside graphs; and keys of more than 32 bits, where
# ranks follow degrees alone
BATCH_RANKS = {
    "uneven": [gg.ba(9000, 12, seed=1), gg.clique(9), (np.zeros(0, np.int32), np.zeros(0, np.int32), 0),
               gg.ba(700, 3, seed=2), gg.ba(20_000, 7, seed=3), gg.clique(2), gg.ba(60, 16, seed=4)],
    # from 2^20 pairs on a thread takes eight, of workgroups that span many graphs
    "many_pairs": [gg.ba(40_000, 16, seed=5), gg.clique(3), gg.ba(36_000, 15, seed=6)]
                  + [gg.clique(2 + i % 11) for i in range(700)],
    "wide_keys": [(np.array([5, 5, 1 << 20], np.int32), np.array([1 << 20, 77, 77], np.int32),
                   (1 << 20) + 1)] + [gg.clique(3 + i % 7) for i in range(4095)],
}


@pytest.mark.parametrize("name", sorted(BATCH_RANKS))
def test_batch_ranks(tclib, name):
    graphs = BATCH_RANKS[name]
    po = np.cumsum([0] + [len(g[0]) for g in graphs])
    vo = np.cumsum([0] + [g[2] for g in graphs])
    src, dst = (np.concatenate([g[k] for g in graphs]) for k in (0, 1))
    g = tclib.Graph.batch(src, dst, po, vo)
    _say("batch ranks", name, "n", int(vo[-1]))
    g.compute()
    r = g.results()
    g.close()
    off = np.repeat(vo[:-1], np.diff(po))
    ref = native.o2_paper((src + off).astype(np.int32), (dst + off).astype(np.int32), int(vo[-1]))
    np.testing.assert_array_equal(r["support"], ref.sup)
    np.testing.assert_array_equal(r["tri"], ref.tri)
    np.testing.assert_array_equal(r["num"], ref.num)
    tri = np.concatenate([[0], np.cumsum(ref.tri)])
    np.testing.assert_array_equal(3 * r["triG"].astype(np.int64), tri[vo[1:]] - tri[vo[:-1]])


def _pairs_over(n, P, seed):
    """P random pairs over n vertices, a clique on the top ids among them."""
    rng = np.random.default_rng(seed)
    s, d, _ = gg.clique(12)
    src, dst = rng.integers(0, n, (2, P)).astype(np.int32)
    k = min(P, s.shape[0])
    src[:k], dst[:k] = s[:k] + (n - 12), d[:k] + (n - 12)
    return src, dst, n


def _edges_over(n, m, seed):
    """m distinct edges over n vertices, a clique on the top ids among them."""
    rng = np.random.default_rng(seed)
    s, d, _ = gg.clique(60)
    k = np.unique(np.concatenate([(s + n - 60) * n + d + n - 60, rng.integers(0, n * n, 3 * m)]))
    a, b = k // n, k % n
    k = np.unique(np.minimum(a, b) * n + np.maximum(a, b))
    k = k[k // n < k % n]
    top = k[k // n >= n - 60]
    k = np.concatenate([top, rng.permutation(k[k // n < n - 60])])[:m]
    assert k.shape[0] == m
    return (k // n).astype(np.int32), (k % n).astype(np.int32), n


# the tiers of the fused launch at 1024 threads: LDS (16384 pairs, 4096
# vertices), LDS for vertices only (2^20 pairs, 21504 vertices), workspace
FUSED_TIERS = {
    "lds_full": lambda: _pairs_over(4096, 16384, 1),
    "lds_pairs_past": lambda: _pairs_over(4096, 16385, 2),
    "lds_vertices_past": lambda: _pairs_over(4097, 16000, 3),
    "tile_full": lambda: _pairs_over(6000, 3 * 8192, 4),
    "tile_past": lambda: _pairs_over(6000, 3 * 8192 + 1, 5),
    "few_pairs": lambda: _pairs_over(21504, 70, 6),
    "vertices_full": lambda: _pairs_over(21504, 100_000, 7),
    "vertices_past": lambda: _pairs_over(21505, 100_000, 8),
    "dense": lambda: gg.clique(400),
    "most_pairs": lambda: gg.rmat(14, 64, seed=9),
    "pairs_past": lambda: gg.rmat(14, 64, seed=9, num_pairs=(1 << 20) + 1),
    "longest_rows": lambda: gg.clique(1440),
    # the merge's LDS cache: every slot of the graph, and one more
    "cache_full": lambda: _edges_over(5000, 153_600 // 4 - 8 - 5000, 10),
    "cache_past": lambda: _edges_over(5000, 153_600 // 4 - 8 - 5000 + 1, 11),
}


def test_fused_tiers(tclib):
    graphs = [FUSED_TIERS[k]() for k in sorted(FUSED_TIERS)]
    refs = [native.o2_paper(*g) for g in graphs]
    for order in ("largest_first", None):
        _say("fused tiers", sorted(FUSED_TIERS), order)
        fb, res = run_fused(tclib, graphs, order=order)
        check_all(fb, res, graphs, refs)



# the same limits at 256 and 512 threads, with the merge's cache (bytes of LDS)
FUSED_CACHE = {256: 41_984, 512: 76_800}


@pytest.mark.parametrize("block", sorted(FUSED_CACHE))
def test_fused_tiers_of_smaller_workgroups(tclib, block):
    b, words = block, FUSED_CACHE[block] // 4 - 8
    graphs = [_pairs_over(4 * b, 16 * b, 1), _pairs_over(4 * b, 16 * b + 1, 2),
              _pairs_over(4 * b + 1, 16 * b - 100, 3), _pairs_over(6 * b, 24 * b, 4),
              _pairs_over(6 * b, 24 * b + 1, 5), _pairs_over(21 * b, 70, 6),
              _pairs_over(21 * b, 100 * b, 7), _pairs_over(21 * b + 1, 100 * b, 8), gg.clique(400),
              gg.rmat(12, 256, seed=9), gg.rmat(12, 256, seed=9, num_pairs=(1 << 20) + 1),
              gg.clique(1440), _edges_over(5 * b, words - 5 * b, 10),
              _edges_over(5 * b, words - 5 * b + 1, 11)]
    refs = [native.o2_paper(*g) for g in graphs]
    for wg in (1, 4):
        _say("fused tiers", block, "threads", wg, "per CU")
        fb, res = run_fused(tclib, graphs, tuning={"block": block, "wg_per_cu": wg})
        check_all(fb, res, graphs, refs)


# one small graph by one workgroup: its largest size and one more of each, and
# rows above the slot merge's limit (the general count on such a build)
SINGLE_GRAPHS = {
    "one_pair": lambda: (np.array([0], np.int32), np.array([1], np.int32), 2),
    "one_loop": lambda: (np.array([0], np.int32), np.array([0], np.int32), 1),
    "full": FUSED_TIERS["lds_full"],
    "pairs_past": FUSED_TIERS["lds_pairs_past"],
    "vertices_past": FUSED_TIERS["lds_vertices_past"],
    "long_rows": lambda: gg.clique(180),
    "star": lambda: _star(4096, 9, np.setdiff1d(np.arange(4096), [9])),
    "repeats": lambda: (np.tile(np.array([1, 2, 0], np.int32), 5000),
                        np.tile(np.array([2, 0, 1], np.int32), 5000), 3),
}


@pytest.mark.parametrize("name", sorted(SINGLE_GRAPHS))
def test_single_workgroup_graphs(tclib, name):
    src, dst, n = SINGLE_GRAPHS[name]()
    ref = native.o2_paper(src, dst, n)
    _say("single workgroup", name, "n", n, "pairs", src.shape[0])
    assert_parity(run_gpu(tclib, src, dst, n), ref)
    assert_parity(run_gpu(tclib, src, dst, n, device=False), ref)
    for algorithm in (tclib.TC_ALGO_LOW_PIVOT, tclib.TC_ALGO_MID_PIVOT):
        assert_parity(run_gpu(tclib, src, dst, n, tuning={"algorithm": algorithm}), ref)
    g = tclib.Graph.from_edges(src, dst, n)
    g.compute()
    np.testing.assert_array_equal(g.numerator_algebraic(), ref.num)
    assert g.work_stats()["triangles"] == ref.triG
    g.compute()  # again on the same handle
    np.testing.assert_array_equal(g.results()["support"], ref.sup)
    g.close()


def _dense_core(n, k, density, seed, extra):
    """A random graph of the given density on k of n vertices, shuffled, and extra random pairs."""
    rng = np.random.default_rng(seed)
    a, b = np.nonzero(np.triu(rng.random((k, k)) < density, 1))
    ids = rng.permutation(n)
    src = np.concatenate([ids[a], rng.integers(0, n, extra)])
    dst = np.concatenate([ids[b], rng.integers(0, n, extra)])
    return src.astype(np.int32), dst.astype(np.int32), n


# the middle pivot's core of the 2048, 4096, ... highest ranks, taken by matrix
# products: the whole graph, one rank below it, a core cut out of a larger
# dense part, several panels of tiles, and a core with all its edges
CORE_GRAPHS = {
    "whole": lambda: _dense_core(2048, 2048, 0.35, 1, 0),
    "one_below": lambda: _dense_core(2049, 2049, 0.35, 2, 0),
    "cut": lambda: _dense_core(9000, 2600, 0.4, 3, 40_000),
    "panels": lambda: _dense_core(20_000, 4200, 0.3, 4, 100_000),
    "clique": lambda: _dense_core(3000, 2100, 2.0, 5, 5000),
    "skewed": lambda: gg.rmat(16, 16, seed=3),
}


@pytest.mark.parametrize("name", sorted(CORE_GRAPHS))
def test_core_products(tclib, name):
    src, dst, n = CORE_GRAPHS[name]()
    _say("core products", name, "n", n)
    assert_parity(run_gpu(tclib, src, dst, n), native.o2_paper(src, dst, n))
    g = tclib.Graph.from_edges(src, dst, n)
    g.compute({"algorithm": tclib.TC_ALGO_LOW_PIVOT})
    a = g.results()
    g.compute()
    ws = g.work_stats()
    assert ws["algorithm"] == tclib.TC_ALGO_MID_PIVOT
    # the candidates scanned: all oriented wedges but the core's
    scanned = ws["cand_light"] + ws["cand_heavy"] + ws["cand_huge"]
    assert scanned == 0 if name == "whole" else scanned <= ws["wedges"]
    b = g.results()
    for k in ("tri", "support", "triG", "num"):
        np.testing.assert_array_equal(a[k], b[k])
    g.close()


# the scan leaves out at least the wedges of the smallest core, the 2048 highest ranks
@pytest.mark.parametrize("name", sorted(set(CORE_GRAPHS) - {"skewed"}))
def test_core_products_are_taken(tclib, name):
    src, dst, n = CORE_GRAPHS[name]()
    k = np.unique(np.minimum(src, dst).astype(np.int64) * n + np.maximum(src, dst))
    u, v = k // n, k % n
    u, v = u[u != v], v[u != v]
    rank = np.empty(n, np.int64)
    rank[np.lexsort((np.arange(n), np.bincount(np.concatenate([u, v]), minlength=n)))] = np.arange(n)
    d = np.bincount(np.minimum(rank[u], rank[v]), minlength=n)
    core = int((d * (d - 1) // 2)[-2048:].sum())
    g = tclib.Graph.from_edges(src, dst, n)
    g.compute()
    ws = g.work_stats()
    g.close()
    _say("core products taken", name, "wedges", ws["wedges"], "of the smallest core", core)
    assert core > 0 and ws["wedges"] == int((d * (d - 1) // 2).sum())
    assert ws["cand_light"] + ws["cand_heavy"] + ws["cand_huge"] <= ws["wedges"] - core


# orientation buckets at the edges of the size classes (8, 16, 32, 64, 128, 256
# and the sorts above), several of a class in one wavefront, in wavefronts of 16
# vertices and of 64 (from 2^19 on)
@pytest.mark.parametrize("n", [3000, (1 << 19) + 5000])
def test_orientation_buckets(tclib, n):
    # every hub links to `size` vertices of higher degree, so its bucket has that many
    sizes = [1, 7, 8, 9, 9, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 66, 127, 128, 129, 255, 256, 257]
    s, d, _ = gg.clique(600)
    src, dst = [s], [d]
    for rep in range(3):
        for i, size in enumerate(sizes):
            v = 600 + rep * len(sizes) + i if rep < 2 else n - 1 - i
            src.append(np.full(size, v, np.int32))
            dst.append(np.arange(size, dtype=np.int32) + 7 * rep)
    src, dst = np.concatenate(src).astype(np.int32), np.concatenate(dst).astype(np.int32)
    _say("orientation buckets", n)
    assert_parity(run_gpu(tclib, src, dst, n), native.o2_paper(src, dst, n))


# the middle pivot's items: short pivots with one, 15 to 17, 31 to 33 and 63 to 65
# pairs, and wavefront pivots (rows of 129 to 200) with one to 70 pairs
def test_mid_pivot_items(tclib):
    src, dst, nxt = [], [], 400
    s, d, _ = gg.clique(400)
    src.append(s), dst.append(d)
    for pairs in (1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 70):
        for row in (2, 60, 128, 129, 200):
            v, nxt = nxt, nxt + 1
            src.append(np.full(row, v)), dst.append(np.arange(row) + pairs)
            low = np.arange(nxt, nxt + pairs)  # lower ends, each also in the pivot's row
            nxt += pairs
            for t in (0, row // 2, row - 1):
                src.append(low), dst.append(np.full(pairs, pairs + t))
            src.append(low), dst.append(np.full(pairs, v))
    src, dst = np.concatenate(src).astype(np.int32), np.concatenate(dst).astype(np.int32)
    _say("mid pivot items", nxt)
    ref = native.o2_paper(src, dst, nxt)
    g = tclib.Graph.from_edges(src, dst, nxt)
    g.compute({"algorithm": tclib.TC_ALGO_MID_PIVOT})
    r = g.results()
    g.close()
    for k, want in (("support", ref.sup), ("tri", ref.tri), ("num", ref.num)):
        np.testing.assert_array_equal(r[k], want)


# a caller's number of pairs holds, the default's is the library's below 2^23 edges:
# which of the two launches has the work of the pivots of 129 to 512 entries
def test_light_bitmap_pairs_as_chosen(tclib):
    src, dst, n = gg.rmat(15, 16, seed=5)
    tclib.tc_set_profiling(True)
    try:
        g = tclib.Graph.from_edges(src, dst, n)
        ms = {}
        for pairs in (64, 1_000_000):
            t = {"algorithm": tclib.TC_ALGO_MID_PIVOT, "light_bitmap_pairs": pairs}
            for _ in range(2):
                g.compute(t)
            ms[pairs] = g.stage_ms()
        g.close()
    finally:
        tclib.tc_set_profiling(False)
    _say("light bitmap pairs", {k: (v["count_light_wave"], v["count_light_bitmap"]) for k, v in ms.items()})
    # no pivot has a million pairs: the wavefront launch has all of the work
    assert ms[1_000_000]["count_light_wave"] > 2 * ms[1_000_000]["count_light_bitmap"]
    assert ms[64]["count_light_bitmap"] > 2 * ms[64]["count_light_wave"]


# a limit between what the low and the middle pivot take: AUTO does without the
# core's matrix, then without the middle pivot, before it gives the limit's error
@pytest.mark.parametrize("name", ["whole", "clique_900"])
def test_counts_under_a_limit(tclib, name):
    src, dst, n = CORE_GRAPHS["whole"]() if name == "whole" else gg.clique(900)
    ref = native.o2_paper(src, dst, n)
    done = {"low": [], "auto": []}
    try:
        for part in range(2, 22, 2):
            for algo in done:
                tclib.tc_set_memory_limit(0)
                g = tclib.Graph.from_edges(src, dst, n)
                room = g.compute_bytes() * part // 20
                tclib.tc_trim_memory()
                tclib.tc_set_memory_limit(tclib.tc_memory_stats()["in_use"] + room)
                _say("counts under a limit", name, algo, part)
                try:
                    g.compute({"algorithm": tclib.TC_ALGO_LOW_PIVOT} if algo == "low" else None)
                    done[algo].append(part)
                except tclib.TCError as e:
                    assert e.status == tclib.TC_ERR_BUDGET
                tclib.tc_set_memory_limit(0)
                if done[algo] and done[algo][-1] == part:
                    r = g.results()
                    np.testing.assert_array_equal(r["support"], ref.sup)
                    np.testing.assert_array_equal(r["num"], ref.num)
                g.close()
    finally:
        tclib.tc_set_memory_limit(0)
        tclib.tc_trim_memory()
    assert 20 in done["auto"] and 20 in done["low"], done
    if ref.m < 600_000:  # there, whatever the low pivot fits into is enough
        assert set(done["low"]) <= set(done["auto"]), done
