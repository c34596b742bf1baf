"""GPU: the fused batch entry point (tc_batch_fused), one persistent launch
for a whole batch of small graphs, against the oracle.

Every graph of every batch is compared with O2 (the appendix's Procedure 2
with counts, then Algorithm 2) run on that graph alone: canonical edges,
support, tri, triG, num and the bit pattern of tc.  Also: every schedule
(workgroup size, workgroups per compute unit, queue order) gives the same
bytes, the per-graph status codes of degenerate and invalid graphs, and
replays of the launch captured in a graph.
"""
import concurrent.futures as cf

import numpy as np
import pytest

from oracle import native
from paper_2105_00110_amd import graphgen as gg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _say(*a):
    print("[case]", *a, flush=True)


def concat(graphs):
    """(src, dst, pair_off, vtx_off) of a list of (src, dst, n) with local ids."""
    src = np.concatenate([np.asarray(g[0], np.int32) for g in graphs]) if graphs else np.zeros(0, np.int32)
    dst = np.concatenate([np.asarray(g[1], np.int32) for g in graphs]) if graphs else np.zeros(0, np.int32)
    po = np.zeros(len(graphs) + 1, np.int64)
    vo = np.zeros(len(graphs) + 1, np.int64)
    np.cumsum([len(g[0]) for g in graphs], out=po[1:])
    np.cumsum([g[2] for g in graphs], out=vo[1:])
    return src, dst, po, vo


def run_fused(tclib, graphs, order="largest_first", tuning=None):
    src, dst, po, vo = concat(graphs)
    ds = torch.from_numpy(src).cuda() if len(src) else torch.zeros(1, dtype=torch.int32, device="cuda")
    dd = torch.from_numpy(dst).cuda() if len(dst) else torch.zeros(1, dtype=torch.int32, device="cuda")
    fb = tclib.FusedBatch(ds, dd, po, vo, order=order, tuning=tuning)
    fb.run()
    torch.cuda.synchronize()
    res = fb.results()
    return fb, res


def oracle_each(graphs):
    with cf.ThreadPoolExecutor(max_workers=native.host_threads()) as ex:
        return list(ex.map(lambda g: native.o2_paper(g[0], g[1], g[2], nthreads=1), graphs))


def check_graph(one, ref):
    np.testing.assert_array_equal(one["eu"], ref.eu)
    np.testing.assert_array_equal(one["ev"], ref.ev)
    np.testing.assert_array_equal(one["support"], ref.sup)
    np.testing.assert_array_equal(one["tri"], ref.tri)
    assert int(one["triG"][0]) == ref.triG
    np.testing.assert_array_equal(one["num"], ref.num)
    np.testing.assert_array_equal(one["tc"].view(np.uint64), ref.tc.view(np.uint64))
    assert one["status"] == ref.status


def check_all(fb, res, graphs, refs=None):
    refs = refs or oracle_each(graphs)
    for g, ref in enumerate(refs):
        check_graph(fb.graph(res, g), ref)
    return refs


SMALL = {
    "K3": lambda: gg.clique(3),
    "K12": lambda: gg.clique(12),
    "K300": lambda: gg.clique(300),
    "bridge_4x6": lambda: gg.bridge_cliques(4, 6),
    "disjoint_5x4": lambda: gg.disjoint_cliques(5, 4),
    "chain_6x5": lambda: gg.clique_chain(6, 5)[:3],
    "ring_5x4": lambda: gg.clique_chain(5, 4, ring=True)[:3],
    "single_tri": lambda: gg.single_triangle_with_pendants((2, 3, 1)),
    "fig1b": lambda: gg.fig1b_four_k6_hub(),
    "ba_3000": lambda: gg.ba(3000, 8, seed=3),
    "rmat_s10": lambda: gg.rmat(10, 16, seed=2),
    "rmat_s14": lambda: gg.rmat(14, 16, seed=5),
}


def test_fused_er_config_alone_and_batched(tclib):
    graphs = [gg.er(2000, 0.005, seed=s) for s in range(1, 6)]
    refs = oracle_each(graphs)
    for s, (g, ref) in enumerate(zip(graphs, refs), start=1):
        _say("fused ER seed", s, "alone")
        fb, res = run_fused(tclib, [g])
        check_graph(fb.graph(res, 0), ref)
    _say("fused ER seeds 1-5 as one batch")
    fb, res = run_fused(tclib, graphs)
    check_all(fb, res, graphs, refs)


def test_fused_small_families(tclib):
    graphs = [f() for f in SMALL.values()]
    _say("fused families", list(SMALL))
    fb, res = run_fused(tclib, graphs)
    check_all(fb, res, graphs)


@pytest.mark.parametrize("tuning", [{"block": 256, "wg_per_cu": 1}, {"block": 512, "wg_per_cu": 2},
                                    {"block": 1024, "wg_per_cu": 1}, {"block": 512, "wg_per_cu": 8}])
def test_fused_every_schedule_same_bytes(tclib, tuning):
    graphs = [f() for f in SMALL.values()] + [gg.er(2000, 0.005, seed=s) for s in range(1, 3)]
    _say("fused schedule", tuning)
    fb, res = run_fused(tclib, graphs, tuning=tuning)
    check_all(fb, res, graphs)


def test_fused_queue_order_does_not_matter(tclib):
    graphs = [gg.er(300 + 50 * i, 0.05, seed=i) for i in range(40)]
    refs = oracle_each(graphs)
    rng = np.random.default_rng(7)
    for order in (None, "largest_first", rng.permutation(len(graphs)).astype(np.int32)):
        _say("fused order", order if order is None or isinstance(order, str) else "random")
        fb, res = run_fused(tclib, graphs, order=order)
        check_all(fb, res, graphs, refs)


def test_fused_random_tiny_graphs(tclib):
    rng = np.random.default_rng(123)
    graphs = []
    for i in range(300):
        n = int(rng.integers(1, 40))
        P = int(rng.integers(0, 3 * n + 1))
        graphs.append((rng.integers(0, n, P).astype(np.int32), rng.integers(0, n, P).astype(np.int32), n))
    _say("fused random tiny", len(graphs))
    fb, res = run_fused(tclib, graphs)
    check_all(fb, res, graphs)


def test_fused_degenerate_and_invalid_graphs(tclib):
    e0 = np.zeros(0, np.int32)
    big_n = 65535
    rng = np.random.default_rng(5)
    far = rng.integers(big_n - 300, big_n, 4000).astype(np.int32)
    star = (np.zeros(50, np.int32), np.arange(1, 51, dtype=np.int32), 51)
    dup = (np.array([0, 1, 1, 0, 2, 2, 0, 1, 2], np.int32),
           np.array([1, 0, 1, 1, 0, 2, 2, 2, 1], np.int32), 3)
    graphs = [
        (e0, e0, 0),                                              # empty, no vertices
        (np.zeros(3, np.int32), np.zeros(3, np.int32), 1),        # only self-loops
        (e0, e0, 17),                                             # isolated vertices only
        star,                                                     # triangle-free
        dup,                                                      # duplicates in both directions
        (far[:2000], far[2000:], big_n),                          # the largest n, ids at its top
        gg.clique(40),
    ]
    valid = len(graphs)
    bad_range = (np.array([0, 1, 5], np.int32), np.array([1, 2, 3], np.int32), 5)   # id 5 >= n
    negative = (np.array([0, -1], np.int32), np.array([1, 2], np.int32), 4)
    too_many = (np.array([0, 1, 65535], np.int32), np.array([1, 2, 0], np.int32), 65536)
    graphs += [bad_range, negative, too_many, gg.clique(5)]
    _say("fused degenerate / invalid")
    fb, res = run_fused(tclib, graphs)
    refs = oracle_each(graphs[:valid]) + [None, None, None] + oracle_each(graphs[-1:])
    for g in list(range(valid)) + [len(graphs) - 1]:
        check_graph(fb.graph(res, g), refs[g])
    for g, st in ((valid, tclib.TC_ERR_VERTEX_RANGE), (valid + 1, tclib.TC_ERR_VERTEX_RANGE),
                  (valid + 2, tclib.TC_ERR_UNSUPPORTED)):
        one = fb.graph(res, g)
        assert one["status"] == st, (g, one["status"])
        assert int(res["num_edges"][g]) == 0
        assert not one["tri"].any() and not one["num"].any() and not one["tc"].any()
    assert fb.graph(res, 0)["status"] == tclib.TC_TRIANGLE_FREE
    assert fb.graph(res, 3)["status"] == tclib.TC_TRIANGLE_FREE


@pytest.mark.parametrize("block", [256, 512, 1024])
def test_fused_rows_after_many_empty_ones(tclib, block):
    # ranks of isolated vertices come first, and vertices without higher
    # neighbours lie between the others: gaps of rows up to a wavefront and above
    rng = np.random.default_rng(17)
    graphs = [gg.clique(5)]
    for n, hubs in ((22000, 1), (30000, 70), (65535, 3)):
        leaves = np.arange(100, 100 + 90 * hubs, dtype=np.int32)
        far = rng.integers(n - 400, n, (2, 700)).astype(np.int32)
        graphs.append((np.concatenate([np.repeat(np.arange(hubs, dtype=np.int32), 90), far[0]]),
                       np.concatenate([leaves, far[1]]), n))
    graphs.append((np.array([3], np.int32), np.array([60000], np.int32), 65535))
    _say("fused rows after empty ones", block)
    fb, res = run_fused(tclib, graphs, tuning={"block": block, "wg_per_cu": 1})
    check_all(fb, res, graphs)


def test_fused_offsets_outside_the_arrays(tclib):
    # graphs 1 and 2 have pair offsets past the end, or decreasing: a status, and
    # the graphs after them are computed
    src, dst, po, vo = concat([gg.clique(3), gg.clique(3), gg.clique(3), gg.clique(5)])
    po[2] = 9999
    _say("fused offsets outside the arrays")
    fb = tclib.FusedBatch(torch.from_numpy(src).cuda(), torch.from_numpy(dst).cuda(), po, vo)
    fb.run()
    torch.cuda.synchronize()
    res = fb.results()
    assert list(res["status"][1:3]) == [tclib.TC_ERR_INVALID_ARG] * 2
    assert not res["num_edges"][1:3].any()
    for g, k in ((0, 3), (3, 5)):
        check_graph(fb.graph(res, g), native.o2_paper(*gg.clique(k), nthreads=1))


def test_fused_ba_batch_4096_every_graph(tclib):
    src, dst, po, vo = gg.batched_ba(4096, seed=4096)
    G = len(po) - 1
    graphs = [(src[po[i]:po[i + 1]], dst[po[i]:po[i + 1]], int(vo[i + 1] - vo[i])) for i in range(G)]
    _say("fused BA batch", G, "graphs", len(src), "pairs")
    fb = tclib.FusedBatch(torch.from_numpy(src).cuda(), torch.from_numpy(dst).cuda(), po, vo)
    fb.run()
    torch.cuda.synchronize()
    res = fb.results()
    _say("oracle O2 on every graph")
    check_all(fb, res, graphs)


def test_fused_graph_capture_replays(tclib):
    # the two launches captured once and replayed; between replays the
    # outputs are overwritten by eager work, and every replay must restore
    # them exactly
    graphs = [gg.er(2000, 0.005, seed=s) for s in range(1, 6)] + [gg.ba(3000, 8, seed=3)]
    src, dst, po, vo = concat(graphs)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        fb = tclib.FusedBatch(torch.from_numpy(src).cuda(), torch.from_numpy(dst).cuda(), po, vo,
                              stream=stream.cuda_stream)
        fb.run()
    torch.cuda.synchronize()
    eager = fb.results()
    refs = check_all(fb, eager, graphs)
    cg = torch.cuda.CUDAGraph()
    with torch.cuda.graph(cg, stream=stream):
        fb.run()
    torch.cuda.synchronize()
    for rep in range(4):
        for t in (fb.tri, fb.num, fb.support, fb.triG, fb.num_edges):
            t.fill_(-1)
        fb.tc.fill_(-1.0)
        fb.status.fill_(99)
        torch.cuda.synchronize()
        cg.replay()
        torch.cuda.synchronize()
        res = fb.results()
        _say("graph replay", rep)
        for k in ("num_edges", "tri", "triG", "num", "status"):
            np.testing.assert_array_equal(res[k], eager[k], err_msg=k)
        np.testing.assert_array_equal(res["tc"].view(np.uint64), eager["tc"].view(np.uint64))
        for g in range(len(graphs)):
            a, b = fb.graph(res, g), fb.graph(eager, g)
            for k in ("eu", "ev", "support"):
                np.testing.assert_array_equal(a[k], b[k], err_msg=k)
    check_all(fb, res, graphs, refs)
