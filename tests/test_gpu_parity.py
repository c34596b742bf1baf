"""GPU parity: libtc (through its C ABI) against the CPU oracle.

Integer outputs (edges, support, tri, triG, num) must be identical and the
float64 quotient bit-identical (the same single IEEE division on both
sides).  Inputs are seeded and shared; no expected value comes from the HIP
path.
"""
import numpy as np
import pytest

from oracle import native
from paper_2105_00110_amd import graphgen as gg
from tests import golden_io

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _say(*a):
    print("[case]", *a, flush=True)


def run_gpu(tc, src, dst, n, device=True, tuning=None):
    if device:
        s = torch.as_tensor(np.ascontiguousarray(src, np.int32)).cuda()
        d = torch.as_tensor(np.ascontiguousarray(dst, np.int32)).cuda()
        g = tc.Graph.from_edges(s, d, n)
    else:
        g = tc.Graph.from_edges(src, dst, n)
    st = g.compute(tuning)
    res = g.results()
    res["eu"], res["ev"] = g.edges()
    res["status"] = st
    res["m"] = g.m
    g.close()
    return res


def assert_parity(gpu, ref):
    assert gpu["m"] == ref.m
    np.testing.assert_array_equal(gpu["eu"], ref.eu)
    np.testing.assert_array_equal(gpu["ev"], ref.ev)
    np.testing.assert_array_equal(gpu["support"], ref.sup)
    np.testing.assert_array_equal(gpu["tri"], ref.tri)
    assert int(gpu["triG"][0]) == ref.triG
    np.testing.assert_array_equal(gpu["num"], ref.num)
    np.testing.assert_array_equal(gpu["tc"].view(np.uint64), ref.tc.view(np.uint64))
    assert gpu["status"] == ref.status


SMALL_FAMILIES = {
    "K3": lambda: gg.clique(3),
    "K12": lambda: gg.clique(12),
    "K200": lambda: gg.clique(200),
    "bridge_4x6": lambda: gg.bridge_cliques(4, 6),
    "disjoint_5x4": lambda: gg.disjoint_cliques(5, 4),
    "chain_6x5": lambda: gg.clique_chain(6, 5)[:3],
    "ring_5x4": lambda: gg.clique_chain(5, 4, ring=True)[:3],
    "single_tri": lambda: gg.single_triangle_with_pendants((2, 3, 1)),
    "er_2000": lambda: gg.er(2000, 0.005, seed=1),
    "ba_3000": lambda: gg.ba(3000, 8, seed=3),
    "rmat_s10": lambda: gg.rmat(10, 16, seed=2),
    "rmat_s14": lambda: gg.rmat(14, 16, seed=5),
}


@pytest.mark.parametrize("name", sorted(SMALL_FAMILIES))
def test_parity_small_families(tclib, name):
    src, dst, n = SMALL_FAMILIES[name]()
    ref = native.o1_definition(src, dst, n)
    _say(name, "n", n, "pairs", len(src), "device input")
    assert_parity(run_gpu(tclib, src, dst, n, device=True), ref)
    _say(name, "host input")
    assert_parity(run_gpu(tclib, src, dst, n, device=False), ref)


def test_device_results_on_another_stream(tclib):
    """Graph.results_device() of a handle whose stream is not the current
    one: the tensors are complete on the current stream even while the
    handle's stream is still busy (long fills are queued there before the
    copies), and equal the oracle's results."""
    src, dst, n = gg.rmat(14, 16, seed=5)
    ref = native.o1_definition(src, dst, n)
    side = torch.cuda.Stream()
    s = torch.as_tensor(np.ascontiguousarray(src, np.int32)).cuda()
    d = torch.as_tensor(np.ascontiguousarray(dst, np.int32)).cuda()
    side.wait_stream(torch.cuda.current_stream())
    g = tclib.Graph.from_edges(s, d, n, stream=side.cuda_stream)
    g.compute()
    busy = torch.empty(1 << 28, device="cuda")
    busy.record_stream(side)
    with torch.cuda.stream(side):
        for _ in range(20):
            busy.fill_(1.0)
    _say("device results on another stream, n", n)
    r = g.results_device()
    got = {k: v.cpu().numpy() for k, v in r.items()}  # on the current stream
    g.close()
    np.testing.assert_array_equal(got["support"][:ref.m].view(np.uint64), ref.sup)
    np.testing.assert_array_equal(got["tri"][:n].view(np.uint64), ref.tri)
    np.testing.assert_array_equal(got["num"][:n].view(np.uint64), ref.num)
    np.testing.assert_array_equal(got["tc"][:n].view(np.uint64), ref.tc.view(np.uint64))
    assert int(got["triG"][0]) == ref.triG


def test_device_pairs_from_another_stream(tclib):
    """Graph.from_edges of device pairs made on the current stream, with a
    handle on another stream: the build waits for the pairs (their copy is
    queued behind long fills), and the results equal the oracle's."""
    src, dst, n = gg.rmat(14, 16, seed=5)
    ref = native.o1_definition(src, dst, n)
    side = torch.cuda.Stream()
    busy = torch.empty(1 << 28, device="cuda")
    for _ in range(20):
        busy.fill_(1.0)
    s = torch.as_tensor(np.ascontiguousarray(src, np.int32)).cuda()
    d = torch.as_tensor(np.ascontiguousarray(dst, np.int32)).cuda()
    _say("device pairs from another stream, n", n)
    g = tclib.Graph.from_edges(s, d, n, stream=side.cuda_stream)
    st = g.compute()
    res = g.results()
    res["eu"], res["ev"] = g.edges()
    res["status"], res["m"] = st, g.m
    g.close()
    assert_parity(res, ref)


@pytest.mark.parametrize("fname", ["fig2_worked_example.txt", "fig1a.txt", "fig1c.txt",
                                   "fig1d.txt"])
def test_parity_paper_figures(tclib, fname):
    src, dst, n, _ = golden_io.load(fname)
    ref = native.o2_paper(src, dst, n)
    _say(fname)
    assert_parity(run_gpu(tclib, src, dst, n), ref)


@pytest.mark.parametrize("seed", [1, 2, 3, 4, 5])
def test_parity_er_config(tclib, seed):
    src, dst, n = gg.er(2000, 0.005, seed=seed)
    ref = native.o2_paper(src, dst, n)
    _say("ER G(2000,0.005) seed", seed)
    assert_parity(run_gpu(tclib, src, dst, n), ref)


@pytest.mark.parametrize("seed", range(12))
def test_parity_random_tiny(tclib, seed):
    rng = np.random.default_rng(100 + seed)
    n = int(rng.integers(1, 40))
    P = int(rng.integers(0, 200))
    src = rng.integers(0, n, P).astype(np.int32)
    dst = rng.integers(0, n, P).astype(np.int32)
    ref = native.o1_definition(src, dst, n)
    _say("tiny seed", seed, "n", n, "P", P)
    assert_parity(run_gpu(tclib, src, dst, n), ref)


_SCHEDULES = [
    {},
    {"light_max_dplus": 2, "heavy_block": 64, "light_block": 64, "lds_max_entries": 16384},
    {"light_max_dplus": 1024, "heavy_block": 1024, "light_block": 1024, "lds_max_entries": 1024},
    {"light_max_dplus": 16, "heavy_block": 512, "light_block": 128, "lds_max_entries": 1024},
    {"light_max_dplus": 37, "heavy_block": 192, "light_block": 320, "lds_max_entries": 2048},
]
# every schedule under both pivot choices (low = 1, middle = 2), and the
# middle pivot's workgroup lookup as hash only, as a small bitmap (pivots
# spanning more than 8192 ranks fall back to the hash) and as a large one
TUNINGS = [None] + [dict(sc, algorithm=a) for a in (1, 2) for sc in _SCHEDULES] + [
    {"algorithm": 2, "bitmap_words": 0, "light_max_dplus": 2},
    {"algorithm": 2, "bitmap_words": 256, "light_max_dplus": 2, "item_pairs": 64},
    {"algorithm": 2, "bitmap_words": 8192, "light_max_dplus": 16, "heavy_block": 1024},
    {"algorithm": 2, "light_bitmap_pairs": 1, "light_max_dplus": 64, "bitmap_words": 256},
    {"algorithm": 2, "light_bitmap_pairs": 16},
]


@pytest.mark.parametrize("ti", range(len(TUNINGS)))
def test_every_schedule_gives_identical_bytes(tclib, ti):
    # heavy tail (R-MAT) plus a clique large enough for the huge-row path
    src, dst, n = gg.rmat(13, 16, seed=9)
    ks, kd, kn = gg.clique(700)
    src = np.concatenate([src, ks + n]).astype(np.int32)
    dst = np.concatenate([dst, kd + n]).astype(np.int32)
    n = n + kn
    ref = native.o1_definition(src, dst, n)
    _say("tuning", TUNINGS[ti])
    assert_parity(run_gpu(tclib, src, dst, n, tuning=TUNINGS[ti]), ref)


@pytest.mark.parametrize("algo", [1, 2])
def test_every_bin_runs(tclib, algo):
    # with an LDS limit of 1024 entries the clique's rows (699 higher
    # neighbours) are looked up in device memory; the work statistics show
    # that light, heavy and huge rows all ran, and the result is exact
    src, dst, n = gg.rmat(13, 16, seed=9)
    ks, kd, kn = gg.clique(700)
    src = np.concatenate([src, ks + n]).astype(np.int32)
    dst = np.concatenate([dst, kd + n]).astype(np.int32)
    n = n + kn
    ref = native.o1_definition(src, dst, n)
    tuning = {"algorithm": algo, "lds_max_entries": 1024, "light_max_dplus": 16}
    _say("bins, algorithm", algo)
    g = tclib.Graph.from_edges(torch.from_numpy(src).cuda(), torch.from_numpy(dst).cuda(), n)
    st = g.compute(tuning)
    ws = g.work_stats()
    res = g.results()
    res["eu"], res["ev"] = g.edges()
    res["status"] = st
    res["m"] = g.m
    g.close()
    assert ws["algorithm"] == algo
    for b in ("light", "heavy", "huge"):
        assert ws["rows_" + b] > 0 and ws["cand_" + b] > 0, b
    assert_parity(res, ref)


@pytest.mark.parametrize("algo", [1, 2])
def test_launch_times_and_heavy_16_statistics(tclib, algo):
    # the middle pivot's count launches are timed one by one inside their
    # stages, and the work statistics of the 16-bit workgroup launch are a
    # part of the heavy bin's (all of it when n <= 2^16); the low pivot
    # reports no such launches
    src, dst, n = gg.rmat(16, 16, seed=16)
    tuning = {"algorithm": algo, "light_max_dplus": 64}
    tclib.tc_set_profiling(True)
    try:
        g = tclib.Graph.from_edges(src, dst, n)
        g.compute(tuning)
        ms = g.stage_ms()
        ws = g.work_stats()
        g.close()
    finally:
        tclib.tc_set_profiling(False)
    _say("launch times", algo, {k: round(v, 3) for k, v in ms.items()})
    sub = ms["count_light_groups"] + ms["count_light_wave"] + ms["count_light_bitmap"]
    if algo == 1:
        assert sub == 0.0 and ms["count_heavy_bitmap16"] == 0.0
        assert ws["cand_heavy_16"] == ws["edges_heavy_16"] == ws["rows_heavy_16"] == 0
        return
    assert abs(sub - ms["count_light"]) <= 0.02 + 0.02 * ms["count_light"]
    assert 0.0 < ms["count_heavy_bitmap16"] <= ms["count_heavy"] + 0.02
    # n = 2^16: every pivot is among the top 2^16 ranks
    assert ws["rows_heavy"] > 0
    assert (ws["cand_heavy_16"], ws["edges_heavy_16"], ws["rows_heavy_16"]) == \
        (ws["cand_heavy"], ws["edges_heavy"], ws["rows_heavy"])


@pytest.mark.parametrize("n", [65536, 65537, 70000])
def test_sixteen_bit_candidates_at_the_base(tclib, n):
    # the middle pivot reads the candidates of pivots among the top 2^16
    # ranks as 16-bit entries: at n = 2^16 every pivot does, at 2^16 + 1 all
    # but rank 0, at 70000 the lowest 4464 ranks do not (BA: every vertex
    # has degree >= 8, so ranks span all of n)
    src, dst, n_ba = gg.ba(n, 8, seed=n)
    assert n_ba == n
    ref = native.o1_definition(src, dst, n)
    for tuning in ({"algorithm": 2}, {"algorithm": 2, "light_max_dplus": 16}):
        _say("16-bit base, n", n, "tuning", tuning)
        assert_parity(run_gpu(tclib, src, dst, n, tuning=tuning), ref)


def test_sixteen_bit_candidates_both_sides_in_one_launch(tclib):
    # ER at average degree 64 over 70000 vertices: even the lowest ranks
    # have rows of about 50 entries, so with light rows of at most 16
    # entries the workgroup launch holds pivots below and above the 16-bit
    # base, under the bitmap and under the hash
    n = 70000
    src, dst, _ = gg.er(n, 64.0 / n, seed=7)
    ref = native.o1_definition(src, dst, n)
    for tuning in ({"algorithm": 2, "light_max_dplus": 16},
                   {"algorithm": 2, "light_max_dplus": 16, "bitmap_words": 0}):
        _say("16-bit base, ER 70000, tuning", tuning)
        assert_parity(run_gpu(tclib, src, dst, n, tuning=tuning), ref)


@pytest.fixture(scope="module")
def rmat_s20():
    src, dst, n = gg.rmat(20, 16, seed=20)
    _say("R-MAT s20 oracle")
    return src, dst, n, native.o1_definition(src, dst, n)


@pytest.mark.parametrize("tuning_name", [None, "rmat_s24_ef16", "batched_ba4096"])
def test_rmat_s20_full_parity(tclib, rmat_s20, tuning_name):
    # library defaults, and the stored schedules the benchmark times on the
    # scale-24 graph and on the batch, all against the full definition
    from paper_2105_00110_amd import autotune
    src, dst, n, ref = rmat_s20
    tuning = autotune.load(tuning_name) if tuning_name else None
    _say("R-MAT s20 gpu, tuning", tuning_name, tuning)
    assert_parity(run_gpu(tclib, src, dst, n, tuning=tuning), ref)


def test_determinism_two_runs(tclib):
    src, dst, n = gg.rmat(16, 16, seed=3)
    _say("determinism s16")
    a = run_gpu(tclib, src, dst, n)
    b = run_gpu(tclib, src, dst, n)
    for k in ("support", "tri", "num", "triG", "eu", "ev"):
        np.testing.assert_array_equal(a[k], b[k])
    np.testing.assert_array_equal(a["tc"].view(np.uint64), b["tc"].view(np.uint64))


def test_from_csr_matches_edges(tclib):
    src, dst, n = gg.rmat(12, 16, seed=4)
    ref = native.o2_paper(src, dst, n)
    # a one-sided CSR holding every input pair once, duplicates included
    order = np.lexsort((dst, src))
    s, d = src[order], dst[order]
    rp = np.zeros(n + 1, np.int64)
    np.add.at(rp, s + 1, 1)
    rp = np.cumsum(rp)
    _say("from_csr host")
    g = tclib.Graph.from_csr(rp, d, n)
    st = g.compute()
    res = g.results()
    res["eu"], res["ev"] = g.edges()
    res["status"], res["m"] = st, g.m
    g.close()
    assert_parity(res, ref)
    _say("from_csr device")
    g = tclib.Graph.from_csr(torch.as_tensor(rp).cuda(), torch.as_tensor(d).cuda(), n)
    st = g.compute()
    res = g.results()
    res["eu"], res["ev"] = g.edges()
    res["status"], res["m"] = st, g.m
    g.close()
    assert_parity(res, ref)


def _csr(rows, cols, n):
    order = np.lexsort((cols, rows))
    r, c = rows[order], cols[order]
    rp = np.zeros(n + 1, np.int64)
    np.add.at(rp, r + 1, 1)
    return np.cumsum(rp), np.ascontiguousarray(c, np.int32)


@pytest.mark.parametrize("scale", [12, 16])
def test_from_simple_sorted_csr(tclib, scale):
    # the fast path of tc_graph_from_csr for a CSR stated to be simple and
    # sorted: the symmetric CSR of the oracle's canonical edges, and its
    # upper triangle alone, give the oracle's results; on the host and on
    # the device
    src, dst, n = gg.rmat(scale, 16, seed=6)
    ref = native.o2_paper(src, dst, n)
    sym = _csr(np.concatenate([ref.eu, ref.ev]), np.concatenate([ref.ev, ref.eu]), n)
    upper = _csr(ref.eu, ref.ev, n)
    for name, (rp, col) in (("symmetric", sym), ("upper", upper)):
        for dev in (False, True):
            _say("simple sorted CSR", name, "device" if dev else "host", "scale", scale)
            if dev:
                g = tclib.Graph.from_csr(torch.as_tensor(rp).cuda(), torch.as_tensor(col).cuda(), n,
                                         assume_simple_sorted=True)
            else:
                g = tclib.Graph.from_csr(rp, col, n, assume_simple_sorted=True)
            st = g.compute()
            res = g.results()
            res["eu"], res["ev"] = g.edges()
            res["status"], res["m"] = st, g.m
            g.close()
            assert_parity(res, ref)


def test_simple_sorted_csr_violations_are_refused(tclib):
    # rows not increasing, a self-loop, a duplicate, an id out of range:
    # with the simple-sorted statement each is refused, without it each is
    # normalised like any pair list
    n = 6
    good_rows = np.array([0, 0, 1, 2, 3], np.int32)
    good_cols = np.array([1, 2, 2, 3, 4], np.int32)
    rp5 = np.array([0, 2, 3, 4, 5, 5, 5], np.int64)  # rows of 2, 1, 1, 1 entries, then empty
    bad = {
        "unsorted": (rp5, np.array([2, 1, 2, 3, 4], np.int32)),
        "loop": (rp5, np.array([1, 2, 1, 3, 4], np.int32)),
        "duplicate": (rp5, np.array([1, 1, 2, 3, 4], np.int32)),
        "range": (rp5, np.array([1, 2, 2, 3, 9], np.int32)),
    }
    rp, col = _csr(good_rows, good_cols, n)
    g = tclib.Graph.from_csr(rp, col, n, assume_simple_sorted=True)
    g.close()
    for name, (rp, col) in bad.items():
        _say("simple sorted CSR violation", name)
        with pytest.raises(tclib.TCError) as ei:
            tclib.Graph.from_csr(rp, col, n, assume_simple_sorted=True)
        assert ei.value.status == tclib.TC_ERR_INVALID_ARG


def test_degenerate_inputs(tclib):
    e = np.zeros(0, np.int32)
    _say("empty n=0")
    r = run_gpu(tclib, e, e, 0, device=False)
    assert r["m"] == 0 and r["status"] == tclib.TC_TRIANGLE_FREE
    _say("empty n=5")
    r = run_gpu(tclib, e, e, 5, device=False)
    assert r["m"] == 0 and np.all(r["tc"] == 0.0) and np.all(r["tri"] == 0)
    _say("triangle-free path")
    src = np.array([0, 1, 2, 3], np.int32)
    dst = np.array([1, 2, 3, 4], np.int32)
    r = run_gpu(tclib, src, dst, 6)
    assert r["status"] == tclib.TC_TRIANGLE_FREE and np.all(r["tc"] == 0.0)
    _say("only loops")
    r = run_gpu(tclib, np.array([2, 2], np.int32), np.array([2, 2], np.int32), 3)
    assert r["m"] == 0


def test_errors(tclib):
    src = np.array([0, 7], np.int32)
    dst = np.array([1, 2], np.int32)
    _say("vertex range host")
    with pytest.raises(tclib.TCError) as ei:
        tclib.Graph.from_edges(src, dst, 5)
    assert ei.value.status == tclib.TC_ERR_VERTEX_RANGE
    _say("vertex range device")
    with pytest.raises(tclib.TCError) as ei:
        tclib.Graph.from_edges(torch.as_tensor(src).cuda(), torch.as_tensor(dst).cuda(), 5)
    assert ei.value.status == tclib.TC_ERR_VERTEX_RANGE
    neg = np.array([-1], np.int32)
    with pytest.raises(tclib.TCError):
        tclib.Graph.from_edges(neg, np.array([0], np.int32), 5)
    _say("results before compute")
    g = tclib.Graph.from_edges(np.array([0], np.int32), np.array([1], np.int32), 2)
    with pytest.raises(tclib.TCError) as ei:
        g.results()
    assert ei.value.status == tclib.TC_ERR_NOT_COMPUTED
    with pytest.raises(tclib.TCError):
        g.compute({"light_max_dplus": 1})
    g.close()


def test_top_k_ranking(tclib):
    src, dst, n = gg.ba(5000, 5, seed=12)
    ref = native.o2_paper(src, dst, n)
    order = np.lexsort((np.arange(n), -ref.tc))
    _say("top-k")
    g = tclib.Graph.from_edges(src, dst, n)
    g.compute()
    verts, vals = g.top_k(50)
    np.testing.assert_array_equal(verts, order[:50])
    np.testing.assert_array_equal(vals.view(np.uint64), ref.tc[order[:50]].view(np.uint64))
    verts, _ = g.top_k(n + 10)
    np.testing.assert_array_equal(verts, order)
    g.close()


@pytest.mark.parametrize("algo", [0, 1, 2])
def test_batch_equals_single(tclib, algo):
    # about 80 graphs and 86 k vertices in all: under the middle pivot the
    # batch's top 2^16 ranks (the 16-bit candidates) span many graphs
    ns, ms = gg.batched_ba_sizes(80, seed=77, n_hi=5000)
    src, dst, po, vo = gg.batched_ba(ns=ns, ms=ms, seed=77)
    _say("batch of", len(ns), "vertices", int(vo[-1]), "algorithm", algo)
    g = tclib.Graph.batch(src, dst, po, vo)
    g.compute({"algorithm": algo})
    res = g.results()
    eu, ev = g.edges()
    eoff = g.edge_offsets()
    g.close()
    for gi in range(len(ns)):
        s, d = src[po[gi]:po[gi + 1]], dst[po[gi]:po[gi + 1]]
        ref = native.o2_paper(s, d, int(ns[gi]), nthreads=2)
        a, b = vo[gi], vo[gi + 1]
        e0, e1 = eoff[gi], eoff[gi + 1]
        np.testing.assert_array_equal(eu[e0:e1] - a, ref.eu)
        np.testing.assert_array_equal(ev[e0:e1] - a, ref.ev)
        np.testing.assert_array_equal(res["support"][e0:e1], ref.sup)
        np.testing.assert_array_equal(res["tri"][a:b], ref.tri)
        assert int(res["triG"][gi]) == ref.triG
        np.testing.assert_array_equal(res["num"][a:b], ref.num)
        np.testing.assert_array_equal(res["tc"][a:b].view(np.uint64), ref.tc.view(np.uint64))


def test_sort_based_orientation_path(tclib, monkeypatch):
    # rows with more higher-ordered neighbours than the LDS limit are
    # oriented by a global sort; lower the limit to run that path here
    monkeypatch.setenv("TC_ORIENT_SEG_MAX", "8")
    src, dst, n = gg.rmat(12, 16, seed=31)
    ks, kd, kn = gg.clique(60)
    src = np.concatenate([src, ks + n]).astype(np.int32)
    dst = np.concatenate([dst, kd + n]).astype(np.int32)
    n = n + kn
    ref = native.o1_definition(src, dst, n)
    for t in (None, {"algorithm": 1}, {"algorithm": 2}):
        _say("sort-based orientation, tuning", t)
        assert_parity(run_gpu(tclib, src, dst, n, tuning=t), ref)


# ---------------------------------------------------------------------------
# Algorithm 3 (algebraic numerator) as a second device path
# ---------------------------------------------------------------------------
ALG_CASES = {
    "K12": lambda: gg.clique(12),
    "bridge_4x6": lambda: gg.bridge_cliques(4, 6),
    "ring_5x4": lambda: gg.clique_chain(5, 4, ring=True)[:3],
    "single_tri": lambda: gg.single_triangle_with_pendants((2, 3, 1)),
    "er_2000": lambda: gg.er(2000, 0.005, seed=3),
    "rmat_s11": lambda: gg.rmat(11, 16, seed=5),
}


@pytest.mark.parametrize("name", list(ALG_CASES))
def test_algebraic_numerator_matches_oracle(tclib, name):
    from oracle import algebraic
    src, dst, n = ALG_CASES[name]()
    _say("algebraic numerator", name, "n", n, "pairs", len(src))
    g = tclib.Graph.from_edges(torch.as_tensor(np.ascontiguousarray(src, np.int32)).cuda(),
                               torch.as_tensor(np.ascontiguousarray(dst, np.int32)).cuda(), n)
    g.compute()
    alg = g.numerator_algebraic()
    num = g.results()["num"]
    g.close()
    np.testing.assert_array_equal(alg, num)
    ref = native.o1_definition(src, dst, n)
    np.testing.assert_array_equal(alg, ref.num)
    if n <= 2500:  # the dense algebraic oracle (Proposition 2 in float64)
        np.testing.assert_array_equal(alg, algebraic.algebraic(src, dst, n).num)


def test_algebraic_numerator_rmat_s20_and_batch(tclib):
    src, dst, n = gg.rmat(20, 16, seed=20)
    _say("algebraic numerator R-MAT s20")
    g = tclib.Graph.from_edges(torch.from_numpy(src).cuda(), torch.from_numpy(dst).cuda(), n)
    g.compute()
    np.testing.assert_array_equal(g.numerator_algebraic(), g.results()["num"])
    g.close()
    s2, d2, po, vo = gg.batched_ba(64, seed=77)
    _say("algebraic numerator, batch of 64 BA graphs")
    b = tclib.Graph.batch(s2, d2, po, vo)
    b.compute()
    np.testing.assert_array_equal(b.numerator_algebraic(), b.results()["num"])
    b.close()


def test_algebraic_numerator_before_compute(tclib):
    g = tclib.Graph.from_edges(*gg.clique(5)[:2], 5)
    with pytest.raises(tclib.TCError):
        g.numerator_algebraic()
    g.close()


def test_big_clique_fold_two_stripe_groups(tclib):
    # K_2100: every row of the orientation up to 2099 entries, so the fold
    # of the largest rows spans two groups of 64 column stripes; pinned by
    # Observation 1's closed forms (sup = k-2, tri = C(k-1,2), tc = 1)
    k = 2100
    src, dst, n = gg.clique(k)
    _say("K2100 closed forms")
    g = tclib.Graph.from_edges(torch.from_numpy(np.ascontiguousarray(src, np.int32)).cuda(),
                               torch.from_numpy(np.ascontiguousarray(dst, np.int32)).cuda(), n)
    g.compute()
    r = g.results()
    g.close()
    assert r["support"].shape[0] == k * (k - 1) // 2
    assert np.all(r["support"] == k - 2)
    assert np.all(r["tri"] == (k - 1) * (k - 2) // 2)
    assert int(r["triG"][0]) == k * (k - 1) * (k - 2) // 6
    assert np.all(r["tc"] == 1.0)


def test_fold_64bit_offsets_path(tclib, monkeypatch):
    # rows of 32768 entries and more fold with 64-bit offsets inside their
    # bit matrix; lower that switch so the path runs on a small graph: every
    # fold row through it (0), and rows from 100 entries up (both kernels in
    # one compute)
    src, dst, n = gg.rmat(13, 16, seed=41)
    ks, kd, kn = gg.clique(300)
    src = np.concatenate([src, ks + n]).astype(np.int32)
    dst = np.concatenate([dst, kd + n]).astype(np.int32)
    n = n + kn
    ref = native.o1_definition(src, dst, n)
    for lim in ("0", "100"):
        monkeypatch.setenv("TC_FOLD_I32_MAX", lim)
        _say("fold with 64-bit offsets from", lim, "entries")
        assert_parity(run_gpu(tclib, src, dst, n, tuning={"algorithm": 2}), ref)


def test_auto_pivot_choice(tclib):
    # TC_ALGO_AUTO: the low pivot for small graphs and for flat ones (all
    # oriented rows under 32 entries) below 3 M edges, the middle pivot from
    # 600000 edges up on skewed graphs; the work statistics report the form
    # that ran
    cases = [(gg.er(2000, 0.005, seed=1), tclib.TC_ALGO_LOW_PIVOT),
             (gg.er(200000, 16.0 / 200000, seed=3), tclib.TC_ALGO_LOW_PIVOT),
             (gg.rmat(17, 16, seed=17), tclib.TC_ALGO_MID_PIVOT)]
    for (src, dst, n), want in cases:
        g = tclib.Graph.from_edges(torch.from_numpy(src).cuda(), torch.from_numpy(dst).cuda(), n)
        g.compute()
        _say("auto pivot, m", g.m)
        assert g.work_stats()["algorithm"] == want
        g.close()


def test_cached_memory_across_streams_and_trim(tclib):
    # blocks freed on one stream are reused on another only after that
    # stream's work on them is done; trimming returns them; results stay exact
    src, dst, n = gg.rmat(15, 16, seed=15)
    ref = native.o1_definition(src, dst, n)
    ds, dd = torch.from_numpy(src).cuda(), torch.from_numpy(dst).cuda()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for rep in range(4):
        st = streams[rep % 2]
        with torch.cuda.stream(st):
            g = tclib.Graph.from_edges(ds, dd, n, stream=st.cuda_stream)
            g.compute({"algorithm": 2})
            r = g.results()
            r["eu"], r["ev"] = g.edges()
            r["status"], r["m"] = g.status, g.m
            g.close()
        assert_parity(r, ref)
        if rep == 2:
            tclib.tc_trim_memory()


def test_device_results_into_pinned_memory(tclib):
    # buffers that the device reaches but that are not its own memory take copies
    src, dst, n = gg.ba(5000, 7, seed=6)
    ref = native.o2_paper(src, dst, n)
    g = tclib.Graph.from_edges(src, dst, n)
    g.compute()
    out = {k: torch.full((c,), -1, dtype=torch.int64, pin_memory=True)
           for k, c in (("tri", n), ("support", g.m), ("triG", 1), ("num", n))}
    out["tc"] = torch.full((n,), -1.0, dtype=torch.float64, pin_memory=True)
    _say("device results into pinned memory")
    tclib.tc_get_results(g.h, *(out[k].data_ptr() for k in ("tri", "support", "triG", "num", "tc")),
                         tclib.TC_MEM_DEVICE, g.stream)
    torch.cuda.synchronize()
    g.close()
    for k, want in (("tri", ref.tri), ("support", ref.sup), ("num", ref.num)):
        np.testing.assert_array_equal(out[k].numpy().view(np.uint64), want)
    assert int(out["triG"][0]) == ref.triG
    np.testing.assert_array_equal(out["tc"].numpy().view(np.uint64), ref.tc.view(np.uint64))
