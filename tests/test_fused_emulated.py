"""The fused launch's kernel (k_fused_graphs with its three tiers, tc_fused.hip and
tc_small.h) compiled for the host with the CPU emulation of tests/emu (one thread
per lane, wavefront and workgroup barriers, AddressSanitizer, a workspace that
starts as garbage), every graph of a batch against the oracle and a status for
every refused one, at each workgroup size.  Host code only: no GPU."""
import pathlib
import shutil
import subprocess

import numpy as np
import pytest

from oracle import native
from paper_2105_00110_amd import graphgen as gg

ROOT = pathlib.Path(__file__).resolve().parents[1]
CSRC = ROOT / "paper_2105_00110_amd" / "csrc"
EMU = ROOT / "tests" / "emu"
VERTEX_RANGE, UNSUPPORTED = -2, -8

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.fixture(scope="module")
def programs(tmp_path_factory):
    """block -> the emulated kernel, compiled when first asked for"""
    work, made = tmp_path_factory.mktemp("fused"), {}
    src = (CSRC / "tc_fused.hip").read_text()
    shutil.copy(CSRC / "tc_small.h", work)  # out of its folder, whose tc_internal.h it would take
    (work / "fused_body.inc").write_text(src[:src.index("int cu_count() {")] + "}\n")

    def get(block):
        if block not in made:
            exe = work / f"fused_{block}"
            subprocess.run(["g++", "-std=c++20", "-O1", "-pthread", "-fsanitize=address", "-w",
                            f"-DEMU_BLOCK={block}", f"-I{EMU / 'fused'}", f"-I{EMU}", f"-I{work}",
                            f"-I{ROOT / 'include'}", str(EMU / "fused_check.cpp"),
                            str(EMU / "emu_rt.cpp"), "-o", str(exe)],
                           check=True, capture_output=True, text=True, timeout=300)
            made[block] = exe
        return made[block]
    return get


def run(exe, graphs):
    po = np.cumsum([0] + [len(g[0]) for g in graphs]).astype(np.int64)
    vo = np.cumsum([0] + [g[2] for g in graphs]).astype(np.int64)
    G, P, N = len(graphs), int(po[-1]), int(vo[-1])
    batch, out = exe.with_suffix(".in"), exe.with_suffix(".out")
    batch.write_bytes(np.array([G, P, N], np.int64).tobytes() + po.tobytes() + vo.tobytes()
                      + b"".join(np.concatenate([g[k] for g in graphs]).astype(np.int32).tobytes()
                                 for k in (0, 1)))
    r = subprocess.run([str(exe), str(batch), str(out)], capture_output=True, text=True, timeout=300,
                       env={"ASAN_OPTIONS": "detect_leaks=0"})
    assert r.returncode == 0, r.stderr[-3000:]
    data, at = out.read_bytes(), 0
    res = {}
    for key, n, dt in (("eu", P, np.int32), ("ev", P, np.int32), ("sup", P, np.uint64),
                       ("m", G, np.int64), ("tri", N, np.uint64), ("triG", G, np.uint64),
                       ("num", N, np.uint64), ("tc", N, np.float64), ("status", G, np.int32)):
        res[key] = np.frombuffer(data, dt, n, at)
        at += n * np.dtype(dt).itemsize
    return po, vo, res


def check(exe, graphs):
    po, vo, r = run(exe, graphs)
    for i, (src, dst, n) in enumerate(graphs):
        v = slice(vo[i], vo[i + 1])
        ids = np.concatenate([src, dst])
        bad = n > 65535 or (len(ids) and (ids.min() < 0 or ids.max() >= n))
        if bad:
            assert r["status"][i] == (UNSUPPORTED if n > 65535 else VERTEX_RANGE), i
            assert r["m"][i] == 0 and r["triG"][i] == 0
            assert not r["tri"][v].any() and not r["num"][v].any() and not r["tc"][v].any()
            continue
        ref = native.o2_paper(src, dst, n, nthreads=1)
        m = int(r["m"][i])
        e = slice(po[i], po[i] + m)
        assert m == ref.m and r["status"][i] == ref.status and int(r["triG"][i]) == ref.triG, i
        for key, got, want in (("eu", r["eu"][e], ref.eu), ("ev", r["ev"][e], ref.ev),
                               ("sup", r["sup"][e], ref.sup), ("tri", r["tri"][v], ref.tri),
                               ("num", r["num"][v], ref.num),
                               ("tc", r["tc"][v].view(np.uint64), ref.tc.view(np.uint64))):
            np.testing.assert_array_equal(got, want, err_msg=f"graph {i} {key}")


def pairs(n, P, seed, bad=False):
    rng = np.random.default_rng(seed)
    s, d = rng.integers(0, n, (2, P)).astype(np.int32)
    k = min(12, n, P)
    s[:k], d[:k] = np.arange(k), np.roll(np.arange(k), 1)
    if bad:
        s[P // 2] = n if seed % 2 else -1
    return s, d, n


def edges(n, m, seed):
    """m distinct edges"""
    rng = np.random.default_rng(seed)
    k = np.unique(rng.integers(0, n * n, 4 * m))
    k = np.unique(np.minimum(k // n, k % n) * n + np.maximum(k // n, k % n))
    k = rng.permutation(k[k // n < k % n])[:m]
    assert k.shape[0] == m
    return (k // n).astype(np.int32), (k % n).astype(np.int32), n


def degenerate():
    e0 = np.zeros(0, np.int32)
    far = np.random.default_rng(5).integers(65235, 65535, 4000).astype(np.int32)
    three = np.array([0, 1, 65535], np.int32), np.array([1, 2, 0], np.int32)
    return [
        (e0, e0, 0), (np.zeros(3, np.int32), np.zeros(3, np.int32), 1), (e0, e0, 17),
        (np.zeros(50, np.int32), np.arange(1, 51, dtype=np.int32), 51),
        (np.array([0, 1, 1, 0, 2, 2, 0, 1, 2], np.int32),
         np.array([1, 0, 1, 1, 0, 2, 2, 2, 1], np.int32), 3),
        (far[:2000], far[2000:], 65535), gg.clique(40),
        (np.array([0, 1, 5], np.int32), np.array([1, 2, 3], np.int32), 5),
        (np.array([0, -1], np.int32), np.array([1, 2], np.int32), 4),
        (*three, 65536), gg.clique(5), (*three, 65535), (three[0][:2], three[1][:2], 65535),
    ]


@pytest.mark.parametrize("block", [256, 512, 1024])
def test_degenerate_and_invalid_graphs(programs, block):
    check(programs(block), degenerate())


# bytes of the arena that the merge's cache of the middle tier shares (Medium::BYTES)
CACHE_BYTES = {256: 41984, 512: 76800}


@pytest.mark.parametrize("block", [256, 512])
def test_edges_of_the_tiers(programs, block):
    """16 pairs and 4 vertices a thread in LDS; 21 vertices a thread with the rest
    in the workspace; above; the merge's cache full and one slot past it; a refused
    graph in each tier between computed ones"""
    b = block
    words = CACHE_BYTES[b] // 4 - 8
    check(programs(b), [
        pairs(4 * b, 16 * b, 1), pairs(4 * b, 16 * b + 1, 2), pairs(4 * b + 1, 16 * b - 1, 3),
        pairs(4 * b, 16 * b, 5, bad=True), pairs(6 * b, 24 * b, 4), pairs(6 * b, 24 * b + 1, 6),
        pairs(6 * b, 20 * b, 7, bad=True), pairs(21 * b, 70, 8), pairs(21 * b, 20 * b, 9),
        pairs(21 * b + 1, 20 * b, 10), pairs(21 * b + 1, 999, 12, bad=True), gg.clique(130),
        edges(5 * b, words - 5 * b, 11), edges(5 * b, words - 5 * b + 1, 13), gg.clique(3),
    ])
