"""The persistent loop of the fused launch (k_fused_graphs, tc_fused.hip) as
compiled for gfx950: the queue fetch and the barrier after it lie in one loop.

Thread 0 fetches the next graph and every thread waits at the barrier behind
it.  Where a way through the loop ended with a test of threadIdx.x == 0 and no
barrier after it (a graph with more than 65535 vertices, or offsets outside the
arrays), the compiler joined that test with the fetch's own one: the lanes other
than thread 0 went from there straight to the barrier, in a loop inside the
fetch's.  Thread 0 waits, masked off, for that inner loop to end; it cannot end,
as no lane in it fetches a graph, and the launch does not return.  Host code
only: the assembly is compiled and read, nothing runs on a GPU."""
import re
import subprocess

import pytest

from paper_2105_00110_amd import _build

BLOCKS = (256, 512, 1024)


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    try:
        cc = _build.hipcc()
    except RuntimeError:
        pytest.skip("needs hipcc")
    out = tmp_path_factory.mktemp("isa") / "tc_fused.s"
    subprocess.run([cc, *_build.HIPCC_FLAGS, "-I", _build.INCLUDE, "-I", _build.CSRC,
                    "--cuda-device-only", "-S", f"{_build.CSRC}/tc_fused.hip", "-o", str(out)],
                   check=True, capture_output=True, timeout=300)
    return out.read_text()


def instructions(asm, name):
    """(instruction, loop depth of its block) of the function."""
    body = asm[re.search(rf"^\S*{name}\S*:", asm, re.M).end():]
    body = body[:body.index(".Lfunc_end")]
    depth, out = 0, []
    for line in body.splitlines():
        code, _, note = line.partition(";")
        if re.match(r"\.LBB\d+_\d+:|\s*$", code):  # a block starts, or its notes go on
            if code.strip() or "%bb." in note:
                depth = 0
            found = re.search(r"(?:in Loop: Header=\S+|This (?:Inner )?Loop Header:) Depth=(\d+)", note)
            if found:
                depth = int(found.group(1))
        else:
            out.append((code.strip(), depth))
    return out


@pytest.mark.parametrize("block", BLOCKS)
def test_queue_fetch_and_its_barrier_lie_in_one_loop(assembly, block):
    code = instructions(assembly, f"k_fused_graphsILi{block}E")
    fetch = [i for i, (c, _) in enumerate(code) if re.match(r"global_atomic_add\b.*\bsc0\b", c)]
    assert len(fetch) == 1  # the only atomic whose value is used
    barrier = next(d for c, d in code[fetch[0]:] if c == "s_barrier")
    assert code[fetch[0]][1] == 1 and barrier == 1, (code[fetch[0]], barrier)
