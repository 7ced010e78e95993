"""The library's host-only rules, compiled for the CPU with its planner
(tests/plan_probe.cpp): index arithmetic that a kernel shares with them, and
plans at the edges of their ranges."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def P(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("plan") / "libplan_probe.so")
    src = [os.path.join(ROOT, "tests", "plan_probe.cpp"),
           os.path.join(ROOT, "paper_2109_07710_amd", "csrc", "plan.cpp")]
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-o", lib] + src, check=True)
    return ctypes.CDLL(lib)


@pytest.mark.parametrize("nsplit", [1, 2, 3, 14, 64, 123, 256])
def test_compacted_list_indices(P, nsplit):
    """Every list entry a split writes or fills lies in its own part of the
    list, whatever the live total: splits past the last block (also with a
    ragged last block), full lists, no live pixel.  The splits' ranks are the
    live pixels, each once and in order."""
    cap = P.probe_compact_list_cap()
    out = (ctypes.c_int32 * 6)()
    totals = sorted({t for b in (0, 1, 2, 5, nsplit - 1, nsplit, nsplit + 1, 7 * nsplit // 2, nsplit * cap // 64)
                     for t in range(64 * b - 65, 64 * b + 66) if 0 <= t <= nsplit * cap})
    for total in totals:
        ranks = blocks = 0
        for z in range(nsplit):
            P.probe_compact_share(total, nsplit, z, out)
            nblk, share, begin, end, first, last = out
            entries = (end - begin) * 64
            assert nblk == -(-total // 64) and 0 <= begin <= end <= nblk and end - begin <= share
            assert 0 <= last - first <= entries <= cap          # list[0, last - first) written, the rest filled
            assert first == last or (first == ranks and first == begin * 64)
            ranks += last - first
            blocks += end - begin
        assert ranks == total and blocks == nblk
