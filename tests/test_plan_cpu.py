"""The library's host-only rules, compiled for the CPU with its planner
(tests/plan_probe.cpp): index arithmetic that a kernel shares with them, and
plans at the edges of their ranges."""
import ctypes
import math
import os
import random
import subprocess

import pytest

import paper_2109_07710_amd as cb

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


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("layer", [
    # N, C, H, W, K, R, S, strides, pads
    (3, 256, 27, 27, 256, 1, 1, (2, 2), (0, 0)),
    (3, 256, 27, 27, 1024, 1, 1, (2, 2), (0, 0)),
    (26, 256, 32, 36, 512, 1, 1, (2, 2), (0, 0)),
    (4, 64, 112, 112, 512, 1, 1, (2, 2), (0, 0)),
    (2, 128, 30, 21, 264, 1, 3, (2, 2), (0, 1)),
    (2, 64, 20, 20, 128, 3, 3, (4, 4), (1, 1)),
    (8, 128, 28, 28, 256, 3, 3, (2, 2), (1, 1)),      # every class has a tap
    (1, 64, 1, 40, 128, 1, 1, (2, 2), (1, 0)),        # no pixel has one
], ids=lambda v: "N%d_%dx%d_C%d_K%d_f%dx%d" % (v[0], v[2], v[3], v[1], v[4], v[5], v[6]))
def test_tap_free_tiles_are_not_split(P, layer, dtype):
    """Strided data gradient: tiles of pixels that no filter tap reaches have no
    partials and take no part in the choice of the split; with them the items
    of a split tiling are at most one a CU.  bf16 splits only where the steps
    saved outweigh the partials: fewer ways, by the cost the planner states."""
    N, C, H, W, K, R, S, st, pd = layer
    d = cb.ConvDesc.make(N, C, H, W, K, R, S, st, pd, dtype=dtype)
    out = (ctypes.c_int64 * 7)()
    assert P.probe_data_plan(ctypes.byref(d), 0, out) == cb.CBW_OK
    bm, rows, groups, ptiles, ptaps, split, partial = out
    pixels = lambda size, s, pad, a: sum((h + pad) % s == a for h in range(size))  # noqa: E731
    tiles = [(-(-N * pixels(H, st[0], pd[0], a) * pixels(W, st[1], pd[1], b) // rows), a < R and b < S)
             for a in range(st[0]) for b in range(st[1])]
    taps, free = (groups * sum(t for t, has in tiles if has == h) for h in (True, False))
    assert (ptaps * groups, ptiles * groups) == (taps, taps + free)
    assert partial == (taps * split * rows * bm * 4 if split > 1 else 0)
    assert split == 1 or (taps and taps * split + free <= 256)
    if 0 < taps and 2 * (taps + free) <= 256:
        steps = -(-R // st[0]) * -(-S // st[1]) * -(-K // (64 if dtype == "bf16" else 32))
        most = min(16, steps, (256 - free) // taps)
        cost = lambda n: 1.1 * -(-steps // n) + (6.0 + rows * bm * 4e-6 * taps * n / 10.0 if n > 1 else 0.0)  # noqa: E731
        assert split == (most if dtype == "f32" else min(range(1, most + 1), key=cost))


def _cheapest_split(part, wgs, nchunks, max_split):
    """The fp32 weight gradient's cost model over every count of splits."""
    best, least = 1, None
    for ns in range(1, min(max_split, 768) + 1):
        per = -(-nchunks // ns)
        if -(-nchunks // per) != ns:
            continue
        w = -(-wgs * ns // 256)
        cost = 1.9 * w * ((per + 3) // 4) + 3.0 * ((w + 2) // 3) + part * ns
        if least is None or cost < least:
            best, least = ns, cost
    return best


def test_f32_weight_splits_are_the_cheapest(P):
    """The planner skips counts that cannot be the cheapest: its choice is the
    one of trying them all, for few and many workgroups, chunks and bytes."""
    rng = random.Random(5)
    log = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))  # noqa: E731
    for C, K, R in ((4, 4, 1), (16, 16, 3), (64, 128, 3), (512, 512, 3), (2048, 1024, 1)):
        d = cb.ConvDesc.make(1, C, 8, 8, K, R, R, 1, (R // 2, R // 2), dtype="f32")
        cases = [(log(1, 3000), n, max(1, n // 4)) for n in [1, 2, 3, 4, 5, 7, 8, 9, 63, 64, 65] + [log(1, 60000) for _ in range(300)]]
        flat = (ctypes.c_int64 * (3 * len(cases)))(*[v for c in cases for v in c])
        got = (ctypes.c_int32 * len(cases))()
        P.probe_f32_weight_splits(ctypes.byref(d), len(cases), flat, got)
        for c, ns in zip(cases, got):
            assert ns == _cheapest_split(K * R * R * C * 8 / 4e6, *c), (C, K, R, c)


@pytest.mark.parametrize("layer", [(2, 16, 16, 16, 3), (16, 128, 28, 128, 3), (8, 256, 28, 256, 3), (4, 64, 112, 64, 3),
                                   (100, 8, 63, 32, 1)], ids=str)
def test_f32_weight_plan(P, layer):
    N, C, H, K, R = layer
    d = cb.ConvDesc.make(N, C, H, H, K, R, R, 1, (R // 2, R // 2), dtype="f32")
    out = (ctypes.c_int64 * 3)()
    assert P.probe_f32_weight_plan(ctypes.byref(d), out) == cb.CBW_OK
    wgs, nchunks, nsplit = out
    assert nsplit == _cheapest_split(K * R * R * C * 8 / 4e6, wgs, nchunks, max(1, nchunks // 4))
