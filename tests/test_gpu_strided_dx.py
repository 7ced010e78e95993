"""GPU parity of the strided data gradient's pixel classes against the fp64
oracle: strides equal and unequal per axis, classes without a tap (1x1,
stride 2), without a pixel (one row or column), more residues than classes are
kept for (5 x 5: every tap of every pixel), pads past the filter, filters
smaller than the stride; tilings split and not; every pixel live (the class tiling) and whole pixels dead (the
live lists).
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2109_07710_amd as cb
from parity import check_values, tol_for

pytestmark = pytest.mark.gpu

CASES = [
    # N, C, H, W, K, R, S, stride, pad, dtype
    (2, 64, 13, 11, 40, 3, 3, (2, 2), (1, 1), "bf16"),      # few tiles of few steps
    (2, 64, 13, 11, 520, 3, 3, (2, 2), (1, 1), "bf16"),     # few tiles of many: split reduction
    (3, 72, 9, 10, 136, 1, 1, (2, 2), (0, 0), "bf16"),      # three classes of four have no tap
    (3, 256, 27, 27, 1024, 1, 1, (2, 2), (0, 0), "bf16"),   # their tiles whole beside split ones
    (1, 64, 1, 40, 128, 1, 1, (2, 2), (1, 0), "bf16"),      # no pixel has a tap
    (7, 208, 41, 39, 32, 1, 1, (2, 2), (0, 0), "bf16"),     # one step a tile, one round: no classes
    (2, 64, 21, 19, 40, 1, 1, (2, 1), (0, 0), "bf16"),      # one step, 64-channel tiles: two classes
    (3, 72, 23, 20, 100, 1, 1, (2, 2), (0, 0), "f32"),
    (1, 128, 1, 37, 64, 1, 3, (2, 3), (0, 1), "bf16"),      # one row: classes without a pixel
    (2, 256, 12, 15, 64, 5, 4, (3, 1), (4, 0), "bf16"),     # nine taps at most, stride 1 along one axis
    (2, 32, 17, 9, 32, 2, 2, (4, 4), (1, 3), "bf16"),       # filter smaller than the stride, pad past the filter
    (2, 64, 16, 16, 24, 3, 3, (5, 5), (1, 1), "bf16"),      # 25 residues: every tap of every pixel
    (5, 128, 130, 94, 16, 3, 3, (2, 2), (1, 1), "bf16"),    # 144 tiles of 448 rows
    (9, 256, 96, 80, 8, 3, 3, (2, 2), (1, 1), "bf16"),      # 312 tiles of 224 rows
    (3, 64, 224, 200, 8, 3, 3, (2, 2), (1, 1), "bf16"),     # 264 tiles of 512 rows
    (2, 36, 21, 18, 20, 3, 3, (2, 2), (1, 1), "f32"),
    (4, 128, 120, 118, 12, 3, 3, (2, 2), (1, 1), "f32"),    # 128 full tiles: split in two
]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cb.lib()


def _rows(desc, st, pd, dt, live):
    """GEMM rows of the skipping call with `live` pixels per channel group: all
    of them where the class tiling's steps (eight more a tile) are fewer than
    the live lists', which walk every tap.  No classes past 16 residues, and none
    where a round of tiles of over 64 channels takes one step each."""
    N, C, H, W, K, R, S = desc.N, desc.C, desc.H, desc.W, desc.K, desc.R, desc.S
    bm, bn, rows = cb.cbw_data_tiling(desc)
    kc, groups, npix = -(-K // (64 if dt == "bf16" else 32)), -(-C // bm), N * H * W
    cost = 0
    for a in range(st[0]):
        for b in range(st[1]):
            pix = N * sum((h + pd[0]) % st[0] == a for h in range(H)) * sum((w + pd[1]) % st[1] == b for w in range(W))
            cost += -(-pix // bn) * groups * (len(range(a, R, st[0])) * len(range(b, S, st[1])) * kc + 8)
    listed = sum(-(-n // bn) for n in live)
    single = R * S * kc == 1 and bm > 64 and -(-npix // rows) * groups <= 256
    classes = st[0] * st[1] <= 16 and not single and listed * (R * S * kc + 8) > cost
    return groups * npix if classes or min(live) == npix else sum(live)


@pytest.mark.parametrize("dead", [False, True, "few", "most"], ids=["live", "dead_pixels", "few_dead", "most_dead"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "%s_N%dC%dK%d_%dx%d_f%dx%d_s%dx%d" % (
    c[9], c[0], c[1], c[4], c[2], c[3], c[5], c[6], *c[7]))
def test_strided_dx(case, dead):
    N, C, H, W, K, R, S, st, pd, dt = case
    print("\n[case] strided dX %s dead=%s" % (case, dead), flush=True)
    rng = np.random.default_rng([210907710, 91, N, C, H, W, K])
    td = torch.bfloat16 if dt == "bf16" else torch.float32
    desc = cb.ConvDesc.make(N, C, H, W, K, R, S, st, pd, dtype=dt)
    x = np.maximum(rng.standard_normal((N, H, W, C), dtype=np.float32), 0.0)
    if dead:
        x[rng.random((N, H, W)) < {True: 0.5, "few": 0.01, "most": 0.9}[dead]] = 0.0
    else:
        x[..., 0] += 0.5
    x = torch.from_numpy(x).to(td)
    w = torch.from_numpy(rng.standard_normal((K, R, S, C), dtype=np.float32)).to(td)
    dy = torch.from_numpy(rng.standard_normal((N, desc.P, desc.Q, K), dtype=np.float32)).to(td)
    dx = {k: torch.full((N, H, W, C), float("nan"), dtype=td, device="cuda") for k in ("dense", "select", "masked")}
    xm = torch.zeros(cb.cbw_mask_words(desc), dtype=torch.int32, device="cuda")
    cb.cbw_relu_mask_pack(desc, x.cuda(), xm)
    ws = cb.workspace(desc, cb.CBW_OP_BWD_DATA_MASKED)
    cb.conv_bwd_data(desc, dy.cuda(), w.cuda(), dx["dense"], ws)
    cb.conv_bwd_data_masked(desc, dy.cuda(), w.cuda(), xm, dx["select"], ws, cb.CBW_FLAG_NO_SKIP)
    cb.conv_bwd_data_masked(desc, dy.cuda(), w.cuda(), xm, dx["masked"], ws)
    stats = cb.cbw_read_stats(desc, cb.CBW_OP_BWD_DATA_MASKED, ws)
    lists = [cb.cbw_read_live_lists(desc, ws, g) for g in range(-(-C // cb.cbw_read_live_lists(desc, ws, 0)[1]))]
    torch.cuda.synchronize()
    for g, (got, width) in enumerate(lists):
        live = (x[..., g * width:(g + 1) * width] > 0).any(dim=3).flatten().nonzero().flatten()
        assert np.array_equal(np.asarray(got), live.numpy())
    # the rows that were computed: every pixel's where the classes ran
    assert stats.rows_total == len(lists) * N * H * W
    assert stats.rows_live == _rows(desc, st, pd, dt, [len(got) for got, _ in lists])
    dy64 = oracle.nhwc_to_nchw(dy.double().numpy())
    w64 = oracle.krsc_to_kcrs(w.double().numpy())
    ref, ab, nt = oracle.conv_bwd_data(dy64, w64, (H, W), st, pd, with_bound=True)
    mask = oracle.relu_mask(oracle.nhwc_to_nchw(x.double().numpy()))
    for k, g in dx.items():
        m = 1 if k == "dense" else mask
        out = oracle.nhwc_to_nchw(g.float().cpu().double().numpy())
        check_values(out, ref * m, ab * m, nt * m, tol_for(dt), dt == "bf16", "strided dX, " + k)
        if k != "dense":   # killed outputs are the +0.0 bit pattern
            bits = g.view(torch.int16 if dt == "bf16" else torch.int32).cpu().numpy()
            assert not (oracle.nchw_to_nhwc(~mask) & (bits != 0)).any()


@pytest.mark.parametrize("fill", [0, -1])
def test_one_workspace_live_and_dead(fill):
    """Calls with every pixel live, few dead (the classes), most dead (the lists)
    and the other way round over one workspace, whatever it held: each the
    result of a workspace of its own (a dead-pixel flag may be stale)."""
    N, C, H, W, K, R, S = 4, 256, 40, 38, 128, 3, 3
    print("\n[case] strided dX, one workspace filled with %d" % fill, flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(9)
    desc = cb.ConvDesc.make(N, C, H, W, K, R, S, 2, (1, 1))
    dy = torch.randn((N, desc.P, desc.Q, K), generator=g, device="cuda").bfloat16()
    w = torch.randn((K, R, S, C), generator=g, device="cuda").bfloat16()
    calls = []
    for dead in (0.0, 0.01, 0.95):
        x = torch.randn((N, H, W, C), generator=g, device="cuda").abs_() + 0.1
        x[torch.rand((N, H, W), generator=g, device="cuda") < dead] = 0.0
        xm = torch.zeros(cb.cbw_mask_words(desc), dtype=torch.int32, device="cuda")
        cb.cbw_relu_mask_pack(desc, x.bfloat16(), xm)
        dx = torch.full((N, H, W, C), float("nan"), dtype=torch.bfloat16, device="cuda")
        ws = cb.workspace(desc, cb.CBW_OP_BWD_DATA_MASKED).zero_()
        cb.conv_bwd_data_masked(desc, dy, w, xm, dx, ws)
        calls.append((xm, dx, cb.cbw_read_stats(desc, cb.CBW_OP_BWD_DATA_MASKED, ws).rows_live))
    assert calls[0][2] == calls[1][2] == N * H * W > 5 * calls[2][2]
    ws = cb.workspace(desc, cb.CBW_OP_BWD_DATA_MASKED)
    ws.fill_(255 if fill else 0) if ws.dtype == torch.uint8 else ws.fill_(fill)
    for i in (0, 2, 1, 0, 1, 2, 2, 0):
        xm, ref, rows = calls[i]
        dx = torch.full_like(ref, float("nan"))
        cb.conv_bwd_data_masked(desc, dy, w, xm, dx, ws)
        assert cb.cbw_read_stats(desc, cb.CBW_OP_BWD_DATA_MASKED, ws).rows_live == rows
        assert torch.equal(dx.view(torch.int16), ref.view(torch.int16)), "call %d" % i
