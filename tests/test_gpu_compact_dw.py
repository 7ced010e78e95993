"""GPU parity of the bf16 weight gradient over compacted pixels: dY footprints
that whole pixels share (most 64-pixel blocks hold a live pixel, few pixels are
live), against the fp64 oracle and the unskipped run.  The compaction applies
where a split has sixteen chunks or more, the live pixels of a k tile fit half
as many blocks as are live and every split saves four of them on average;
cases lie on both sides of these lines, with k tiles that differ, ragged last chunks,
packed taps, strides, every pixel dead, and more live pixels per split than
the list holds (the chunked path again).
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2109_07710_amd as cb
from parity import check_dw_regrouped, check_values, tol_for

pytestmark = pytest.mark.gpu

CASES = [
    # N, C, H, W, K, R, S, stride, pad, share of live pixels per k tile
    (36, 256, 20, 20, 512, 3, 3, 1, 1, (0.1, 0.1)),        # 17 chunks a split
    (36, 256, 20, 20, 512, 3, 3, 1, 1, (0.45, 0.02)),      # just under half, and few
    (36, 256, 20, 20, 512, 3, 3, 1, 1, (0.6, 0.6)),        # past half: chunks
    (30, 136, 17, 19, 520, 3, 3, 1, 1, (0.02, 1.0, 0.3)),  # three k tiles, ragged channels and last chunk
    (550, 48, 31, 29, 40, 3, 3, 2, 1, (0.2,)),             # packed taps, stride 2, 64-wide k tile
    (520, 320, 16, 16, 72, 1, 1, 1, 0, (0.01,)),
    (200, 256, 12, 12, 256, 3, 3, 1, 1, (0.0,)),           # nothing live
    # few chunks a split: live pixels are not recorded, live chunks are walked
    (6, 256, 20, 20, 256, 3, 3, 1, 1, (0.1,)),
    (6, 256, 20, 20, 256, 3, 3, 1, 1, (0.45,)),
    (6, 256, 20, 20, 256, 3, 3, 1, 1, (0.6,)),
    (5, 136, 17, 19, 520, 3, 3, 1, 1, (0.02, 1.0, 0.3)),
    (7, 48, 31, 29, 40, 3, 3, 2, 1, (0.2,)),           # packed taps, stride 2, 64-wide k tile
    (4, 320, 16, 16, 72, 1, 1, 1, 0, (0.01,)),
    (3, 256, 12, 12, 256, 3, 3, 1, 1, (0.0,)),
]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cb.lib()


def _dy(rng, npq, K, shares):
    dy = rng.standard_normal((npq, K), dtype=np.float32)
    for i, d in enumerate(shares):
        dy[rng.random(npq) >= d, i * 256:(i + 1) * 256] = 0.0
    return dy


@pytest.mark.parametrize("case", CASES, ids=lambda c: "N%dC%dK%d_%dx%d_f%d_s%d_live%s" % (
    c[0], c[1], c[4], c[2], c[3], c[5], c[7], "_".join("%g" % d for d in c[9])))
def test_compacted_weight_gradient(case):
    N, C, H, W, K, R, S, st, pd, shares = case
    print("\n[case] compacted dW %s" % (case,), flush=True)
    rng = np.random.default_rng([210907710, 93, N, C, H, W, K, int(1000 * shares[0])])
    desc = cb.ConvDesc.make(N, C, H, W, K, R, S, st, (pd, pd))
    npq = N * desc.P * desc.Q
    x = torch.from_numpy(np.maximum(rng.standard_normal((N, H, W, C), dtype=np.float32), 0.0)).bfloat16()
    dy = torch.from_numpy(_dy(rng, npq, K, shares)).bfloat16()
    xd, dyd = x.cuda(), dy.cuda()
    bits = torch.zeros(cb.cbw_dy_mask_words(desc), dtype=torch.int32, device="cuda")
    cb.cbw_nonzero_mask_pack(desc.dtype, dyd.numel(), dyd, bits)
    ws = cb.workspace(desc, cb.CBW_OP_BWD_WEIGHT)
    dw = [torch.full((K, R, S, C), float("nan"), device="cuda") for _ in range(3)]
    cb.conv_bwd_weight_sparse(desc, xd, dyd, bits, dw[0], ws)
    stats, work = cb.cbw_read_stats(desc, cb.CBW_OP_BWD_WEIGHT, ws), cb.cbw_read_weight_work(desc, ws)
    occ, chunk, kw = cb.cbw_read_occupancy(desc, ws)
    cb.conv_bwd_weight_sparse(desc, xd, dyd, bits, dw[1], ws)
    cb.conv_bwd_weight_sparse(desc, xd, dyd, bits, dw[2], ws, cb.CBW_FLAG_NO_SKIP)
    torch.cuda.synchronize()
    assert torch.equal(dw[0].view(torch.int32), dw[1].view(torch.int32))
    # blocks executed per k tile: the live pixels' own blocks, or the live chunks
    flat = dy.float().numpy()
    ref_occ = oracle.block_occupancy(flat, chunk, kw)
    assert np.array_equal(occ, ref_occ)
    expect = []
    for kt in range(ref_occ.shape[1]):
        blocks = -(-int((flat[:, kt * kw:(kt + 1) * kw] != 0).any(axis=1).sum()) // chunk)
        live = int(ref_occ[:, kt].sum())
        long = -(-ref_occ.shape[0] // work.shape[0]) >= 16
        saves = 2 * blocks <= live and live - blocks >= 4 * work.shape[0]
        expect.append(blocks if long and saves else live)
    per_tile = work.sum(axis=0)
    assert np.array_equal(per_tile, np.array([expect[t % len(expect)] for t in range(work.shape[1])]))
    assert np.array_equal(work.max(axis=0), -(-per_tile // work.shape[0]))
    assert stats.blocks_skipped == stats.blocks_total - int(per_tile.sum())
    x64 = oracle.nhwc_to_nchw(x.double().numpy())
    dy64 = oracle.nhwc_to_nchw(dy.view(N, desc.P, desc.Q, K).double().numpy())
    ref, ab, nt = oracle.conv_bwd_weight(x64, dy64, (R, S), (st, st), (pd, pd), with_bound=True)
    check_values(oracle.krsc_to_kcrs(dw[0].cpu().double().numpy()), ref, ab, nt, tol_for("bf16"), False, "compacted dW")
    check_dw_regrouped(dw[0], dw[2], stats.blocks_skipped, "compacted dW against no skipping")


def test_more_live_pixels_than_the_list_holds():
    """A 1x1 layer whose four channel tiles leave 64 splits: of a million
    pixels 49% are live, over 7168 per split, so the chunks are walked."""
    desc = cb.ConvDesc.make(20, 1024, 224, 224, 8, 1, 1)
    print("\n[case] compacted dW, list too small", flush=True)
    npq = 20 * 224 * 224
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    x = torch.randn((npq, 1024), generator=g, device="cuda").bfloat16()
    dy = torch.randn((npq, 8), generator=g, device="cuda")
    dy[torch.rand(npq, generator=g, device="cuda") >= 0.49] = 0.0
    dy = dy.bfloat16()
    bits = torch.zeros(cb.cbw_dy_mask_words(desc), dtype=torch.int32, device="cuda")
    cb.cbw_nonzero_mask_pack(desc.dtype, dy.numel(), dy, bits)
    ws = cb.workspace(desc, cb.CBW_OP_BWD_WEIGHT)
    a, b = (torch.empty((8, 1, 1, 1024), device="cuda") for _ in range(2))
    cb.conv_bwd_weight_sparse(desc, x, dy, bits, a, ws)
    st = cb.cbw_read_stats(desc, cb.CBW_OP_BWD_WEIGHT, ws)
    cb.conv_bwd_weight_sparse(desc, x, dy, bits, b, ws, cb.CBW_FLAG_NO_SKIP)
    live = (dy != 0).any(dim=1).sum().item()
    nsplit = cb.cbw_read_weight_work(desc, ws).shape[0]
    assert -(-(-(-live // 64)) // nsplit) * 64 > 7168, "the case has to exceed the list"
    assert st.blocks_skipped == 0
    assert torch.equal(a, b)


def _pack(desc, a):
    bits = torch.zeros(cb.cbw_dy_mask_words(desc), dtype=torch.int32, device="cuda")
    cb.cbw_nonzero_mask_pack(desc.dtype, a.numel(), a, bits)
    return bits


@pytest.mark.parametrize("form", ["x_mask", "x_values", "superset"])
def test_compaction_beside_x_blocks(form):
    """X-block skipping: a tile compacts where the live pixels of dY's footprint
    (here also a strict superset of dY's non-zeros) fit half its blocks live in
    both operands, and then runs every one of them.  Three channel tiles: X
    live everywhere, in half the images (compacts too), in a few (the live
    blocks are walked)."""
    N, C, H, W, K, R, S = 24, 576, 20, 20, 256, 3, 3
    print("\n[case] compacted dW beside X blocks, %s" % form, flush=True)
    rng = np.random.default_rng([210907710, 94])
    desc = cb.ConvDesc.make(N, C, H, W, K, R, S, 1, (1, 1))
    xf = np.maximum(rng.standard_normal((N, H, W, C), dtype=np.float32), 0.0)
    xf[N // 2:, :, :, 256:512] = 0.0
    xf[4:, :, :, 512:] = 0.0
    dyf = _dy(rng, N * H * W, K, (0.1 if form == "superset" else 0.2,))
    foot = dyf.copy()
    if form == "superset":
        foot[rng.random(N * H * W) < 0.1, 7] = 1.0
    x, dy = torch.from_numpy(xf).bfloat16().cuda(), torch.from_numpy(dyf).bfloat16().cuda()
    bits = _pack(desc, torch.from_numpy(foot).bfloat16().cuda())
    xm = None
    if form == "x_mask":
        xm = torch.zeros(cb.cbw_mask_words(desc), dtype=torch.int32, device="cuda")
        cb.cbw_nonzero_mask_pack(desc.dtype, x.numel(), x, xm)
    ws = cb.workspace(desc, cb.CBW_OP_BWD_WEIGHT)
    a, b = (torch.full((K, R, S, C), float("nan"), device="cuda") for _ in range(2))
    cb.conv_bwd_weight_sparse_x(desc, x, dy, xm, bits, a, ws)
    stats, work = cb.cbw_read_stats(desc, cb.CBW_OP_BWD_WEIGHT, ws), cb.cbw_read_weight_work(desc, ws)
    _, chunk, kw = cb.cbw_read_occupancy(desc, ws)
    cb.conv_bwd_weight_sparse_x(desc, x, dy, xm, bits, b, ws, cb.CBW_FLAG_NO_SKIP)
    torch.cuda.synchronize()
    pix = foot.reshape(N, H, W, K).transpose(0, 3, 1, 2) != 0
    live = oracle.weight_block_liveness(oracle.nhwc_to_nchw(x.float().cpu().numpy()) != 0, pix, (R, S), (1, 1), (1, 1),
                                        chunk, kw, 256, 1).sum(axis=3).reshape(-1)   # per tile, in the work items' order
    blocks = -(-int((foot != 0).any(axis=1).sum()) // chunk)
    nsplit = work.shape[0]
    assert -(-(-(-N * H * W // chunk)) // nsplit) >= 16
    compacts = (2 * blocks <= live) & (live - blocks >= 4 * nsplit)
    assert compacts.reshape(R * S, 3)[:, :2].all() and not compacts.reshape(R * S, 3)[:, 2].any()
    assert np.array_equal(work.sum(axis=0), np.where(compacts, blocks, live))
    assert stats.blocks_skipped == stats.blocks_total - int(work.sum())
    ref, ab, nt = oracle.conv_bwd_weight(oracle.nhwc_to_nchw(x.double().cpu().numpy()),
                                         dy.double().cpu().numpy().reshape(N, H, W, K).transpose(0, 3, 1, 2).copy(),
                                         (R, S), (1, 1), (1, 1), with_bound=True)
    check_values(oracle.krsc_to_kcrs(a.cpu().double().numpy()), ref, ab, nt, tol_for("bf16"), False, "compacted dW, X blocks")
    check_dw_regrouped(a, b, stats.blocks_skipped, "compacted dW, X blocks, against no skipping")


@pytest.mark.parametrize("flags", [0, cb.CBW_FLAG_SKIP_X_BLOCKS], ids=["dy", "x_blocks"])
@pytest.mark.parametrize("act,filters", [("nhwc", "krsc"), ("nhwc", "kcrs"), ("nchw", "krsc"), ("nchw", "kcrs")])
def test_compaction_in_the_combined_call(act, filters, flags):
    """conv_bwd_sparse records the live pixels in its preparation launch: the
    gradients are the separate calls' bit for bit and the same blocks run."""
    N, C, H, W, K, R, S = 36, 256, 20, 20, 512, 3, 3
    print("\n[case] compacted dW in the combined call, %s %s flags %d" % (act, filters, flags), flush=True)
    rng = np.random.default_rng([210907710, 95])
    desc = cb.ConvDesc.make(N, C, H, W, K, R, S, 1, (1, 1), w_layout=filters, act_layout=act)
    xf = np.maximum(rng.standard_normal((N, H, W, C), dtype=np.float32), 0.0)
    xf[rng.random((N, H, W)) < 0.5] = 0.0
    xf[N - 2:] = 0.0   # whole windows of X dead
    dyf = _dy(rng, N * H * W, K, (0.3, 0.05)).reshape(N, H, W, K)
    x, dy = (torch.from_numpy(v).bfloat16() for v in (xf, dyf))
    w = torch.from_numpy(rng.standard_normal((K, R, S, C), dtype=np.float32)).bfloat16()
    if act == "nchw":
        x, dy = (v.permute(0, 3, 1, 2).contiguous() for v in (x, dy))
    if filters == "kcrs":
        w = w.permute(0, 3, 1, 2).contiguous()
    x, dy, w = x.cuda(), dy.cuda(), w.cuda()
    bits = _pack(desc, dy)
    xm = torch.zeros(cb.cbw_mask_words(desc), dtype=torch.int32, device="cuda")
    cb.cbw_relu_mask_pack(desc, x, xm)
    dx, sdx = (torch.full_like(x, float("nan")) for _ in range(2))
    dw, sdw = (torch.full(w.shape, float("nan"), device="cuda") for _ in range(2))
    wb, wd, ww = (cb.workspace(desc, op) for op in (cb.CBW_OP_BWD_BOTH, cb.CBW_OP_BWD_DATA_MASKED, cb.CBW_OP_BWD_WEIGHT))
    cb.conv_bwd_sparse(desc, x, dy, w, xm, bits, dx, dw, wb, flags)
    cb.conv_bwd_data_masked(desc, dy, w, xm, sdx, wd)
    if flags:
        cb.conv_bwd_weight_sparse_x(desc, x, dy, xm, bits, sdw, ww)
    else:
        cb.conv_bwd_weight_sparse(desc, x, dy, bits, sdw, ww)
    both, weight = (cb.cbw_read_stats(desc, op, v) for op, v in ((cb.CBW_OP_BWD_BOTH, wb), (cb.CBW_OP_BWD_WEIGHT, ww)))
    torch.cuda.synchronize()
    assert torch.equal(dx.view(torch.int16), sdx.view(torch.int16))
    assert torch.equal(dw.view(torch.int32), sdw.view(torch.int32))
    work = cb.cbw_read_weight_work(desc, ww)
    blocks = [-(-int((dyf[..., 256 * k:256 * k + 256] != 0).any(axis=3).sum()) // 64) for k in (0, 1)]
    assert list(work.sum(axis=0)) == blocks * (work.shape[1] // 2)   # every tile compacts
    assert both.blocks_skipped == weight.blocks_skipped == both.blocks_total - int(work.sum())


def test_one_workspace_compacted_and_not():
    """Calls that compact, walk live chunks, skip nothing and compact another
    footprint, in turn over one workspace: each the result of its own."""
    N, C, H, W, K, R, S = 36, 256, 20, 20, 512, 3, 3
    print("\n[case] one workspace, compacted and not", flush=True)
    rng = np.random.default_rng([210907710, 96])
    desc = cb.ConvDesc.make(N, C, H, W, K, R, S, 1, (1, 1))
    x = torch.from_numpy(np.maximum(rng.standard_normal((N, H, W, C), dtype=np.float32), 0.0)).bfloat16().cuda()
    calls = []
    for shares in ((0.1, 0.1), (1.0, 1.0), (0.7, 0.7), (0.02, 0.3), (0.0, 0.0), (0.1, 1.0)):
        dyf = _dy(rng, N * H * W, K, shares)
        if shares == (0.7, 0.7):
            dyf[:N * H * W // 3] = 0.0   # dead chunks beside dense ones
        dy = torch.from_numpy(dyf).bfloat16().cuda()
        fresh = torch.full((K, R, S, C), float("nan"), device="cuda")
        ws = cb.workspace(desc, cb.CBW_OP_BWD_WEIGHT)
        cb.conv_bwd_weight_sparse(desc, x, dy, _pack(desc, dy), fresh, ws)
        calls.append((dy, _pack(desc, dy), fresh, cb.cbw_read_stats(desc, cb.CBW_OP_BWD_WEIGHT, ws).blocks_skipped))
    assert calls[1][3] == 0 and all(c[3] > 0 for i, c in enumerate(calls) if i != 1)
    shared = cb.workspace(desc, cb.CBW_OP_BWD_WEIGHT)
    for i in (0, 1, 2, 3, 4, 5, 1, 0, 2, 0, 4, 3):
        dy, bits, fresh, skipped = calls[i]
        dw = torch.full((K, R, S, C), float("nan"), device="cuda")
        cb.conv_bwd_weight_sparse(desc, x, dy, bits, dw, shared)
        assert cb.cbw_read_stats(desc, cb.CBW_OP_BWD_WEIGHT, shared).blocks_skipped == skipped
        assert torch.equal(dw.view(torch.int32), fresh.view(torch.int32)), "call %d" % i
