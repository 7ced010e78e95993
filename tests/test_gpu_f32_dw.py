"""GPU parity of the float32 weight gradient against the fp64 oracle: widths
around the 64-column parts and the 256-channel tiles, images narrower than the
four pixels of a step, chunks that cross rows and images, a ragged last chunk,
strides and pads (also so wide that the columns of a row span more than 2^31
bytes), several splits, and runs of dead chunks longer than one ballot (64
chunks per wave), skipped and not.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2109_07710_amd as cb
from parity import check_dw_regrouped, check_values, tol_for

pytestmark = pytest.mark.gpu

CASES = [
    # N, C, H, W, K, R, S, stride, pad, images with a zero dY
    (1, 4, 5, 3, 4, 3, 3, (1, 1), (1, 1), 0),        # one vector of channels, rows of three pixels
    (3, 64, 7, 1, 68, 1, 1, (1, 1), (0, 0), 1),      # rows of one pixel
    (2, 68, 9, 33, 64, 3, 3, (2, 2), (1, 1), 1),
    (2, 260, 8, 10, 260, 1, 1, (1, 1), (0, 0), 0),   # two tiles of 256 along both
    (5, 128, 13, 11, 60, 2, 3, (1, 2), (0, 2), 2),
    (1, 1 << 20, 1, 1, 4, 1, 1, (1, 32), (1, 512), 0),   # columns of the padding 2^31 bytes from the image
    (9, 32, 40, 64, 16, 3, 3, (1, 1), (1, 1), 7),    # 720 chunks, 560 of them dead in one run
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "N%dC%dK%d_%dx%d_f%dx%d_dead%d" % (
    c[0], c[1], c[4], c[2], c[3], c[5], c[6], c[9]))
def test_f32_weight_gradient(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    N, C, H, W, K, R, S, st, pd, dead = case
    print("\n[case] f32 dW %s" % (case,), flush=True)
    rng = np.random.default_rng([210907710, 92, N, C, H, W, K])
    desc = cb.ConvDesc.make(N, C, H, W, K, R, S, st, pd, dtype="f32")
    x = np.maximum(rng.standard_normal((N, H, W, C), dtype=np.float32), 0.0)
    dy = rng.standard_normal((N, desc.P, desc.Q, K), dtype=np.float32)
    dy[1:1 + dead] = 0.0
    xd, dyd = torch.from_numpy(x).cuda(), torch.from_numpy(dy).cuda()
    ws = cb.workspace(desc, cb.CBW_OP_BWD_WEIGHT)
    dw = {f: torch.full((K, R, S, C), float("nan"), device="cuda") for f in (0, cb.CBW_FLAG_NO_SKIP)}
    skipped = 0
    for f, g in dw.items():
        cb.conv_bwd_weight_sparse(desc, xd, dyd, None, g, ws, f)
        st_ = cb.cbw_read_stats(desc, cb.CBW_OP_BWD_WEIGHT, ws)
        work = cb.cbw_read_weight_work(desc, ws)
        assert int(work.sum()) == st_.blocks_total - st_.blocks_skipped
        skipped = max(skipped, st_.blocks_skipped)
    occ = oracle.block_occupancy(dy.reshape(-1, K), 32, 256)
    assert skipped == int((occ == 0).sum()) * R * S * (-(-C // 256))
    x64, dy64 = oracle.nhwc_to_nchw(x.astype(np.float64)), oracle.nhwc_to_nchw(dy.astype(np.float64))
    ref, ab, nt = oracle.conv_bwd_weight(x64, dy64, (R, S), st, pd, with_bound=True)
    for f, g in dw.items():
        check_values(oracle.krsc_to_kcrs(g.cpu().double().numpy()), ref, ab, nt, tol_for("f32"), False, "f32 dW %d" % f)
    check_dw_regrouped(dw[0], dw[cb.CBW_FLAG_NO_SKIP], skipped, "f32 dW, skipping against not")
