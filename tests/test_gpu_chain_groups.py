"""The chained block where the middle channels do not fill the channel groups of the chained norm pass (needs an
MI355X): 42 channels in 8 groups are 7 groups of 6, and one of none, whose plane of partial norms (and of
maxima) the selection adds all the same.  The workspace holds large finite numbers before the call, so that
a plane left unwritten decides the index set."""
import numpy as np
import pytest
import torch

from paper_2205_12268_amd import synth, wcc
from tests.util import check_block_without_middle_outputs, dev, upload_weights

pytestmark = pytest.mark.gpu
F32, BF16, I8 = synth.W_F32, synth.W_BF16, synth.W_I8

# B, C, expansion, H, W, levels, keep, weights, bits
CASES = [
    (2, 14, 3, 72, 84, 2, (1, 5), BF16, 8),      # 7 of 8 groups
    (1, 24, 6, 48, 64, 3, (1, 4), BF16, 8),      # 144 channels, 29 of 32
    (1, 40, 6, 24, 32, 3, (1, 8), I8, 8),        # 240 channels, 30 of 32
    (3, 35, 2, 8, 64, 3, (1, 16), I8, 0),        # 14 of 16, no quantiser
    (2, 53, 5, 8, 80, 3, (1, 8), F32, 0),        # 53 of 64
    (1, 43, 4, 16, 400, 3, (1, 10), BF16, 8),    # a row shared by two waves
    (1, 7, 6, 6, 1020, 1, (1, 5), I8, 8),        # by four; one level, 7 of 8 groups
    (4, 72, 6, 64, 128, 2, (1, 4), BF16, 8),     # 432 channels, alpha before the keep pass: maxima too
]


@pytest.mark.parametrize("norm", [wcc.NORM_L1, wcc.NORM_L2])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_channels_that_do_not_fill_the_groups(ref, case, norm):
    B, C, e, H, W, lv, (num, den), wt, bits = case
    cfg = synth.BlockCfg("groups", B, C, e, H, W, lv, num, den, wt, bits, sigma=1.0,
                         seed=synth.SEED_BASE + 0x1400 + C + e)
    print(cfg, flush=True)
    x, w1, w_dw, w3 = synth.make_block_inputs(cfg)
    d = wcc.make_block_desc(B, C, e, H, W, lv, num, den, wt, bits, wcc.F32, norm)
    assert wcc.block_is_chained(d)
    ctx = wcc.Context(0)
    ctx.ensure_workspace(d)
    w1d, w1s = upload_weights(w1)
    w3d, w3s = upload_weights(w3)
    xd, wdd = dev(x), dev(w_dw)
    y, y_c = (torch.full(x.shape, float("nan"), device="cuda") for _ in range(2))
    t1, t2 = (torch.full((B, cfg.C_mid, H, W), float("nan"), device="cuda") for _ in range(2))
    idx3, idx3_c = (torch.full((B, cfg.k), -7, dtype=torch.int32, device="cuda") for _ in range(2))
    ctx.wcc_block_forward(d, xd, w1d, w1s, wdd, w3d, w3s, y, t1, t2, None, idx3)
    torch.cuda.synchronize()
    ctx._ws.fill_(0x7E)      # 8.4e37 wherever a float is read that nobody wrote
    if norm == wcc.NORM_L1:
        tol = 1e-5 if (wt == F32 and bits == 0) else 1e-2
        check_block_without_middle_outputs(ref, ctx, cfg, d, xd, x.astype(np.float64), w1d, w1s, wdd, w3d, w3s, w3,
                                           t2.cpu().numpy(), y, idx3, tol)
    else:
        # the sums of squares of both routes agree but for their rounding: at most a few positions next to the
        # threshold may differ
        ctx.wcc_block_forward(d, xd, w1d, w1s, wdd, w3d, w3s, y_c, None, None, None, idx3_c)
        torch.cuda.synchronize()
        coef = ref.haar_fwd(t2.cpu().numpy().astype(np.float64), lv).reshape(B, cfg.C_mid, cfg.N)
        sq = (coef ** 2).sum(axis=1)
        for b in range(B):
            sel = idx3_c[b].cpu().numpy().astype(np.int64)
            kth = np.sort(sq[b])[::-1][cfg.k - 1]
            assert np.all(np.diff(sel) > 0) and sq[b][sel].min() >= kth * (1 - 1e-5)
    ctx.close()
