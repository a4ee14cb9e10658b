"""Four levels: lanes of two columns (needs an MI355X).  Planes of one and several 16-row strips, one
and several column segments, lanes outside the plane; kept counts a strip's packed lists hold (4, 8
and 16 rows of 64) and do not hold; fp32 and bf16 maps, both routes of alpha; and the residual block,
whose K_dw is folded into these passes."""
import numpy as np
import pytest
import torch

from paper_2205_12268_amd import synth, wcc
from tests.util import assert_valid_index_set, check_block_without_middle_outputs, dev, layer_with_index_set, rel_l2, tol_for, upload_weights

pytestmark = pytest.mark.gpu

# B, C_in, C_out, H, W, keep, weights, bits
LAYERS = [
    (1, 5, 3, 16, 16, (1, 1), synth.W_F32, 0),
    (2, 12, 20, 32, 48, (1, 16), synth.W_BF16, 8),
    (1, 24, 16, 16, 272, (1, 8), synth.W_I8, 8),
    (1, 16, 24, 48, 144, (3, 10), synth.W_I4, 8),
    (1, 9, 7, 32, 160, (1, 2), synth.W_F32, 0),
    (2, 8, 8, 64, 128, (1, 1), synth.W_BF16, 8),
]


@pytest.mark.parametrize("maps", [wcc.F32, wcc.BF16])
@pytest.mark.parametrize("case", LAYERS, ids=lambda c: "x".join(map(str, c)))
def test_layer(ref, case, maps):
    B, Ci, Co, H, W, (num, den), wt, bits = case
    cfg = synth.LayerCfg("four", B, Ci, Co, H, W, 4, num, den, wt, bits, sigma=2.0, clip_hi=4.0,
                         seed=synth.SEED_BASE + 0xE00 + H + W)
    print(cfg, flush=True)
    x, w = synth.make_inputs(cfg)
    if maps == wcc.BF16:
        x = np.rint(x * 16.0).astype(np.float32) / 16.0     # below 4: exact in bf16
    ctx = wcc.Context(0)
    d = wcc.make_desc(B, Ci, Co, H, W, 4, num, den, wt, bits, maps)
    ctx.ensure_workspace(d)
    wd, ws = upload_weights(w)
    t = torch.bfloat16 if maps == wcc.BF16 else torch.float32
    for alpha_in in ([0.0, 1.5] if bits else [0.0]):
        y = torch.full((B, Co, H, W), float("nan"), dtype=t, device="cuda")
        idx = torch.full((B, cfg.k), -7, dtype=torch.int32, device="cuda")
        ctx.wcc_forward(d, dev(x).to(t), wd, ws, alpha_in, y, idx)
        want, o_idx, _ = ref.forward(x, w.values, w.scale, 4, num, den, act_bits=bits, alpha_in=alpha_in)
        np.testing.assert_array_equal(idx.cpu().numpy().astype(np.int64), o_idx)
        assert rel_l2(y.float().cpu().numpy(), want) <= (1e-2 if maps == wcc.BF16 else tol_for(cfg))
    ctx.close()


@pytest.mark.parametrize("H,W,num,den", [(16, 32, 1, 8), (48, 160, 1, 4), (32, 272, 1, 2)])
def test_block(ref, H, W, num, den):
    cfg = synth.BlockCfg("four_block", 1, 6, 3, H, W, 4, num, den, synth.W_BF16, 8, sigma=2.0,
                         seed=synth.SEED_BASE + 0xE80 + W)
    x, w1, w_dw, w3 = synth.make_block_inputs(cfg)
    d = wcc.make_block_desc(1, 6, 3, H, W, 4, num, den, synth.W_BF16, 8)
    ctx = wcc.Context(0)
    ctx.ensure_workspace(d)
    w1d, w1s = upload_weights(w1)
    w3d, w3s = upload_weights(w3)
    mid = (1, cfg.C_mid, H, W)
    y, t1, t2 = (torch.full(s, float("nan"), device="cuda") for s in (x.shape, mid, mid))
    idx1, idx3 = (torch.empty((1, cfg.k), dtype=torch.int32, device="cuda") for _ in range(2))
    ctx.wcc_block_forward(d, dev(x), w1d, w1s, dev(w_dw), w3d, w3s, y, t1, t2, idx1, idx3)
    torch.cuda.synchronize()
    g_t2 = t2.cpu().numpy()
    assert rel_l2(g_t2, ref.depthwise3x3(t1.cpu().numpy(), w_dw)) <= 1e-6
    sel = idx3.cpu().numpy().astype(np.int64)
    want, norm = layer_with_index_set(ref, cfg.layer(1), w3, g_t2.astype(np.float64), sel)
    assert_valid_index_set(norm[0], sel[0], cfg.k)
    assert rel_l2(y.cpu().numpy() - x, want) <= 1e-2
    check_block_without_middle_outputs(ref, ctx, cfg, d, dev(x), x.astype(np.float64), w1d, w1s, dev(w_dw),
                                       w3d, w3s, w3, g_t2, y, idx3, 1e-2)
    ctx.close()
