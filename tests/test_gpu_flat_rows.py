"""Rows longer than a wave whose lanes follow each other from strip to strip (needs an MI355X): widths
of 80, 160, 152 and 136 lanes (two columns a lane at d = 4), waves that cross one strip's end, a last
wave that is not full, every level, storage type and keep form."""
import numpy as np
import pytest
import torch

from paper_2205_12268_amd import synth, wcc
from tests.util import dev, rel_l2, tol_for, upload_weights

pytestmark = pytest.mark.gpu

# B, C_in, C_out, H, W, levels, keep, weights, bits
CASES = [
    (1, 6, 5, 2, 320, 1, (1, 3), synth.W_BF16, 8),
    (2, 9, 7, 10, 320, 1, (1, 1), synth.W_F32, 0),
    (1, 20, 8, 12, 640, 2, (1, 4), synth.W_I8, 8),
    (2, 8, 12, 28, 608, 2, (1, 16), synth.W_BF16, 8),
    (1, 12, 6, 24, 320, 3, (1, 8), synth.W_BF16, 8),
    (1, 7, 9, 40, 640, 3, (1, 2), synth.W_F32, 0),
    (3, 18, 4, 8, 608, 3, (1, 1), synth.W_I4, 8),
    (1, 10, 6, 48, 272, 4, (1, 8), synth.W_BF16, 8),
    (2, 4, 5, 16, 160, 4, (2, 3), synth.W_F32, 0),
]


@pytest.mark.parametrize("maps", [wcc.F32, wcc.BF16])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_layer(ref, case, maps):
    B, Ci, Co, H, W, lv, (num, den), wt, bits = case
    cfg = synth.LayerCfg("flat", B, Ci, Co, H, W, lv, num, den, wt, bits, sigma=1.5, clip_hi=4.0,
                         seed=synth.SEED_BASE + 0x1200 + W + lv)
    print(cfg, flush=True)
    x, w = synth.make_inputs(cfg)
    if maps == wcc.BF16:
        x = np.rint(x * 16.0).astype(np.float32) / 16.0     # below 4: exact in bf16
    d = wcc.make_desc(B, Ci, Co, H, W, lv, num, den, wt, bits, maps)
    ctx = wcc.Context(0)
    ctx.ensure_workspace(d)
    wd, ws = upload_weights(w)
    t = torch.bfloat16 if maps == wcc.BF16 else torch.float32
    # a guard band behind y
    flat = torch.full((B * Co * H * W + 4096,), float("nan"), dtype=t, device="cuda")
    y = flat[:B * Co * H * W].view(B, Co, H, W)
    idx = torch.full((B, cfg.k), -7, dtype=torch.int32, device="cuda")
    ctx.wcc_forward(d, dev(x).to(t), wd, ws, 0.0, y, idx)
    want, o_idx, _ = ref.forward(x, w.values, w.scale, lv, num, den, act_bits=bits)
    np.testing.assert_array_equal(idx.cpu().numpy().astype(np.int64), o_idx)
    assert rel_l2(y.float().cpu().numpy(), want) <= (1e-2 if maps == wcc.BF16 else tol_for(cfg))
    assert bool(torch.isnan(flat[B * Co * H * W:]).all())
    if maps == wcc.F32:
        coef = ref.haar_fwd(x.astype(np.float64), lv).reshape(B, Ci, cfg.N)
        g = torch.full((B, Ci, cfg.N), float("nan"), device="cuda")
        norm = torch.full((B, cfg.N), float("nan"), device="cuda")
        ctx.wcc_haar_fwd(d, dev(x), g, norm)
        np.testing.assert_array_equal(g.cpu().numpy(), coef.astype(np.float32))
        np.testing.assert_array_equal(norm.cpu().numpy(), np.abs(coef).sum(axis=1).astype(np.float32))
    ctx.close()
