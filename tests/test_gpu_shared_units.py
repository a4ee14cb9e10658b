"""The norm pass where several waves of a workgroup share a strip unit and add their channel sums in
LDS (needs an MI355X): channel counts below, at and beyond the waves (so that waves have none, one or
a ragged share), the three wave counts a level takes, channel groups on top, every storage type and
norm, widths that are and are not multiples of four -- norms through wcc_haar_fwd bit for bit, the
fused index set, alpha and output through wcc_forward."""
import numpy as np
import pytest
import torch

from paper_2205_12268_amd import synth, wcc
from tests.util import desc_of, dev, rel_l2, upload_weights

pytestmark = pytest.mark.gpu

# B, C_in, H, W, levels
SHAPES = [
    (1, 8, 16, 24, 1),      # four waves, two channels each
    (1, 31, 16, 20, 1),     # one channel short of sixteen waves
    (1, 33, 6, 10, 1),      # W % 4 != 0; sixteen waves, three channels, the last waves idle
    (2, 100, 32, 64, 1),    # sixteen waves and several groups
    (1, 7, 16, 24, 2),      # too few channels to share
    (1, 45, 40, 52, 2),     # sixteen waves, three channels each, the last wave none
    (3, 130, 16, 272, 2),   # two column segments
    (1, 15, 64, 64, 3),     # four waves (eight need sixteen channels)
    (1, 17, 64, 64, 3),     # eight waves, three channels, the last two waves none
    (2, 200, 24, 40, 3),    # eight waves and several groups
    (1, 40, 32, 48, 4),     # four waves at most
]


def layer(B, C, H, W, d, **kw):
    return synth.LayerCfg("shared", B, C, 8, H, W, d, 1, 3, synth.W_BF16, 8, sigma=1.0, clip_hi=4.0,
                          seed=synth.SEED_BASE + 0xD00 + C + 8 * d, **kw)


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_norms_and_index_sets(ref, shape):
    cfg = layer(*shape)
    print(cfg, flush=True)
    x, w = synth.make_inputs(cfg)
    coef = ref.haar_fwd(x.astype(np.float64), cfg.levels).reshape(cfg.B, cfg.C_in, cfg.N)
    d = desc_of(cfg)
    ctx = wcc.Context(0)
    ctx.ensure_workspace(d)
    g_coef = torch.empty((cfg.B, cfg.C_in, cfg.N), device="cuda")
    g_norm = torch.full((cfg.B, cfg.N), float("nan"), device="cuda")
    ctx.wcc_haar_fwd(d, dev(x), g_coef, g_norm)
    np.testing.assert_array_equal(g_norm.cpu().numpy(), np.abs(coef).sum(axis=1).astype(np.float32))
    wd, _ = upload_weights(w)
    want, o_idx, o_alpha = ref.forward(x, w.values, None, cfg.levels, 1, 3, act_bits=8)
    for act in (wcc.F32, wcc.BF16):
        # (multiples of 1/64 below 4 are bf16 numbers only after rounding: fp32 maps and, with
        # the same index set expected, maps that bf16 holds exactly)
        xx = x if act == wcc.F32 else np.rint(x * 16.0).astype(np.float32) / 16.0
        if act == wcc.BF16:
            want, o_idx, o_alpha = ref.forward(xx, w.values, None, cfg.levels, 1, 3, act_bits=8)
        dd = wcc.make_desc(cfg.B, cfg.C_in, 8, cfg.H, cfg.W, cfg.levels, 1, 3, wcc.BF16, 8, act)
        t = torch.float32 if act == wcc.F32 else torch.bfloat16
        y = torch.empty((cfg.B, 8, cfg.H, cfg.W), dtype=t, device="cuda")
        idx = torch.full((cfg.B, cfg.k), -7, dtype=torch.int32, device="cuda")
        alpha = torch.zeros(1, device="cuda")
        ctx.ensure_workspace(dd)
        ctx.wcc_forward(dd, dev(xx).to(t), wd, None, 0.0, y, idx, alpha)
        np.testing.assert_array_equal(idx.cpu().numpy().astype(np.int64), o_idx)
        assert float(alpha.item()) == o_alpha
        # fp32 maps: exact products, at most 200 additions of 2^-24 each, then the inverse; bf16: one rounding of y
        assert rel_l2(y.float().cpu().numpy(), want) <= (1e-5 if act == wcc.F32 else 1e-2)
    ctx.close()


@pytest.mark.parametrize("shape", [SHAPES[3], SHAPES[5], SHAPES[8]], ids=lambda s: "x".join(map(str, s)))
def test_sums_of_squares(ref, shape):
    cfg = layer(*shape)
    x, w = synth.make_inputs(cfg)
    x = np.rint(x * 4.0).astype(np.float32) / 4.0      # every sum of squares is exact in fp32
    norm = (ref.haar_fwd(x.astype(np.float64), cfg.levels).reshape(cfg.B, cfg.C_in, cfg.N) ** 2).sum(axis=1)
    assert np.array_equal(norm, norm.astype(np.float32))
    order = [np.sort(np.lexsort((np.arange(cfg.N), -norm[b]))[:cfg.k]) for b in range(cfg.B)]
    d = wcc.make_desc(cfg.B, cfg.C_in, 8, cfg.H, cfg.W, cfg.levels, 1, 3, wcc.BF16, 8, wcc.F32, wcc.NORM_L2)
    ctx = wcc.Context(0)
    ctx.ensure_workspace(d)
    wd, _ = upload_weights(w)
    y = torch.empty((cfg.B, 8, cfg.H, cfg.W), device="cuda")
    idx = torch.full((cfg.B, cfg.k), -7, dtype=torch.int32, device="cuda")
    ctx.wcc_forward(d, dev(x), wd, None, 0.0, y, idx)
    np.testing.assert_array_equal(idx.cpu().numpy().astype(np.int64), np.stack(order))
    ctx.close()
