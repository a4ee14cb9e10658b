"""The contraction on packed weights (needs an MI355X), reached through wcc_forward with 256 input
channels and more: each of its three tiles, output rows and positions that end inside a tile, channel
counts that end inside a stage, all coded weight types, packing beside both selections and by a
launch of its own, a compressed signal too small to leave room for the weights, a caller's alpha with
and without a selection."""
import numpy as np
import pytest
import torch

from paper_2205_12268_amd import synth, wcc
from tests.util import dev, rel_l2, upload_weights

pytestmark = pytest.mark.gpu
BF16, I8, I4 = synth.W_BF16, synth.W_I8, synth.W_I4

# B, C_in, C_out, H, W, keep_num, keep_den, weights
CASES = [
    (1, 256, 65, 16, 16, 1, 4, BF16),        # one tile, 63 rows of nothing; k = 64
    (2, 264, 200, 32, 64, 1, 3, BF16),       # a last stage of 8 channels, k = 683
    (1, 272, 300, 32, 64, 3, 10, I8),        # a last stage of 16 channels, two row tiles, k = 615
    (3, 400, 72, 16, 32, 1, 5, I4),          # 4-bit codes widened while packing
    (1, 1024, 700, 8, 16, 1, 1, BF16),       # 44 pieces a thread: packed by its own launch
    (1, 2048, 4096, 2, 4, 1, 4, I8),         # two positions kept: the weights do not fit beside the codes
    (1, 256, 132, 200, 656, 1, 2, I8),       # 256 x 128 tiles: 513 of them, ragged rows and columns; large selection
    (4, 256, 128, 128, 512, 1, 4, BF16),     # 128 x 128 tiles
    (5, 288, 96, 128, 512, 5001, 20000, I8), # the same, ragged; k = 16388
    (2, 260, 80, 32, 64, 1, 4, BF16),        # rows of 520 bytes: not packed
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_layer(ref, case):
    B, Ci, Co, H, W, num, den, wt = case
    cfg = synth.LayerCfg("packed", B, Ci, Co, H, W, 1, num, den, wt, 8, sigma=1.0, clip_hi=4.0,
                         seed=synth.SEED_BASE + 0xF00 + Ci + Co)
    print(f"{cfg} k={cfg.k}", flush=True)
    x, w = synth.make_inputs(cfg)
    d = wcc.make_desc(B, Ci, Co, H, W, 1, num, den, wt, 8)
    ctx = wcc.Context(0)
    need = wcc.workspace_bytes(d)
    ws = torch.full((need + 4096,), 255, dtype=torch.uint8, device="cuda")
    ctx.set_workspace(ws[:need])
    wd, wsd = upload_weights(w)
    xd = dev(x)
    idx = torch.full((B, cfg.k), -7, dtype=torch.int32, device="cuda")
    for alpha_in in (0.0, 1.75):
        y = torch.full((B, Co, H, W), float("nan"), dtype=torch.float32, device="cuda")
        ctx.wcc_forward(d, xd, wd, wsd, alpha_in, y, idx)
        want, o_idx, _ = ref.forward(x, w.values, w.scale, 1, num, den, act_bits=8, alpha_in=alpha_in)
        np.testing.assert_array_equal(idx.cpu().numpy().astype(np.int64), o_idx)
        # products are exact; C_in additions in fp32 (int8: exact), then the two scales
        assert rel_l2(y.cpu().numpy(), want) <= 1e-6
    if alpha_in:    # the index list given, the weights packed by their own launch
        y2 = torch.full_like(y, float("nan"))
        ctx.wcc_forward_fixed(d, xd, wd, wsd, alpha_in, idx, y2)
        assert torch.equal(y, y2)
    assert bool((ws[need:] == 255).all())
    ctx.close()


def test_rows_and_positions_outside_do_not_reach_the_output(ref):
    """NaN weights in one row stay in that row, also across the packed blocks and tiles."""
    cfg = synth.LayerCfg("rows", 1, 264, 200, 32, 64, 1, 1, 4, BF16, 8, sigma=1.0, clip_hi=4.0, seed=synth.SEED_BASE + 0xFE0)
    x, w = synth.make_inputs(cfg)
    d = wcc.make_desc(1, 264, 200, 32, 64, 1, 1, 4, BF16, 8)
    ctx = wcc.Context(0)
    ctx.ensure_workspace(d)
    got = []
    for bad in (False, True):
        stored = w.stored.copy()
        if bad:
            stored[127] = 0x7FC0
        y = torch.empty((1, 200, 32, 64), device="cuda")
        ctx.wcc_forward(d, dev(x), dev(stored), None, 0.0, y)
        got.append(y.cpu().numpy())
    keep = [c for c in range(200) if c != 127]
    assert np.array_equal(got[0][:, keep], got[1][:, keep])
    ctx.close()
