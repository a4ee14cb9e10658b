"""The kernel that takes contraction and inverse in one (needs an MI355X): layers of few channels, three levels and
a long kept signal, at the edges of what it takes.  Every operand type, one step of channels and two, rows of
weights that end inside a 16-byte load, output channels that are no multiple of 16, units that keep nothing, units
that keep everything (more than the LDS holds of two steps), a last unit that is not full, each way to the index list and
to alpha, and both storage types; the stage times say that the one kernel ran."""
import numpy as np
import pytest
import torch

from paper_2205_12268_amd import synth, wcc
from tests.util import check_block_without_middle_outputs, dev, layer_with_index_set, rel_l2, tol_for, upload_weights

pytestmark = pytest.mark.gpu

# B, C_in, C_out, H, W, keep, weights, bits, the maps' types with which the layer runs contraction and inverse as one kernel:
# at least 48 MiB of output coefficients and 900 units of 512 positions
F32, BF16 = wcc.F32, wcc.BF16
CASES = [
    (4, 64, 52, 264, 512, (3, 4), synth.W_BF16, 8, {F32, BF16}),   # a whole step; 4 channels in the last block
    (8, 10, 50, 256, 256, (3, 4), synth.W_BF16, 8, {F32, BF16}),   # a row of 20 bytes
    (4, 24, 49, 256, 512, (3, 4), synth.W_I4, 8, {F32, BF16}),     # one channel in the last block
    (9, 5, 64, 152, 352, (1, 2), synth.W_F32, 0, {F32}),     # 88 lanes a strip, units across strips, a last one of 8 lanes
    (4, 8, 184, 256, 360, (1, 1), synth.W_I8, 8, {F32, BF16}),     # all kept: rows that are not whole lines
    (4, 8, 184, 264, 360, (1, 1), synth.W_I8, 8, {F32, BF16}),     # the same, units across strips, a last one of 10 lanes
    (6, 128, 100, 256, 320, (1, 2), synth.W_I8, 8, {F32, BF16}),   # two steps; units that the LDS does not hold
    (4, 68, 100, 264, 448, (1, 2), synth.W_I8, 8, {F32, BF16}),    # one channel quad in the second step
    (4, 72, 104, 264, 448, (2, 5), synth.W_I4, 8, {F32, BF16}),
    (4, 32, 68, 264, 512, (1, 2), synth.W_F32, 0, {F32, BF16}),    # two steps of fp32
    (4, 20, 72, 256, 512, (1, 2), synth.W_F32, 8, {F32, BF16}),
    # next to them, in the two kernels: two steps and more than half kept
    (7, 128, 36, 256, 320, (2, 3), synth.W_I8, 8, set()),
    (4, 68, 40, 264, 480, (2, 3), synth.W_I8, 8, set()),
    (4, 32, 36, 264, 512, (2, 3), synth.W_F32, 0, set()),
    (4, 20, 40, 256, 512, (2, 3), synth.W_F32, 8, set()),
]


def _input(cfg, maps):
    x, w = synth.make_inputs(cfg)
    # a part of every plane is zero: with three quarters kept its units hold nothing but ties, which go to the lower
    # positions; another is loud, and keeps everything
    x[:, :, :64, :128] = 0.0
    x[:, :, 128:192, :64] *= 8.0
    if maps == wcc.BF16:
        x = np.rint(x * 8.0).astype(np.float32) / 8.0      # below 32: exact in bf16
    return x, w


@pytest.mark.parametrize("maps", [wcc.F32, wcc.BF16])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[:-1])))
def test_layer(ref, case, maps):
    B, Ci, Co, H, W, (num, den), wt, bits, one_kernel = case
    cfg = synth.LayerCfg("tail", B, Ci, Co, H, W, 3, num, den, wt, bits, sigma=1.0, clip_hi=3.0,
                         seed=synth.SEED_BASE + 0x1500 + Ci)
    print(cfg, flush=True)
    x, w = _input(cfg, maps)
    d = wcc.make_desc(B, Ci, Co, H, W, 3, num, den, wt, bits, maps)
    ctx = wcc.Context(0)
    need = wcc.workspace_bytes(d)
    ws = torch.full((need + 4096,), 255, dtype=torch.uint8, device="cuda")  # NaN patterns, a guard band behind
    ctx.set_workspace(ws[:need])
    wd, wsd = upload_weights(w)
    t = torch.bfloat16 if maps == wcc.BF16 else torch.float32
    tol = 1e-2 if maps == wcc.BF16 else tol_for(cfg)
    flat = torch.full((B * Co * H * W + 4096,), float("nan"), dtype=t, device="cuda")
    y = flat[:B * Co * H * W].view(B, Co, H, W)
    idx = torch.full((B, cfg.k), -7, dtype=torch.int32, device="cuda")
    alpha = torch.zeros(1, device="cuda")
    xd = dev(x).to(t)
    ctx.set_profiling(True)
    ctx.wcc_forward(d, xd, wd, wsd, 0.0, y, idx, alpha if bits else None)
    ms = ctx.stage_times()
    ctx.set_profiling(False)
    assert ms["scatter_ihaar"] > 0 and (ms["pointwise"] == 0) == (maps in one_kernel)
    want, o_idx, o_alpha = ref.forward(x, w.values, w.scale, 3, num, den, act_bits=bits)
    np.testing.assert_array_equal(idx.cpu().numpy().astype(np.int64), o_idx)
    if bits:
        assert float(alpha.item()) == np.float32(o_alpha)
    assert rel_l2(y.float().cpu().numpy(), want) <= tol
    first = y.clone()
    # the same list given, and the list "first k": alpha is found in the second pass, which leaves fp32
    y.fill_(float("nan"))
    ctx.wcc_forward_fixed(d, xd, wd, wsd, 0.0, idx, y)
    assert torch.equal(y, first)
    y.fill_(float("nan"))
    ctx.wcc_forward_fixed(d, xd, wd, wsd, 0.0, None, y)
    lists = np.broadcast_to(np.arange(cfg.k), (B, cfg.k)).copy()
    want, _ = ref.forward_with_list(x, w.values, w.scale, 3, lists, act_bits=bits)[:2]
    assert rel_l2(y.float().cpu().numpy(), want) <= tol
    if bits:  # a given alpha
        y.fill_(float("nan"))
        ctx.wcc_forward(d, xd, wd, wsd, 2.5, y)
        want, _, _ = ref.forward(x, w.values, w.scale, 3, num, den, act_bits=bits, alpha_in=2.5)
        assert rel_l2(y.float().cpu().numpy(), want) <= tol
    assert bool(torch.isnan(flat[B * Co * H * W:]).all()) and bool((ws[need:] == 255).all())
    ctx.close()


def test_a_row_of_weights_does_not_reach_into_the_row_before():
    """20 channels: the last 16-byte load of a row of 40 bytes brings in the next row's first weights."""
    cfg = synth.LayerCfg("tail_rows", 4, 20, 36, 264, 512, 3, 3, 4, synth.W_BF16, 8, sigma=1.0, seed=synth.SEED_BASE + 0x1580)
    x, w = synth.make_inputs(cfg)
    d = wcc.make_desc(4, 20, 36, 264, 512, 3, 3, 4, synth.W_BF16, 8)
    ctx = wcc.Context(0)
    ctx.ensure_workspace(d)
    got = []
    for bad in (False, True):
        stored = w.stored.copy()
        if bad:
            stored[7] = 0x7FC0  # NaN
        y = torch.empty((4, 36, 264, 512), dtype=torch.float32, device="cuda")
        ctx.wcc_forward(d, dev(x), dev(stored), None, 0.0, y)
        got.append(y)
    keep = [c for c in range(36) if c != 7]
    assert torch.equal(got[0][:, keep], got[1][:, keep])
    ctx.close()


def test_in_the_static_scratch_memory(ref):
    """A layer with the tail in one kernel whose intermediates fit wcc_forward_static: the same bits, and the oracle's."""
    cfg = synth.LayerCfg("tail_static", 4, 8, 104, 256, 480, 3, 1, 4, synth.W_F32, 0, sigma=1.0, seed=synth.SEED_BASE + 0x1590)
    x, w = synth.make_inputs(cfg)
    d = wcc.make_desc(4, 8, 104, 256, 480, 3, 1, 4, wcc.F32, 0)
    assert wcc.workspace_bytes(d) <= 64 << 20
    ctx = wcc.Context(0)
    ctx.ensure_workspace(d)
    xd, (wd, _) = dev(x), upload_weights(w)
    y, y_static = (torch.full((4, 104, 256, 480), float("nan"), device="cuda") for _ in range(2))
    idx, idx_static = (torch.full((4, cfg.k), -7, dtype=torch.int32, device="cuda") for _ in range(2))
    ctx.set_profiling(True)
    ctx.wcc_forward(d, xd, wd, None, 0.0, y, idx)
    assert ctx.stage_times()["pointwise"] == 0
    ctx.wcc_forward_static(d, xd, wd, None, 0.0, y_static, idx_static)
    assert torch.equal(y, y_static) and torch.equal(idx, idx_static)
    want, o_idx, _ = ref.forward(x, w.values, w.scale, 3, 1, 4, act_bits=0)
    np.testing.assert_array_equal(idx.cpu().numpy().astype(np.int64), o_idx)
    assert rel_l2(y.cpu().numpy(), want) <= tol_for(cfg)
    ctx.close()


@pytest.mark.parametrize("maps", [wcc.F32, wcc.BF16])
def test_expand_layer_of_a_block(ref, maps):
    """Half kept, so that the block forms its middle tensor: the expand layer ends in the one kernel, the project layer in
    the two.  bf16 maps round the middle tensor and y once each."""
    cfg = synth.BlockCfg("tail_block", 8, 16, 6, 256, 256, 3, 1, 2, synth.W_BF16, 8, sigma=1.0, seed=synth.SEED_BASE + 0x15A0)
    x, w1, w_dw, w3 = synth.make_block_inputs(cfg)
    if maps == wcc.BF16:
        x = synth.round_to_bf16(x)
    t = torch.bfloat16 if maps == wcc.BF16 else torch.float32
    d = wcc.make_block_desc(cfg.B, cfg.C, cfg.expansion, cfg.H, cfg.W, 3, 1, 2, cfg.w_dtype, 8, maps)
    assert not wcc.block_is_chained(d)
    ctx = wcc.Context(0)
    ctx.ensure_workspace(d)
    ctx.set_block_profile_layer(0)
    ctx.set_profiling(True)
    xd, (w1d, _), (w3d, _) = dev(x).to(t), upload_weights(w1), upload_weights(w3)
    y, t1 = torch.full_like(xd, float("nan")), torch.empty((cfg.B, cfg.C_mid, cfg.H, cfg.W), dtype=t, device="cuda")
    idx1, idx3 = (torch.empty((cfg.B, cfg.k), dtype=torch.int32, device="cuda") for _ in range(2))
    ctx.wcc_block_forward(d, xd, w1d, None, dev(w_dw), w3d, None, y, t1, None, idx1, idx3)
    assert ctx.stage_times()["pointwise"] == 0
    want, o_idx, _ = ref.forward(x, w1.values, w1.scale, 3, 1, 2, act_bits=8)
    np.testing.assert_array_equal(idx1.cpu().numpy().astype(np.int64), o_idx)
    got_t1 = t1.float().cpu().numpy().astype(np.float64)
    assert rel_l2(got_t1, want) <= 1e-2
    branch, _ = layer_with_index_set(ref, cfg.layer(1), w3, ref.depthwise3x3(got_t1, w_dw),
                                     idx3.cpu().numpy().astype(np.int64))
    assert rel_l2(y.float().cpu().numpy(), x.astype(np.float64) + branch) <= 1e-2
    ctx.close()


def test_expand_layer_of_a_block_that_may_run_chained(ref):
    """A quarter kept: the middle tensor that a caller asks for comes from the contraction that the chained call runs, so that
    both calls give the same bits, although the layer by itself would take the one kernel."""
    cfg = synth.BlockCfg("tail_chain", 8, 16, 8, 256, 256, 3, 1, 4, synth.W_BF16, 8, sigma=1.0, seed=synth.SEED_BASE + 0x15A1)
    x, w1, w_dw, w3 = synth.make_block_inputs(cfg)
    d = wcc.make_block_desc(cfg.B, cfg.C, cfg.expansion, cfg.H, cfg.W, 3, 1, 4, cfg.w_dtype, 8)
    assert wcc.block_is_chained(d)
    ctx = wcc.Context(0)
    ctx.ensure_workspace(d)
    ctx.set_block_profile_layer(0)
    ctx.set_profiling(True)
    xd, wdd, (w1d, _), (w3d, _) = dev(x), dev(w_dw), upload_weights(w1), upload_weights(w3)
    y = torch.full_like(xd, float("nan"))
    t1, t2 = (torch.empty((cfg.B, cfg.C_mid, cfg.H, cfg.W), device="cuda") for _ in range(2))
    idx3 = torch.empty((cfg.B, cfg.k), dtype=torch.int32, device="cuda")
    ctx.wcc_block_forward(d, xd, w1d, None, wdd, w3d, None, y, t1, t2, None, idx3)
    assert ctx.stage_times()["pointwise"] > 0
    ctx.set_profiling(False)
    check_block_without_middle_outputs(ref, ctx, cfg, d, xd, x.astype(np.float64), w1d, None, wdd, w3d, None, w3,
                                       t2.cpu().numpy(), y, idx3, 1e-2)
    lone = wcc.make_desc(cfg.B, cfg.C, cfg.C_mid, cfg.H, cfg.W, 3, 1, 4, cfg.w_dtype, 8)
    ctx.set_profiling(True)
    ctx.wcc_forward(lone, xd, w1d, None, 0.0, t2)
    assert ctx.stage_times()["pointwise"] == 0 and rel_l2(t2.cpu().numpy(), t1.double().cpu().numpy()) <= 1e-6
    ctx.close()
