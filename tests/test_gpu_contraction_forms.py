"""The contraction on every form of its operands that is not whole tiles of whole words (needs an
MI355X): the fp32 matrix-instruction kernel through wcc_pointwise (any types, rows of the compressed
signal that no word load can read, every tile choice and its remainders), and the 8-bit stream
kernel on channel counts whose weight rows are not whole 16-byte loads, through wcc_forward with kept
counts that are not multiples of four."""
import numpy as np
import pytest
import torch

from paper_2205_12268_amd import synth, wcc
from tests.util import desc_of, dev, rel_l2, tol_for, upload_weights

pytestmark = pytest.mark.gpu
F32, BF16, I8, I4 = synth.W_F32, synth.W_BF16, synth.W_I8, synth.W_I4

# B, C_in, C_out, H, W, keep_num, keep_den, weights, act bits
STAGED = [
    (1, 1, 1, 2, 6, 1, 4, F32, 0),          # k = 3: less than one load
    (2, 17, 33, 16, 20, 1, 7, F32, 0),      # k = 46, one channel past a stage, one row past a tile
    (1, 32, 32, 64, 64, 1, 2, F32, 0),      # 32-row tiles, whole words
    (3, 15, 64, 30, 34, 1, 3, BF16, 0),     # k = 340
    (1, 48, 65, 30, 34, 101, 1020, I8, 0),  # k = 101: odd rows
    (2, 20, 97, 16, 20, 1, 3, I8, 8),       # k = 107, codes by bytes
    (2, 21, 40, 16, 20, 1, 4, BF16, 8),     # odd channel count, codes by words
    (1, 22, 70, 16, 20, 1, 3, I4, 8),        # 4-bit codes widened first, k = 107
    (4, 24, 96, 128, 256, 1, 4, F32, 0),    # 96-row tiles, 256 workgroups
    (4, 33, 90, 128, 256, 8191, 32768, F32, 0),   # k = 8191: the same with odd rows
    (4, 40, 200, 128, 256, 1, 4, F32, 8),   # 128-row tiles, codes widened
    (2, 31, 120, 128, 256, 16381, 32768, BF16, 0),  # 128-row tiles, k odd, a short last stage
]


@pytest.mark.parametrize("case", STAGED, ids=lambda c: "x".join(map(str, c)))
def test_fp32_matrix_contraction_matches_oracle(ref, case):
    B, Ci, Co, H, W, num, den, wt, bits = case
    cfg = synth.LayerCfg("f32mm", B, Ci, Co, H, W, 1, num, den, wt, bits, seed=synth.SEED_BASE + 0xC00 + Ci)
    k, rng = cfg.k, np.random.default_rng(cfg.seed)
    print(f"{cfg} k={k}", flush=True)
    w = synth.make_w(cfg)
    if bits:
        xc = rng.integers(-127, 128, size=(B, Ci, k), dtype=np.int8)
    else:
        xc = rng.standard_normal((B, Ci, k)).astype(np.float32)
    alpha = np.float32(2.75)
    d = desc_of(cfg)
    ctx = wcc.Context(0)
    ctx.ensure_workspace(d)
    wd, ws = upload_weights(w)
    flat = torch.full((B * Co * k + 64,), float("nan"), dtype=torch.float32, device="cuda")
    ctx.wcc_pointwise(d, wd, ws, dev(xc), dev(np.array([alpha], np.float32)) if bits else None,
                      flat[:B * Co * k].view(B, Co, k))
    torch.cuda.synchronize()
    assert bool(torch.isnan(flat[B * Co * k:]).all())      # nothing written past the end
    got = flat[:B * Co * k].view(B, Co, k).cpu().numpy()
    scale = np.full(Co, float(alpha) / 127.0 if bits else 1.0)
    if w.scale is not None:
        scale = scale * w.scale.astype(np.float64)
    want = ref.pointwise(w.values, scale, xc.astype(np.float64))
    # a chain of C_in fp32 multiply-adds is off by at most C_in * 2^-24 of the sum of |terms|
    # (twice: the scale factors round as well)
    bound = ref.pointwise(np.abs(w.values), np.abs(scale), np.abs(xc.astype(np.float64)))
    assert np.all(np.abs(got - want) <= (Ci + 2) * 2.0 ** -24 * bound)
    ctx.close()


# B, C_in, C_out, H, W, levels, keep_num, keep_den, weights: fused, 8-bit activations
FUSED = [
    (1, 10, 8, 16, 24, 1, 1, 5, BF16),       # K = 10: five dwords a row; k = 77
    (2, 20, 130, 32, 64, 2, 1, 3, I8),       # K = 20, k = 683, two 64-row tiles and two rows
    (1, 76, 70, 64, 96, 3, 1, 7, I8),        # a second chunk of 12 channels, k = 878
    (3, 66, 40, 100, 212, 2, 1, 3, BF16),    # a second chunk of two channels, k = 7067
    (1, 36, 300, 128, 256, 3, 1, 3, I4),     # 256-row tiles are too few: 128-row ones, k = 10923
    (8, 12, 160, 128, 256, 3, 1, 3, BF16),   # 256-row tiles walked by one workgroup, k = 10923
    (1, 3, 5, 16, 24, 1, 1, 5, BF16),        # odd channel count: the fp32 matrix kernel on codes
]


@pytest.mark.parametrize("alpha_in", [0.0, 2.5])
@pytest.mark.parametrize("case", FUSED, ids=lambda c: "x".join(map(str, c)))
def test_ragged_kept_counts_and_channels_through_the_layer(ref, case, alpha_in):
    B, Ci, Co, H, W, lv, num, den, wt = case
    cfg = synth.LayerCfg("ragged", B, Ci, Co, H, W, lv, num, den, wt, 8, sigma=1.5,
                         seed=synth.SEED_BASE + 0xC80 + Ci)
    print(f"{cfg} k={cfg.k} alpha_in={alpha_in}", flush=True)
    assert cfg.k % 4 != 0
    x, w = synth.make_inputs(cfg)
    d = desc_of(cfg)
    ctx = wcc.Context(0)
    need = wcc.workspace_bytes(d)
    # a workspace of exactly the bytes asked for, full of NaN patterns (the padding of the rows
    # then holds NaN), with a guard band behind it
    ws = torch.full((need + 4096,), 255, dtype=torch.uint8, device="cuda")
    ctx.set_workspace(ws[:need])
    wd, wsd = upload_weights(w)
    y = torch.full((B, Co, H, W), float("nan"), dtype=torch.float32, device="cuda")
    idx = torch.full((B, cfg.k), -7, dtype=torch.int32, device="cuda")
    ctx.wcc_forward(d, dev(x), wd, wsd, alpha_in, y, idx)
    torch.cuda.synchronize()
    assert bool((ws[need:] == 255).all())
    want, o_idx, _ = ref.forward(x, w.values, w.scale, lv, num, den, act_bits=8, alpha_in=alpha_in)
    np.testing.assert_array_equal(idx.cpu().numpy().astype(np.int64), o_idx)
    assert rel_l2(y.cpu().numpy(), want) <= tol_for(cfg)
    ctx.close()


@pytest.mark.parametrize("wt", [BF16, I8])
def test_a_row_of_weights_does_not_reach_into_the_row_before(ref, wt):
    """C_in = 20: the last 16-byte load of a row also brings in the first weights of the next one.
    With that row all NaN (bf16) or at the ends of its range (int8) the others must not change."""
    cfg = synth.LayerCfg("rows", 1, 20, 64, 32, 32, 2, 1, 4, wt, 8, sigma=1.5, seed=synth.SEED_BASE + 0xCC0)
    x, w = synth.make_inputs(cfg)
    d = desc_of(cfg)
    ctx = wcc.Context(0)
    ctx.ensure_workspace(d)
    got = []
    for bad in (False, True):
        stored = w.stored.copy()
        if bad:
            stored[7] = 0x7FC0 if wt == BF16 else 127
        y = torch.empty((1, 64, 32, 32), dtype=torch.float32, device="cuda")
        ctx.wcc_forward(d, dev(x), dev(stored), None if w.scale is None else dev(w.scale), 0.0, y)
        got.append(y.cpu().numpy())
    keep = [c for c in range(64) if c != 7]
    assert np.array_equal(got[0][:, keep], got[1][:, keep])
    ctx.close()


def test_static_entry_takes_a_layer_that_fits_only_without_padding():
    """The largest layer of this family that the fixed array holds without the padding of its rows
    is one it does not hold with it; it is still accepted, and gives what its own workspace gives."""
    found = None
    for co in range(16384, 1, -1):
        d = wcc.make_desc(1, 64, co, 64, 96, 2, 1, 5, wcc.BF16, 8)    # k = 1229: three positions of padding
        if wcc.workspace_bytes(d) <= wcc.STATIC_SCRATCH_BYTES:
            found = co
            break
    k = -(-64 * 96 // 5)
    padded = (wcc.workspace_bytes(wcc.make_desc(1, 64, found, 64, 96, 2, 1, 5, wcc.BF16, 8)) +
              (64 + found) * 4 * (-k % 4))
    assert found is not None and padded > wcc.STATIC_SCRATCH_BYTES
    cfg = synth.LayerCfg("nopad", 1, 64, found, 64, 96, 2, 1, 5, BF16, 8, sigma=1.5, seed=synth.SEED_BASE + 0xCD0)
    x, w = synth.make_inputs(cfg)
    wd, _ = upload_weights(w)
    ctx = wcc.Context(0)
    d = desc_of(cfg)
    ctx.ensure_workspace(d)
    ys = [torch.full((1, found, 64, 96), float("nan"), dtype=torch.float32, device="cuda") for _ in range(2)]
    ctx.wcc_forward_static(d, dev(x), wd, None, 0.0, ys[0])
    ctx.wcc_forward(d, dev(x), wd, None, 0.0, ys[1])
    torch.cuda.synchronize()
    assert bool(torch.isfinite(ys[0]).all()) and torch.equal(ys[0], ys[1])
    ctx.close()
