"""alpha found after the kept coefficients (needs an MI355X): fixed index lists and the stage call, with
few workgroups (their maxima side by side) and with many (the slots), and the caller's alpha, for
which the stage call gathers straight into codes; kept counts that are and are not whole words."""
import numpy as np
import pytest
import torch

from paper_2205_12268_amd import synth, wcc
from tests.util import desc_of, dev, rel_l2, upload_weights

pytestmark = pytest.mark.gpu

# B, C_in, H, W, levels, keep_num, keep_den
SHAPES = [
    (1, 8, 4, 4, 1, 1, 2),          # one workgroup
    (1, 600, 2, 2, 1, 1, 2),        # more workgroups than the plane's partial maxima have room for
    (2, 40, 32, 48, 2, 1, 5),       # k = 308
    (3, 30, 64, 72, 3, 1, 7),       # k = 659
    (2, 700, 16, 24, 2, 1, 3),      # over 1024 gather workgroups: the slots
    (15, 400, 14, 10, 1, 1, 5),     # planes of one strip unit: fewer channel groups, so that the maxima fit
    (40, 64, 16, 16, 2, 1, 4),      # the same with whole words; more samples than keep workgroups for the maxima
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("alpha_in", [0.0, 1.25])
def test_stage_call_and_fixed_lists(ref, shape, alpha_in):
    B, C, H, W, lv, num, den = shape
    cfg = synth.LayerCfg("late", B, C, 6, H, W, lv, num, den, synth.W_BF16, 8, sigma=1.0, clip_hi=4.0,
                         seed=synth.SEED_BASE + 0x1100 + C + H)
    k, N = cfg.k, cfg.N
    x, w = synth.make_inputs(cfg)
    coef = ref.haar_fwd(x.astype(np.float64), lv).reshape(B, C, N)
    rng = np.random.default_rng(cfg.seed)
    idx = np.stack([np.sort(rng.permutation(N)[:k]) for _ in range(B)])
    kept = ref.gather(coef, idx)
    alpha = alpha_in or float(np.abs(kept).max())
    want = ref.quant_codes(kept, float(np.float32(alpha)), 8)
    d = desc_of(cfg)
    ctx = wcc.Context(0)
    need = ctx.ensure_workspace(d)
    ctx._ws.fill_(255)                               # NaN patterns wherever a maximum could be read too early
    codes = torch.full((B, C, k), 99, dtype=torch.int8, device="cuda")
    a = torch.zeros(1, device="cuda")
    ctx.wcc_gather_quant(d, dev(coef.astype(np.float32)), dev(idx.astype(np.int32)), alpha_in, codes, a)
    assert float(a.item()) == np.float32(alpha)
    np.testing.assert_array_equal(codes.cpu().numpy().astype(np.int64), np.asarray(want).astype(np.int64))
    wd, _ = upload_weights(w)
    for given in (idx, None):
        ctx._ws.fill_(255)
        y = torch.full((B, 6, H, W), float("nan"), device="cuda")
        a.zero_()
        ctx.wcc_forward_fixed(d, dev(x), wd, None, alpha_in, None if given is None else dev(given.astype(np.int32)), y, a)
        use = idx if given is not None else np.tile(np.arange(k), (B, 1))
        kp = ref.gather(coef, use)
        al = alpha_in or float(np.abs(kp).max())
        assert float(a.item()) == np.float32(al)
        q = np.asarray(ref.quant_codes(kp, float(np.float32(al)), 8), dtype=np.float64)
        yc = ref.pointwise(w.values, np.full(6, float(np.float32(al)) / 127.0), q)
        assert rel_l2(y.cpu().numpy(), ref.haar_inv(ref.scatter(yc, use, N), H, W, lv)) <= 1e-5
    assert need > 0
    ctx.close()
