"""The two-launch selection where the norms come as two to 256 planes of partial norms (needs an MI355X).  Its first kernel looks
for crowded digits in plane 0, and in the sums where it finds some; from 32 planes on they are added up first.  Planes that
are crowded, sums that are, both and neither, against a host sort and the stage calls; and the time, which must not
grow with the planes."""
import numpy as np
import pytest
import torch

from paper_2205_12268_amd import wcc

pytestmark = pytest.mark.gpu

# of the channels' amplitudes (multiples of 1/64), a in [1, 2) a block of pixels: the sums are equal where two channels add up to 3
KINDS = {
    "spread": lambda a, c, C: a,
    "first": lambda a, c, C: torch.ones_like(a) if c < C // 2 else a,
    "halves": lambda a, c, C: a if c < C // 2 else 3 - a,
    "pairs": lambda a, c, C: a if c % 2 else 3 - a,
    "equal": lambda a, c, C: torch.ones_like(a),
}


@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("B,C,H,W,levels", [
    (2, 64, 128, 160, 1),     # 2 planes
    (1, 256, 128, 160, 1),    # 8
    (2, 128, 128, 144, 4),    # 16
    (1, 640, 128, 144, 4),    # 32: added up first
])
def test_planes_and_sums(B, C, H, W, levels, kind):
    # One pixel of each 2 x 2 square is not zero, its amplitude the same all over a block of 2^levels: all coefficients of the
    # first level's three bands are half of it.
    co, N, s = 24, H * W, 1 << levels
    gen = torch.Generator(device="cuda")
    gen.manual_seed(C + W)
    a = 1 + torch.randint(0, 64, (B, H // s, W // s), generator=gen, device="cuda").float() / 64
    a = a.repeat_interleave(s // 2, 1).repeat_interleave(s // 2, 2)
    x = torch.zeros((B, C, H, W), device="cuda")
    for c in range(C):
        x[:, c, ::2, ::2] = KINDS[kind](a, c, C)
    w = torch.randint(-7, 8, (co, C), generator=gen, device="cuda").bfloat16()
    ctx = wcc.Context(0)
    for num, den in ((1, 8), (5, 9), (15, 16)):
        d = wcc.make_desc(B, C, co, H, W, levels, num, den, wcc.BF16, 8)
        k = wcc.k_of(d)
        new = lambda shape, dtype=torch.float32: torch.full(shape, -7, dtype=dtype, device="cuda")
        ctx.ensure_workspace(d)
        coef, norm, idx = new((B, C, N)), new((B, N)), new((B, k), torch.int32)
        xc, yc, y, alpha = new((B, C, k), torch.int8), new((B, co, k)), new((B, co, H, W)), new((1,))
        ctx.wcc_haar_fwd(d, x, coef, norm)
        ctx.wcc_joint_topk(d, None, norm, idx)
        ctx.wcc_gather_quant(d, coef, idx, 0.0, xc, alpha)
        ctx.wcc_pointwise(d, w, None, xc, alpha, yc)
        ctx.wcc_scatter_ihaar(d, yc, idx, y)
        ctx._ws.fill_(0x7E)
        y2, idx2, alpha2 = new((B, co, H, W)), new((B, k), torch.int32), new((1,))
        ctx.wcc_forward(d, x, w, None, 0.0, y2, idx2, alpha2)
        torch.cuda.synchronize()
        bits = norm.cpu().numpy().view(np.uint32).astype(np.int64)
        if kind not in ("spread", "first"):
            assert len(np.unique(bits)) <= 3
        for b in range(B):
            want = np.sort(np.lexsort((np.arange(N), -bits[b]))[:k])
            np.testing.assert_array_equal(idx[b].cpu().numpy(), want)
            np.testing.assert_array_equal(idx2[b].cpu().numpy(), want)
        assert torch.equal(alpha, alpha2) and torch.equal(y, y2)
    ctx.close()


# A block whose second norm pass leaves 256 planes of norms and 256 of maxima: a few workgroups that read them all took 1.6 to
# 2.1 times as long as that pass.
def test_many_planes_take_less_than_the_pass_that_wrote_them():
    B, C, e, H, W = 1, 256, 5, 80, 560
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    x = torch.randn((B, C, H, W), generator=gen, device="cuda").bfloat16()
    w1, w3 = (torch.randn(s, generator=gen, device="cuda").bfloat16() / 16 for s in ((C * e, C), (C, C * e)))
    wdw = torch.randn((C * e, 3, 3), generator=gen, device="cuda")
    d = wcc.make_block_desc(B, C, e, H, W, 3, 3, 4, wcc.BF16, 8, wcc.BF16)
    ctx = wcc.Context(0)
    ctx.ensure_workspace(d)
    ctx.set_profiling(True)
    ctx.set_block_profile_layer(1)
    y, times = torch.empty_like(x), []
    for _ in range(12):
        ctx.wcc_block_forward(d, x, w1, None, wdw, w3, None, y)
        torch.cuda.synchronize()
        times.append(ctx.stage_times())
    best = lambda stage: min(t[stage] for t in times[2:])
    assert best("norm_select") < 1.1 * best("haar_fwd")
    ctx.close()
