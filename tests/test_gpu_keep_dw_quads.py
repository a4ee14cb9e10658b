"""The block's second keep pass, which leaves codes of four channels a word with K_dw in front (needs an MI355X): against the
two layers and the depthwise convolution as calls of their own, bit for bit.  Everything is kept, so the index sets are the
same by construction; the weights are small integers, so the contractions' sums are exact.  One to four levels, rows that
one wave holds and that several share (with and without lanes left idle), channels that do not fill the last quad, quads that do not fill
the last group; and blocks whose quads fit the launch badly, which stay with bytes.  What the workspace holds says which
of the two a call took."""
import pytest
import torch

from paper_2205_12268_amd import wcc
from tests.util import codes_in_workspace

pytestmark = pytest.mark.gpu

# B, C, expansion, H, W, levels
CASES = [
    (4, 64, 2, 64, 256, 1),
    (2, 64, 3, 136, 136, 1),      # rows shared by waves, idle lanes
    (2, 42, 3, 192, 96, 1),       # idle lanes; 126 channels: a quad of two
    (6, 14, 3, 136, 136, 1),      # the same with rows shared; 11 quads in groups of 3
    (8, 80, 4, 128, 128, 2),      # 320 channels, several quads a group
    (2, 42, 3, 96, 192, 2),       # rows shared by waves
    (12, 14, 3, 136, 136, 2),
    (16, 64, 4, 64, 64, 3),
    (8, 64, 3, 96, 192, 3),       # rows shared by waves
    (2, 42, 3, 136, 136, 3),
    (4, 54, 3, 256, 96, 3),       # idle lanes; 41 quads in groups of 3, the last a quad of two
    (6, 54, 3, 136, 136, 3),      # ... and rows shared
    (4, 32, 4, 64, 128, 4),
    (4, 64, 3, 128, 288, 4),      # rows shared by waves
    (2, 42, 3, 144, 176, 4),
    (6, 54, 3, 144, 176, 4),
]
BYTES = [
    (2, 36, 3, 128, 320, 2),
    (4, 64, 3, 128, 128, 3),
    (4, 22, 5, 96, 96, 3),        # (fp32: a small layer)
    (2, 40, 4, 64, 768, 3),
    (4, 24, 6, 128, 160, 4),
    (6, 192, 5, 48, 56, 3),       # 720 workgroups of two quads
]


@pytest.mark.parametrize("wt", [wcc.BF16, wcc.I8])
@pytest.mark.parametrize("case", CASES + BYTES, ids=lambda c: "x".join(map(str, c)))
def test_block_against_its_layers(case, wt):
    B, C, e, H, W, lv = case
    mid, N = C * e, H * W
    if wt == wcc.I8 and (C % 4 or mid % 4):
        pytest.skip("rows of int8 weights are whole dwords")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(H * W + C)
    x = torch.randn((B, C, H, W), generator=gen, device="cuda")
    ints = lambda *s: torch.randint(-7, 8, s, generator=gen, device="cuda")
    dt = torch.bfloat16 if wt == wcc.BF16 else torch.int8
    w1, w3, wdw = ints(mid, C).to(dt), ints(C, mid).to(dt), torch.randn((mid, 3, 3), generator=gen, device="cuda")
    s1 = None if wt == wcc.BF16 else torch.rand(mid, generator=gen, device="cuda") + 0.5
    s3 = None if wt == wcc.BF16 else torch.rand(C, generator=gen, device="cuda") + 0.5
    ctx = wcc.Context(0)
    d = wcc.make_block_desc(B, C, e, H, W, lv, 1, 1, wt, 8)
    assert not wcc.block_is_chained(d)
    ctx.ensure_workspace(d)
    ctx._ws.fill_(0x7E)
    y = torch.full_like(x, float("nan"))
    ctx.wcc_block_forward(d, x, w1, s1, wdw, w3, s3, y)
    d1, d3 = wcc.make_desc(B, C, mid, H, W, lv, 1, 1, wt, 8), wcc.make_desc(B, mid, C, H, W, lv, 1, 1, wt, 8)
    t1, t2 = (torch.empty((B, mid, H, W), device="cuda") for _ in range(2))
    y3 = torch.empty_like(x)
    apart = wcc.Context(0)
    apart.ensure_workspace(d1)
    apart.wcc_forward(d1, x, w1, s1, 0.0, t1)
    apart.wcc_depthwise3x3(t1, wdw, t2)
    apart.ensure_workspace(d3)
    apart.wcc_forward(d3, t2, w3, s3, 0.0, y3)
    torch.cuda.synchronize()
    assert torch.equal(y, x + y3)
    coef, xc, alpha = torch.empty((B, mid, N), device="cuda"), torch.empty((B, mid, N), dtype=torch.int8, device="cuda"), torch.empty(1, device="cuda")
    idx = torch.arange(N, dtype=torch.int32, device="cuda").repeat(B, 1)
    apart.wcc_haar_fwd(d3, t2, coef)
    apart.wcc_gather_quant(d3, coef, idx, 0.0, xc, alpha)
    took = codes_in_workspace(ctx, xc)
    assert took == "words" if case in CASES else took != "words"
    apart.close()
    ctx.close()
