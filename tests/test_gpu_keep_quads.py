"""Layers whose second pass leaves codes of four channels a word (needs an MI355X): against the five stage calls, whose
codes are bytes.  Weights are small integers, so every sum is exact and the results agree bit for bit.  One to four levels,
packed list and word a slot, list forms of 4 to 16 rows, channels that do not fill the last quad, more and fewer quads
than groups, groups of unequal length, planes with idle lanes and lanes of all strips in a row, the contraction kernels
that read words, bf16 maps, the caller's alpha; and layers whose quads fit the launch badly, which stay with bytes.  What the
workspace holds says which of the two a call took."""
import pytest
import torch

from paper_2205_12268_amd import wcc
from tests.util import codes_in_workspace

pytestmark = pytest.mark.gpu

# B, C_in, C_out, H, W, levels, keep, weights
CASES = [
    (4, 64, 24, 64, 128, 1, (1, 4), wcc.I8),
    (4, 130, 40, 34, 50, 1, (1, 2), wcc.BF16),       # two columns a lane, a quad of two channels
    (4, 128, 72, 64, 128, 2, (1, 8), wcc.I8),        # 4 rows
    (2, 134, 40, 100, 212, 2, (1, 3), wcc.BF16),     # 8 rows, idle lanes, rows of yc that are padded
    (4, 128, 16, 64, 128, 2, (9, 10), wcc.I8),       # a word a slot
    (4, 64, 96, 256, 256, 3, (1, 8), wcc.BF16),
    (8, 128, 136, 96, 128, 3, (1, 2), wcc.I8),       # 16 rows and a word a slot, side by side
    (3, 256, 130, 128, 128, 3, (1, 3), wcc.I8),      # packed weights
    (8, 64, 40, 256, 256, 2, (1, 16), wcc.I4),       # several quads a group
    (4, 64, 40, 128, 320, 3, (1, 4), wcc.BF16),      # 12 rows, lanes of all strips follow each other
    (4, 128, 72, 128, 320, 3, (3, 4), wcc.I8),
    (2, 256, 72, 64, 512, 2, (1, 4), wcc.BF16),      # packed bf16 weights
    (2, 58, 24, 128, 256, 3, (1, 3), wcc.BF16),      # 15 quads in 8 groups, the last a quad of two
    (2, 114, 40, 192, 320, 1, (1, 2), wcc.BF16),     # 29 quads in 16 groups, the last a quad of two
    (8, 64, 40, 128, 128, 4, (1, 8), wcc.BF16),      # four levels: a packed list
    (8, 64, 48, 128, 128, 4, (3, 4), wcc.I8),        # a word a slot
    (8, 64, 40, 128, 112, 4, (1, 3), wcc.I8),        # idle lanes
    (2, 58, 40, 128, 320, 4, (1, 3), wcc.BF16),      # 15 quads in 8 groups, lanes of all strips follow each other
]
BYTES = [
    (4, 66, 40, 128, 320, 3, (1, 4), wcc.BF16),      # 17 quads for 16 groups
    (2, 264, 72, 64, 512, 2, (1, 4), wcc.BF16),      # 66 for 32
    (4, 64, 40, 128, 128, 4, (1, 8), wcc.BF16),      # too few waves by quads
    (4, 64, 48, 128, 96, 4, (3, 4), wcc.I8),
    (8, 128, 136, 96, 160, 3, (1, 2), wcc.I8),       # 768 workgroups of one quad: a round and a half-empty one
    (4, 128, 72, 128, 320, 3, (1, 4), wcc.I8),       # 640
    (11, 456, 24, 64, 48, 3, (1, 8), wcc.BF16),     # 704 of two
    (9, 484, 24, 80, 32, 4, (1, 4), wcc.BF16),
]


@pytest.mark.parametrize("alpha", [0.0, 3.0])
@pytest.mark.parametrize("case", CASES + BYTES, ids=lambda c: "x".join(map(str, c)))
def test_words_against_the_stage_calls(case, alpha):
    B, ci, co, H, W, lv, (num, den), wt = case
    gen = torch.Generator(device="cuda")
    gen.manual_seed(H * W + ci)
    # (multiples of 1/8 below 8: exact in bf16, and so are the channel norms in fp32)
    x = torch.randint(-63, 64, (B, ci, H, W), generator=gen, device="cuda").float() / 8
    x *= torch.rand((B, 1, H, W), generator=gen, device="cuda") < 0.7
    w = torch.randint(-7, 8, (co, ci), generator=gen, device="cuda")
    scale = None
    if wt == wcc.BF16:
        stored = w.bfloat16()
    elif wt == wcc.I8:
        stored = w.to(torch.int8)
    else:
        nib = w.to(torch.int8).view(torch.uint8) & 15
        stored = (nib[:, 0::2] | (nib[:, 1::2] << 4)).contiguous()
    if wt != wcc.BF16:
        scale = torch.ones(co, device="cuda")
    d = wcc.make_desc(B, ci, co, H, W, lv, num, den, wt, 8)
    k, N = wcc.k_of(d), H * W
    new = lambda shape, dtype=torch.float32: torch.full(shape, -7, dtype=dtype, device="cuda")
    ctx = wcc.Context(0)
    ctx.ensure_workspace(d)
    coef, norm, idx = new((B, ci, N)), new((B, N)), new((B, k), torch.int32)
    xc, yc, y, a = new((B, ci, k), torch.int8), new((B, co, k)), new((B, co, H, W)), new((1,))
    ctx.wcc_haar_fwd(d, x, coef, norm)
    ctx.wcc_joint_topk(d, None, norm, idx)
    ctx.wcc_gather_quant(d, coef, idx, alpha, xc, a)
    ctx.wcc_pointwise(d, stored, scale, xc, a, yc)
    ctx.wcc_scatter_ihaar(d, yc, idx, y)
    ctx._ws.fill_(0x7E)
    y2, idx2, a2 = new((B, co, H, W)), new((B, k), torch.int32), new((1,))
    ctx.wcc_forward(d, x, stored, scale, alpha, y2, idx2, a2)
    torch.cuda.synchronize()
    assert torch.equal(idx, idx2) and torch.equal(a, a2)
    assert torch.equal(y, y2)
    form = "bytes" if case in BYTES else "words"
    assert codes_in_workspace(ctx, xc) == form
    if W % 4 == 0:
        dh = wcc.make_desc(B, ci, co, H, W, lv, num, den, wt, 8, wcc.BF16)
        ctx.ensure_workspace(dh)
        y3 = torch.empty((B, co, H, W), dtype=torch.bfloat16, device="cuda")
        ctx._ws.fill_(0x7E)
        ctx.wcc_forward(dh, x.bfloat16(), stored, scale, alpha, y3, idx2, a2)
        torch.cuda.synchronize()
        assert torch.equal(idx, idx2) and torch.equal(y.bfloat16(), y3)
        assert codes_in_workspace(ctx, xc) == form
    ctx.close()
