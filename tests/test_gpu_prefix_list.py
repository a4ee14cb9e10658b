"""The fixed list of the first k positions, which the keep pass and the inverse read off the positions themselves, against
the same list given by the caller, which goes through a rank map (needs an MI355X): bit for bit, at one to four
levels, rows with idle lanes, bf16 maps, with and without the quantiser, with the caller's alpha (whose launch stays)."""
import pytest
import torch

from paper_2205_12268_amd import wcc

pytestmark = pytest.mark.gpu

# B, C_in, C_out, H, W, levels, keep, weights, bits, alpha, bf16 maps
CASES = [
    (1, 3, 5, 2, 2, 1, (1, 4), wcc.F32, 0, 0.0, False),
    (2, 8, 12, 16, 26, 1, (2, 5), wcc.BF16, 8, 0.0, False),
    (2, 16, 24, 36, 96, 2, (1, 3), wcc.I8, 8, 0.0, True),
    (1, 24, 40, 64, 256, 3, (1, 8), wcc.BF16, 8, 0.0, False),     # waves of a workgroup share a unit's ranks
    (2, 32, 48, 64, 320, 3, (1, 4), wcc.F32, 0, 0.0, True),       # lanes of all strips follow each other
    (1, 16, 32, 128, 128, 3, (9, 10), wcc.BF16, 8, 0.0, False),   # more positions a strip than a list holds
    (1, 16, 8, 32, 64, 4, (1, 16), wcc.BF16, 8, 0.0, False),
    (1, 16, 8, 48, 80, 4, (1, 1), wcc.I8, 0, 0.0, False),
    (2, 16, 24, 32, 64, 3, (1, 4), wcc.I8, 8, 2.5, False),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_prefix_is_the_list_of_the_first_positions(case):
    B, ci, co, H, W, lv, (num, den), wt, bits, alpha, half = case
    gen = torch.Generator(device="cuda")
    gen.manual_seed(H * W + ci)
    x = torch.randn((B, ci, H, W), generator=gen, device="cuda")
    x = x.bfloat16() if half else x
    w = torch.randn((co, ci), generator=gen, device="cuda")
    scale = None
    if wt == wcc.BF16:
        w = w.bfloat16()
    elif wt == wcc.I8:
        w, scale = (w * 40).clamp(-127, 127).to(torch.int8), torch.rand(co, generator=gen, device="cuda") + 0.5
    d = wcc.make_desc(B, ci, co, H, W, lv, num, den, wt, bits, wcc.BF16 if half else wcc.F32)
    k = wcc.k_of(d)
    idx = torch.arange(k, dtype=torch.int32, device="cuda").repeat(B, 1).contiguous()
    ctx = wcc.Context(0)
    ctx.ensure_workspace(d)
    got = []
    for given in (None, idx, None):
        ctx._ws.fill_(0x7E)
        y = torch.full((B, co, H, W), float("nan"), dtype=x.dtype, device="cuda")
        a = torch.zeros(1, device="cuda")
        ctx.wcc_forward_fixed(d, x, w, scale, alpha, given, y, a if bits else None)
        got.append((y, a))
    torch.cuda.synchronize()
    assert torch.isfinite(got[1][0].float()).all()
    for y, a in (got[0], got[2]):
        assert torch.equal(y, got[1][0]) and torch.equal(a, got[1][1])
    ctx.close()
