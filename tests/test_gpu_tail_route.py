"""Which layers run contraction and inverse as one kernel (needs an MI355X): both sides of every line of the rule, each at a
shape where the other route was measured the slower one.  The stage times say which ran: the contraction's bracket is
exactly 0 where it has no kernel of its own."""
import pytest
import torch

from paper_2205_12268_amd import wcc

pytestmark = pytest.mark.gpu

# one kernel?, B, C_in, C_out, H, W, keep, weights, bits, maps
FEW_OUT = [
    (False, 8, 16, 4, 512, 2048, (1, 2), wcc.BF16, 8, wcc.F32),
    (False, 4, 64, 8, 512, 1024, (1, 1), wcc.BF16, 8, wcc.F32),
    (False, 4, 64, 17, 512, 1024, (1, 2), wcc.BF16, 8, wcc.F32),
    (False, 4, 64, 32, 512, 1024, (1, 2), wcc.BF16, 8, wcc.F32),
    (False, 5, 32, 41, 432, 608, (1, 4), wcc.BF16, 8, wcc.F32),
    (True, 7, 32, 33, 424, 576, (1, 1), wcc.BF16, 8, wcc.F32),
    (True, 13, 8, 35, 760, 352, (1, 3), wcc.I4, 8, wcc.F32),
    (True, 9, 16, 48, 184, 576, (1, 2), wcc.I4, 8, wcc.F32),
    (True, 4, 16, 96, 256, 512, (1, 4), wcc.BF16, 8, wcc.F32),
    (True, 4, 64, 256, 512, 1024, (1, 8), wcc.BF16, 8, wcc.F32),
]
# X in two steps: a unit that keeps more than the LDS holds stages it again for every block
TWO_STEPS = [
    (False, 3, 80, 160, 376, 640, (3, 5), wcc.I4, 8, wcc.F32),
    (False, 10, 128, 224, 600, 128, (3, 4), wcc.I8, 8, wcc.F32),
    (False, 4, 20, 128, 256, 512, (3, 4), wcc.F32, 8, wcc.F32),
    (False, 15, 128, 66, 312, 256, (1, 2), wcc.I8, 8, wcc.F32),
    (False, 3, 128, 66, 616, 736, (1, 1), wcc.I8, 8, wcc.F32),    # all kept, rows that are not whole lines
    (True, 3, 64, 369, 752, 288, (3, 4), wcc.BF16, 8, wcc.F32),    # one step
    (True, 6, 88, 335, 152, 1024, (1, 2), wcc.I4, 8, wcc.F32),
    (True, 5, 30, 61, 400, 352, (1, 2), wcc.F32, 0, wcc.F32),
    (True, 5, 64, 48, 592, 832, (1, 3), wcc.I8, 8, wcc.F32),
    (True, 4, 80, 48, 768, 416, (1, 4), wcc.I4, 8, wcc.F32),
]
# little kept: bf16 maps, and fewer than eight channels
LITTLE = [
    (False, 5, 12, 272, 232, 768, (1, 16), wcc.I8, 8, wcc.BF16),
    (False, 2, 6, 89, 712, 960, (1, 6), wcc.BF16, 8, wcc.BF16),
    (False, 11, 128, 128, 392, 256, (1, 8), wcc.I4, 8, wcc.BF16),
    (False, 6, 1, 170, 304, 480, (1, 10), wcc.F32, 0, wcc.F32),
    (False, 2, 6, 248, 456, 928, (1, 10), wcc.F32, 0, wcc.F32),
    (False, 4, 8, 112, 624, 736, (1, 16), wcc.I4, 8, wcc.F32),
    (False, 14, 16, 373, 360, 128, (1, 16), wcc.F32, 0, wcc.F32),
    (True, 5, 8, 198, 336, 992, (1, 10), wcc.I8, 8, wcc.F32),
    (True, 6, 52, 144, 136, 960, (1, 5), wcc.I8, 8, wcc.BF16),
    (True, 7, 112, 69, 280, 576, (1, 3), wcc.I4, 8, wcc.BF16),
    (True, 5, 64, 147, 552, 896, (1, 16), wcc.BF16, 8, wcc.F32),
    (True, 1, 4, 77, 864, 1120, (1, 3), wcc.BF16, 8, wcc.F32),
]


@pytest.mark.parametrize("case", FEW_OUT + TWO_STEPS + LITTLE, ids=lambda c: "x".join(map(str, c)))
def test_route(case):
    one, B, ci, co, H, W, (num, den), wt, bits, maps = case
    d = wcc.make_desc(B, ci, co, H, W, 3, num, den, wt, bits, maps)
    ctx = wcc.Context(0)
    ctx.ensure_workspace(d)
    t = torch.bfloat16 if maps == wcc.BF16 else torch.float32
    x, y = (torch.zeros((B, c, H, W), dtype=t, device="cuda") for c in (ci, co))
    wd = {wcc.F32: torch.float32, wcc.BF16: torch.bfloat16}.get(wt, torch.int8)
    w = torch.zeros((co, ci // 2 if wt == wcc.I4 else ci), dtype=wd, device="cuda")
    ctx.set_profiling(True)
    ctx.wcc_forward(d, x, w, torch.ones(co, device="cuda") if wt in (wcc.I8, wcc.I4) else None, 0.0, y)
    ms = ctx.stage_times()
    assert ms["scatter_ihaar"] > 0 and (ms["pointwise"] == 0) == one
    ctx.close()
