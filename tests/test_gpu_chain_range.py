"""The chained block against the route that forms the middle tensors (needs an MI355X), bit for bit: the powers of two that
its transforms carry along must cancel at every level, for both norms, and must not take anything off the range of
fp32.  With four middle channels both routes add a position's norm in one group, in the order of the channels, so norms
and index sets are the same bits.  The 3x3 kernels are scaled until the largest norm lies just below 2^127, and down as
far as squares and sums stay normal numbers; the project weights take the power back."""
import math

import pytest
import torch

from paper_2205_12268_amd import wcc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("norm", [wcc.NORM_L1, wcc.NORM_L2])
@pytest.mark.parametrize("H,W,levels", [(16, 256, 1), (14, 260, 1), (16, 20, 2), (12, 776, 2), (32, 64, 3), (24, 96, 3), (16, 512, 3)])
def test_powers_of_two_up_to_the_largest_norm(H, W, levels, norm):
    B, C, e = 2, 2, 2
    N, k = H * W, -(-H * W // 4)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(H + W + levels)
    x = torch.randn((B, C, H, W), generator=gen, device="cuda")
    w1 = torch.randn((C * e, C), generator=gen, device="cuda")
    w3 = torch.randint(1, 8, (C, C * e), generator=gen, device="cuda").float()  # (exact times any power of two)
    wdw = torch.randn((C * e, 3, 3), generator=gen, device="cuda")
    wdw[0] = 0.0
    wdw[0, 1, 1] = 1.0
    d = wcc.make_block_desc(B, C, e, H, W, levels, 1, 4, wcc.F32, 0, wcc.F32, norm)
    assert wcc.block_is_chained(d)
    ctx = wcc.Context(0)
    ctx.ensure_workspace(d)

    def run(power, formed):
        y, t2 = torch.full_like(x, float("nan")), torch.full((B, C * e, H, W), float("nan"), device="cuda")
        i1, i3 = (torch.full((B, k), -7, dtype=torch.int32, device="cuda") for _ in range(2))
        ctx.wcc_block_forward(d, x, w1, None, wdw * 2.0 ** power, w3 * 2.0 ** -power, None, y, None, t2 if formed else None, i1, i3)
        torch.cuda.synchronize()
        return y, i1, i3, t2

    y, i1, i3, t2 = run(0, True)
    dl = wcc.make_desc(B, C * e, C, H, W, levels, 1, 4, wcc.F32, 0, wcc.F32, norm)
    coef, nrm = torch.empty((B, C * e, N), device="cuda"), torch.empty((B, N), device="cuda")
    ctx.ensure_workspace(dl)
    ctx.wcc_haar_fwd(dl, t2, coef, nrm)
    top = 126 - math.floor(math.log2(float(nrm.max())))  # power of the largest norm
    powers = [0, top, -60] if norm == wcc.NORM_L1 else [0, top // 2, -20]
    ctx.ensure_workspace(d)
    assert torch.isfinite(y).all()
    for power in powers:
        for formed in (True, False):
            got = run(power, formed)
            assert torch.equal(got[2], i3), (power, formed)
            assert torch.equal(got[0], y) and torch.equal(got[1], i1), (power, formed)
    ctx.close()
