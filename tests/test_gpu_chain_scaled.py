"""The chained block carries powers of two through its transforms instead of the butterflies' halves (needs an MI355X).
A block without a quantiser on inputs scaled by a power of two gives that power times its result, bit for bit, and keeps
the same positions.  (That the powers of the levels cancel, test_gpu_chain_range.py compares with the other route.)"""
import pytest
import torch

from paper_2205_12268_amd import wcc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("norm", [wcc.NORM_L1, wcc.NORM_L2])
@pytest.mark.parametrize("H,W,levels", [(16, 20, 2), (32, 64, 3), (24, 96, 3), (8, 512, 3), (16, 256, 1)])
def test_powers_of_two_pass_through(H, W, levels, norm):
    B, C, e = 2, 12, 3
    gen = torch.Generator(device="cuda")
    gen.manual_seed(H + W)
    x = torch.randn((B, C, H, W), generator=gen, device="cuda")
    w1 = torch.randn((C * e, C), generator=gen, device="cuda")
    w3 = torch.randn((C, C * e), generator=gen, device="cuda")
    wdw = torch.randn((C * e, 3, 3), generator=gen, device="cuda")
    d = wcc.make_block_desc(B, C, e, H, W, levels, 1, 4, wcc.F32, 0, wcc.F32, norm)
    assert wcc.block_is_chained(d)
    ctx = wcc.Context(0)
    ctx.ensure_workspace(d)
    k = -(-H * W // 4)
    # (squares stay normal numbers)
    results = []
    for power in (0, 40, -40):
        y = torch.full_like(x, float("nan"))
        i1, i3 = (torch.full((B, k), -7, dtype=torch.int32, device="cuda") for _ in range(2))
        ctx.wcc_block_forward(d, x * 2.0 ** power, w1, None, wdw, w3, None, y, None, None, i1, i3)
        torch.cuda.synchronize()
        results.append((y * 2.0 ** -power, i1, i3))
    assert torch.isfinite(results[0][0]).all()
    for r in results[1:]:
        assert all(torch.equal(a, b) for a, b in zip(r, results[0]))
    ctx.close()
