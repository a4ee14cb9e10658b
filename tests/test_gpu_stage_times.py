"""Stage times of a context that profiles one call after another (needs an MI355X): a stage that the last call did not run
takes no time, whatever ran before it."""
import pytest
import torch

from paper_2205_12268_amd import wcc

pytestmark = pytest.mark.gpu


def _call(ctx, d, fixed=False):
    ctx.ensure_workspace(d)
    x = torch.ones((d.B, d.C_in, d.H, d.W), device="cuda")
    w = torch.zeros((d.C_out, d.C_in), dtype=torch.bfloat16, device="cuda")
    y = torch.empty((d.B, d.C_out, d.H, d.W), device="cuda")
    if fixed:
        ctx.wcc_forward_fixed(d, x, w, None, 0.0, None, y)
    else:
        ctx.wcc_forward(d, x, w, None, 0.0, y)
    return ctx.stage_times()


def test_stages_are_the_last_calls():
    plain = wcc.make_desc(1, 32, 32, 64, 64, 2, 1, 4, wcc.BF16, 8)
    # few channels and 128 MiB of output coefficients: contraction and inverse are one kernel
    one_kernel = wcc.make_desc(4, 32, 128, 256, 512, 3, 1, 2, wcc.BF16, 8)
    ctx = wcc.Context(0)
    ctx.ensure_workspace(one_kernel)
    ctx.set_profiling(True)
    ran = ("haar_fwd", "norm_select", "gather", "pointwise", "scatter_ihaar")
    ms = _call(ctx, plain)
    assert all(ms[n] > 0 for n in ran) and ms["depthwise"] == 0
    ms = _call(ctx, one_kernel)
    assert ms["pointwise"] == 0
    assert all(ms[n] > 0 for n in ran if n != "pointwise")
    ms = _call(ctx, plain, fixed=True)
    assert ms["haar_fwd"] == 0
    assert all(ms[n] > 0 for n in ran if n != "haar_fwd")
    assert all(_call(ctx, plain)[n] > 0 for n in ran)
    ctx.close()
