"""The two ways to a layer's channel norms (needs an MI355X): the norm-only pass of wcc_forward and the storing
pass of wcc_haar_fwd, which on large maps, and on middling ones of few strip units, gives the parts of a
channel group launch rows and planes of their own.  Both add in one order, so the index sets agree on any input; the storing pass stays
inside its buffers; the norm-only pass reads inputs over 256 MB past the cache, with 8 and 16 waves a unit."""
import numpy as np
import pytest
import torch

from paper_2205_12268_amd import wcc

pytestmark = pytest.mark.gpu

# B, C, H, W, levels
SHAPES = [
    (6, 432, 56, 504, 3),    # 293 MB: two groups of eight parts
    (1, 1030, 72, 504, 3),   # 150 MB: eight groups, the last one short, of eight ragged parts
    (1, 1024, 96, 352, 2),   # 138 MB: sixteen parts, rows that run on from strip to strip
    (2, 260, 128, 128, 2),   # 34 MB in 32 units: two groups of sixteen parts, the last ones short
    (4, 96, 384, 320, 3),    # 189 MB, too few channels for planes of their own: waves share a unit
    (2, 100, 32, 64, 1),     # small: shared units, several groups
    (2, 200, 24, 40, 3),
    (1, 200, 96, 96, 4),
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_staged_and_fused_selection_agree_where_rounding_decides(shape):
    """Every block of 2^d x 2^d pixels holds one of the same C values in each channel, in an order of its own:
    the norms of the coarsest band are sums of the same numbers in different orders, equal but for their
    rounding, and half of them are kept."""
    B, C, H, W, lv = shape
    h, w = H >> lv, W >> lv
    gen = torch.Generator(device="cuda")
    gen.manual_seed(C + W)
    v = torch.rand(C, generator=gen, device="cuda") + 0.1
    x = torch.empty((B, C, H, W), device="cuda")
    for b in range(B):
        order = torch.rand((C, h, w), generator=gen, device="cuda").argsort(dim=0)
        x[b] = v[order].repeat_interleave(1 << lv, dim=1).repeat_interleave(1 << lv, dim=2)
    N, k = H * W, h * w // 2
    d = wcc.make_desc(B, C, 4, H, W, lv, k, N, wcc.F32, 0)
    ctx = wcc.Context(0)
    ctx.ensure_workspace(d)
    coef, norm = torch.empty((B, C, N), device="cuda"), torch.empty((B, N), device="cuda")
    ctx.wcc_haar_fwd(d, x, coef, norm)
    for b in range(B):
        assert torch.equal(norm[b, h * w:], torch.zeros(N - h * w, device="cuda"))
        assert torch.unique(norm[b, :h * w]).numel() > 1      # rounding does decide
    staged, fused = (torch.full((B, k), -7, dtype=torch.int32, device="cuda") for _ in range(2))
    ctx.wcc_joint_topk(d, None, norm, staged)
    y = torch.empty((B, 4, H, W), device="cuda")
    ctx.wcc_forward(d, x, torch.ones((4, C), device="cuda"), None, 0.0, y, fused)
    assert torch.equal(staged, fused)
    ctx.close()


def wavelet_vectors(x, levels):
    """[..., N] of [..., H, W], the coarsest bands first."""
    details = []
    for _ in range(levels):
        a, b, c, d = x[..., 0::2, 0::2], x[..., 0::2, 1::2], x[..., 1::2, 0::2], x[..., 1::2, 1::2]
        details.append([(a - b + c - d) / 2, (a + b - c - d) / 2, (a - b - c + d) / 2])
        x = (a + b + c + d) / 2
    return torch.cat([t.flatten(-2) for t in [x] + [t for lev in reversed(details) for t in lev]], dim=-1)


def dyadic(shape, seed):
    """Multiples of 1/8 below 4: every coefficient and every sum here is exact in fp32, in any order."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return torch.randint(0, 32, shape, generator=gen, device="cuda").float() / 8.0


@pytest.mark.parametrize("keep", [(1, 4), (1, 1024)])
@pytest.mark.parametrize("shape", SHAPES[:4], ids=lambda s: "x".join(map(str, s)))
def test_storing_pass_stays_inside_its_buffers(shape, keep):
    """A workspace of exactly the bytes asked for: with a quarter kept it holds the planes of the parts, with
    1/1024 kept it does not (and waves share a unit again)."""
    B, C, H, W, lv = shape
    N = H * W
    x = dyadic((B, C, H, W), C)
    d = wcc.make_desc(B, C, 4, H, W, lv, *keep, wcc.F32, 0)
    need = wcc.workspace_bytes(d)
    ws = torch.full((need + 4096,), 255, dtype=torch.uint8, device="cuda")
    ctx = wcc.Context(0)
    ctx.set_workspace(ws[:need])
    coef = torch.full((B * C * N + 1024,), float("nan"), device="cuda")
    norm = torch.full((B * N + 1024,), float("nan"), device="cuda")
    ctx.wcc_haar_fwd(d, x, coef[:B * C * N].view(B, C, N), norm[:B * N].view(B, N))
    assert bool((ws[need:] == 255).all())
    assert bool(torch.isnan(coef[B * C * N:]).all()) and bool(torch.isnan(norm[B * N:]).all())
    for b in range(B):
        want = wavelet_vectors(x[b], lv)
        assert torch.equal(coef[:B * C * N].view(B, C, N)[b], want)
        assert torch.equal(norm[:B * N].view(B, N)[b], want.double().abs().sum(dim=0).float())
    ctx.close()


@pytest.mark.parametrize("shape", [(6, 432, 56, 512, 3), (1, 1024, 96, 704, 2)], ids=lambda s: "x".join(map(str, s)))
def test_streamed_norm_pass_with_shared_units(shape):
    """Inputs over 256 MB whose rows are whole lines: 8 waves a unit, two groups; 16 waves a unit, rows that run on
    from strip to strip."""
    B, C, H, W, lv = shape
    N = H * W
    k = N // 8
    x = dyadic((B, C, H, W), C + 1)
    w = torch.randint(-8, 9, (4, C), device="cuda").float() / 8.0
    d = wcc.make_desc(B, C, 4, H, W, lv, 1, 8, wcc.F32, 0)
    ctx = wcc.Context(0)
    ctx.ensure_workspace(d)
    y = torch.full((B, 4, H, W), float("nan"), device="cuda")
    idx = torch.full((B, k), -7, dtype=torch.int32, device="cuda")
    ctx.wcc_forward(d, x, w, None, 0.0, y, idx)
    for b in range(B):
        c = wavelet_vectors(x[b], lv).double()
        want = torch.sort(c.abs().sum(dim=0), descending=True, stable=True).indices[:k].sort().values
        assert torch.equal(idx[b].long(), want)
        z = torch.zeros((4, N), dtype=torch.float64, device="cuda")
        z[:, want] = w.double() @ c[:, want]
        got = wavelet_vectors(y[b].double(), lv)
        # fp32 sums of at most 1024 exact terms, then at most three levels of the inverse
        assert float((got - z).norm() / z.norm()) <= 1e-6
    ctx.close()
