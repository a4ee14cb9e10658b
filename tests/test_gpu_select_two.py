"""The selection of planes above 16384 positions in two launches (needs an MI355X): its digits (zero alone, 64
steps an octave between 2^-32 and 2^32, the rest in the first and last step), digits whose keys fit in LDS (32768)
or are read from memory, classes of equal keys, one and several chunks of 4096, 8192 and 16384 positions, the
largest plane it takes and the next one, which the four launches take.  The tables say into which chunks a
plane was cut, and where they lie, in the memory of the histograms or of Y_wt."""
import numpy as np
import pytest
import torch

from paper_2205_12268_amd import wcc

pytestmark = pytest.mark.gpu

KINDS = {
    "equal": lambda r, n: np.full(n, 0x40490FDB, np.uint32),
    "zeros": lambda r, n: np.where(r.random(n) < 0.7, 0, r.integers(0x3F000000, 0x42000000, n)).astype(np.uint32),
    "two": lambda r, n: np.where(r.random(n) < 0.5, 0x3F800000, 0x3F800001).astype(np.uint32),
    "step": lambda r, n: (0x3F800000 + r.integers(0, 1 << 17, n)).astype(np.uint32),         # all with one digit
    "step_ties": lambda r, n: (0x3F800000 + 4096 * r.integers(0, 32, n)).astype(np.uint32),
    "norms": lambda r, n: np.exp(r.normal(3.0, 1.0, n)).astype(np.float32).view(np.uint32),
    "smooth": lambda r, n: (100 + 50 * np.sin(np.arange(n) / 777.0)).astype(np.float32).view(np.uint32),
    "tiny": lambda r, n: r.integers(0, 0x20000000, n).astype(np.uint32),                     # below 2^-32 mostly
    "huge": lambda r, n: r.integers(0x4F000000, 0x7F800000, n).astype(np.uint32),            # above 2^31 mostly
    "noise": lambda r, n: (100 + 3 * r.normal(0, 1, n)).astype(np.float32).view(np.uint32),    # close together
    "any": lambda r, n: r.integers(0, 0x7F800001, n).astype(np.uint32),
}


def check(B, H, W, kind, ks):
    N = H * W
    rng = np.random.default_rng(N + sum(map(ord, kind)))
    key = np.stack([KINDS[kind](rng, N) for _ in range(B)])
    norm = torch.from_numpy(key.view(np.float32)).cuda()
    ctx = wcc.Context(0)
    order = [np.lexsort((np.arange(N), -key[b].astype(np.int64))) for b in range(B)]
    for k in ks:
        d = wcc.make_desc(B, 1, 1, H, W, 1, k, N, wcc.F32, 0)
        assert wcc.k_of(d) == k
        ctx.ensure_workspace(d)
        idx = torch.full((B, k), -7, dtype=torch.int32, device="cuda")
        ctx.wcc_joint_topk(d, None, norm, idx)
        got = idx.cpu().numpy()
        for b in range(B):
            np.testing.assert_array_equal(got[b], np.sort(order[b][:k]))
    ctx.close()


@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("H,W", [(2, 8194), (128, 130), (100, 212), (128, 256), (256, 514)])
def test_two_launch_selection(H, W, kind):
    N = H * W
    check(2, H, W, kind, sorted({1, 2, 4096, 8191, N // 8 + 1, N // 3, N // 2, N - 1, N}))


@pytest.mark.parametrize("kind", ["equal", "zeros", "step", "two", "norms", "smooth", "noise", "huge", "any"])
@pytest.mark.parametrize("B,H,W", [
    (8, 256, 514),      # 8192 positions a chunk
    (8, 512, 514),      # 16384 positions a chunk
    (1, 1024, 1024),    # the largest plane (128 chunks of 8192: Y_wt of one channel holds no more tables)
    (1, 1024, 1026),    # four launches
    (17, 512, 514),     # too many chunks: four launches
])
def test_two_launch_selection_chunks(B, H, W, kind):
    N = H * W
    check(B, H, W, kind, [1, N // 8 + 1, N // 2, N])


DIGITS = 4096  # 16-bit counts a chunk in the tables, the first of a row that of all its keys


def chunks_of_tables(ctx, d, in_yc):
    """Keys of the first sample's chunks as the tables have them, at the start of Y_wt's memory, the workspace's last, or of
    the histograms', behind a plane of partial norms and one of norms."""
    lines = lambda n: -(-n // 256) * 256
    yc = ctx._ws.numel() - lines(d.B * d.C_out * (-(-wcc.k_of(d) // 4) * 4) * 4)
    at = yc if in_yc else 2 * lines(d.B * d.H * d.W * 4)
    return ctx._ws[at:at + 2 * DIGITS * 256].view(torch.uint16).view(-1, DIGITS)[:, 0].cpu().numpy().astype(int)


@pytest.mark.parametrize("kind", ["equal", "norms", "smooth", "noise", "any"])
@pytest.mark.parametrize("B,H,W,co,chunk,in_yc", [
    (1, 1024, 1024, 32, 4096, True),   # 256 chunks, the largest plane
    (1, 1022, 1026, 32, 4096, True),   # 256, the last one short
    (2, 512, 1024, 32, 4096, True),    # 128 a sample
    (2, 512, 1020, 16, 4096, False),   # 128, the last one short
    (2, 1024, 1024, 32, 8192, True),
    (4, 512, 1022, 32, 8192, True),    # 64 a sample, the last one short
    (7, 512, 514, 24, 8192, False),    # 33, the last one of 1024 keys
    (8, 512, 770, 24, 16384, False),   # 25, the last one of 1024 keys
])
def test_two_launch_selection_tables(B, H, W, co, chunk, in_yc, kind):
    N = H * W
    rng = np.random.default_rng(N + co)
    key = np.stack([KINDS[kind](rng, N) for _ in range(B)])
    norm = torch.from_numpy(key.view(np.float32)).cuda()
    order = [np.lexsort((np.arange(N), -key[b].astype(np.int64))) for b in range(B)]
    sizes = [chunk] * (N // chunk) + ([N % chunk] if N % chunk else [])
    ctx = wcc.Context(0)
    for k in (N // 16, N // 3 + 1, N - 5):
        d = wcc.make_desc(B, 4, co, H, W, 1, k, N, wcc.F32, 0)
        ctx.set_workspace(torch.full((wcc.workspace_bytes(d),), 0x7E, dtype=torch.uint8, device="cuda"))
        idx = torch.full((B, k), -7, dtype=torch.int32, device="cuda")
        ctx.wcc_joint_topk(d, None, norm, idx)
        got = idx.cpu().numpy()
        for b in range(B):
            np.testing.assert_array_equal(got[b], np.sort(order[b][:k]))
        np.testing.assert_array_equal(chunks_of_tables(ctx, d, in_yc)[:len(sizes)], sizes)
    ctx.close()


# Fused layers in chunks of 8192 and 16384: the rank map and the largest kept coefficient as well.  Dyadic maps: exact norms.
@pytest.mark.parametrize("B,H,W", [(3, 512, 1024), (8, 512, 768)])
def test_fused_layers_of_large_chunks(B, H, W):
    C, co, N = 8, 24, H * W
    gen = torch.Generator(device="cuda")
    gen.manual_seed(W)
    x = torch.randint(-63, 64, (B, C, H, W), generator=gen, device="cuda").float() / 8
    x *= torch.rand((B, 1, H, W), generator=gen, device="cuda") < 0.6
    w = torch.randint(-7, 8, (co, C), generator=gen, device="cuda").bfloat16()
    for num, den in ((1, 8), (2, 3)):
        d = wcc.make_desc(B, C, co, H, W, 2, num, den, wcc.BF16, 8)
        k = wcc.k_of(d)
        ctx = wcc.Context(0)
        ctx.ensure_workspace(d)
        ctx._ws.fill_(0x7E)
        new = lambda shape, dtype=torch.float32: torch.full(shape, -7, dtype=dtype, device="cuda")
        y, idx, alpha = new((B, co, H, W)), new((B, k), torch.int32), new((1,))
        ctx.wcc_forward(d, x, w, None, 0.0, y, idx, alpha)
        coef, norm = new((B, C, N)), new((B, N))
        ctx.wcc_haar_fwd(d, x, coef, norm)
        bits = norm.cpu().numpy().view(np.uint32).astype(np.int64)
        for b in range(B):
            np.testing.assert_array_equal(idx[b].cpu().numpy(), np.sort(np.lexsort((np.arange(N), -bits[b]))[:k]))
        xc, yc, y2, alpha2 = new((B, C, k), torch.int8), new((B, co, k)), new((B, co, H, W)), new((1,))
        ctx.wcc_gather_quant(d, coef, idx, 0.0, xc, alpha2)
        ctx.wcc_pointwise(d, w, None, xc, alpha2, yc)
        ctx.wcc_scatter_ihaar(d, yc, idx, y2)
        torch.cuda.synchronize()
        assert torch.equal(alpha, alpha2) and torch.equal(y, y2)
        ctx.close()


# ... and from several planes of partial norms, which only K_dw in front leaves on planes of this size: chained blocks.  Small
# integers throughout, so the norms are exact however they are summed.
@pytest.mark.parametrize("B", [3, 5])  # chunks of 8192, 16384
def test_chained_blocks_of_large_chunks(B):
    C, e, H, W = 4, 4, 512, 1024
    N, k = H * W, H * W // 4
    gen = torch.Generator(device="cuda")
    gen.manual_seed(B)
    ints = lambda *s: torch.randint(-1, 2, s, generator=gen, device="cuda").float()
    x, w1, w3, wdw = ints(B, C, H, W), ints(C * e, C), ints(C, C * e), ints(C * e, 3, 3)
    d = wcc.make_block_desc(B, C, e, H, W, 3, 1, 4, wcc.F32, 0)
    assert wcc.block_is_chained(d)
    ctx = wcc.Context(0)
    ctx.ensure_workspace(d)
    ctx._ws.fill_(0x7E)
    y, y2 = (torch.full_like(x, float("nan")) for _ in range(2))
    i3, j3 = (torch.full((B, k), -7, dtype=torch.int32, device="cuda") for _ in range(2))
    t2 = torch.empty((B, C * e, H, W), device="cuda")
    ctx.wcc_block_forward(d, x, w1, None, wdw, w3, None, y, None, None, None, i3)
    ctx.wcc_block_forward(d, x, w1, None, wdw, w3, None, y2, None, t2, None, j3)
    dl = wcc.make_desc(B, C * e, C, H, W, 3, 1, 4, wcc.F32, 0)
    coef, norm = torch.empty((B, C * e, N), device="cuda"), torch.empty((B, N), device="cuda")
    ctx.ensure_workspace(dl)
    ctx.wcc_haar_fwd(dl, t2, coef, norm)
    bits = norm.cpu().numpy().view(np.uint32).astype(np.int64)
    for b in range(B):
        np.testing.assert_array_equal(i3[b].cpu().numpy(), np.sort(np.lexsort((np.arange(N), -bits[b]))[:k]))
    assert torch.equal(i3, j3) and torch.equal(y, y2)
    ctx.close()
