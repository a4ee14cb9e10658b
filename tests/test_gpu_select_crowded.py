"""The two-launch selection of planes whose norms lie close together or are equal, so that one of its digits would hold
more keys than its second kernel keeps in LDS (needs an MI355X): the sample's own keys then part it.  Index sets against a
host sort, norms summed from one to many planes of partial norms, the largest
kept coefficient, and the time, which such a plane shares with any other of its size."""
import numpy as np
import pytest
import torch

from paper_2205_12268_amd import wcc

pytestmark = pytest.mark.gpu

KINDS = {
    "equal": lambda r, n: np.full(n, 0x40490FDB, np.uint32),
    "blank": lambda r, n: np.where(np.arange(n) < n // 4, 0x43000000, 0).astype(np.uint32),
    "mostly": lambda r, n: np.where(r.random(n) < 0.6, 0x42C80000, 0x42C80000 + r.integers(-(1 << 16), 1 << 16, n)).astype(np.uint32),
    "few": lambda r, n: (0x3F800000 + 77 * r.integers(0, 5, n)).astype(np.uint32),
    "ulps": lambda r, n: (0x3F800000 + r.integers(0, 600, n)).astype(np.uint32),
    "across": lambda r, n: (0x40000000 + r.integers(-900, 900, n)).astype(np.uint32),        # two octaves
    "sorted": lambda r, n: np.sort(0x3F800000 + r.integers(0, 1 << 16, n)).astype(np.uint32),
    "noise": lambda r, n: (100 + 0.5 * r.normal(0, 1, n)).astype(np.float32).view(np.uint32),
    "tiny": lambda r, n: r.integers(1, 0x20000000, n).astype(np.uint32),                     # all below 2^-32
    "ends": lambda r, n: r.choice(np.array([0, 1, 0x7F7FFFFF, 0x7F800000], np.uint32), n),
}


@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("B,H,W", [(2, 2, 8194), (1, 128, 256), (3, 250, 262), (2, 256, 514), (8, 512, 514), (1, 1024, 1024)])
def test_crowded_planes(B, H, W, kind):
    N = H * W
    rng = np.random.default_rng(N + sum(map(ord, kind)))
    key = np.stack([KINDS[kind](rng, N) for _ in range(B)])
    norm = torch.from_numpy(key.view(np.float32)).cuda()
    order = [np.lexsort((np.arange(N), -key[b].astype(np.int64))) for b in range(B)]
    ctx = wcc.Context(0)
    for k in sorted({1, N // 16, N // 4, N // 4 + 1, N // 2, N - 1}):
        d = wcc.make_desc(B, 16, 16, H, W, 1, k, N, wcc.F32, 0)
        ctx.ensure_workspace(d)
        ctx._ws.fill_(0x7E)
        idx = torch.full((B, k), -7, dtype=torch.int32, device="cuda")
        ctx.wcc_joint_topk(d, None, norm, idx)
        got = idx.cpu().numpy()
        for b in range(B):
            np.testing.assert_array_equal(got[b], np.sort(order[b][:k]))
    ctx.close()


# One pixel of four is not zero: at one level all four bands of a 2 x 2 square hold the same magnitude, so a few amplitudes
# give a few norms to the whole plane.  Amplitudes are multiples of 1/512 below 2: norms and sums are exact in any order.
@pytest.mark.parametrize("amplitudes", [1, 2, 40])
@pytest.mark.parametrize("C", [4, 8, 16, 32, 64, 128])  # 1 to 32 planes of partial norms
@pytest.mark.parametrize("H,W", [(128, 160), (192, 340)])
def test_crowded_layers(C, H, W, amplitudes):
    B, co, N = 2, 24, H * W
    gen = torch.Generator(device="cuda")
    gen.manual_seed(C + W + amplitudes)
    a = 1 + torch.randint(0, amplitudes, (B, 1, H // 2, W // 2), generator=gen, device="cuda").float() / 512
    x = torch.zeros((B, C, H, W), device="cuda")
    x[:, :, ::2, ::2] = a * torch.tensor([1.0, 2.0, 0.5], device="cuda").repeat(C)[:C].view(1, C, 1, 1)
    w = torch.randint(-7, 8, (co, C), generator=gen, device="cuda").bfloat16()
    ctx = wcc.Context(0)
    for num, den in ((1, 8), (5, 9)):
        d = wcc.make_desc(B, C, co, H, W, 1, num, den, wcc.BF16, 8)
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
        assert len(np.unique(bits)) <= amplitudes
        for b in range(B):
            want = np.sort(np.lexsort((np.arange(N), -bits[b]))[:k])
            np.testing.assert_array_equal(idx[b].cpu().numpy(), want)
            np.testing.assert_array_equal(idx2[b].cpu().numpy(), want)
        assert torch.equal(alpha, alpha2) and torch.equal(y, y2)
    ctx.close()


# Digits read from memory by every workgroup took such planes 5 to 24 times as long as others; they take 1.1 to 2.
@pytest.mark.parametrize("kind", ["equal", "few", "noise", "blank"])
@pytest.mark.parametrize("B,H,W", [(1, 256, 512), (1, 512, 1024)])
def test_crowded_planes_take_about_as_long(B, H, W, kind):
    N = H * W
    rng = np.random.default_rng(5)
    d = wcc.make_desc(B, 16, 16, H, W, 1, 1, 8, wcc.F32, 0)
    ctx = wcc.Context(0)
    ctx.ensure_workspace(d)
    idx = torch.empty((B, wcc.k_of(d)), dtype=torch.int32, device="cuda")

    def micros(key):
        norm = torch.from_numpy(np.stack([key] * B).view(np.float32)).cuda()
        times = []
        for _ in range(9):
            start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            start.record()
            for _ in range(20):
                ctx.wcc_joint_topk(d, None, norm, idx)
            end.record()
            torch.cuda.synchronize()
            times.append(start.elapsed_time(end) * 50)
        return min(times)

    spread = micros(np.exp(rng.normal(3.0, 1.0, N)).astype(np.float32).view(np.uint32))
    assert micros(KINDS[kind](rng, N)) < 2.5 * spread
    ctx.close()
