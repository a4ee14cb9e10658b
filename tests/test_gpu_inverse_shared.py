"""The inverse where the four waves of a workgroup share a strip unit and pack one list of its kept positions (needs an
MI355X): three and four levels, channel groups that are uneven, units that keep nothing, units that keep more than a list
holds, a last unit that is not full, planes narrower and wider than a unit, both storage types, and the skip connection."""
import numpy as np
import pytest
import torch

from paper_2205_12268_amd import synth, wcc
from tests.util import dev, layer_with_index_set, rel_l2, upload_weights

pytestmark = pytest.mark.gpu

# B, C, H, W, levels, keep
CASES = [
    (1, 16, 8, 16, 3, (1, 3)),      # one unit, mostly outside the plane; four groups
    (2, 17, 64, 64, 3, (1, 3)),     # uneven groups
    (1, 33, 40, 104, 3, (1, 4)),    # units across strips, a last one that is not full
    (3, 67, 16, 1032, 3, (1, 8)),   # strips of several units
    (1, 18, 48, 40, 3, (1, 1920)),  # one position kept
    (2, 19, 64, 48, 4, (1, 3)),
    (1, 64, 48, 1040, 4, (1, 5)),
    (2, 19, 64, 48, 4, (1, 6)),     # four levels share up to a sixth kept
    (1, 64, 48, 1040, 4, (1, 8)),   # strips of several units
    (2, 17, 32, 32, 4, (1, 3)),     # half a unit, four levels
    (2, 18, 16, 16, 4, (1, 256)),   # one position kept, one unit mostly outside the plane
]


@pytest.mark.parametrize("shape", CASES, ids=lambda c: "x".join(map(str, c)))
def test_inverse(ref, shape):
    B, C, H, W, levels, (num, den) = shape
    N = H * W
    d = wcc.make_desc(B, 8, C, H, W, levels, num, den, wcc.F32, 0)
    d16 = wcc.make_desc(B, 8, C, H, W, levels, num, den, wcc.F32, 0, wcc.BF16)
    k = wcc.k_of(d)
    rng = np.random.default_rng(synth.SEED_BASE + 0x1600 + N + C)
    upper = np.zeros((1, 1, H, W))
    upper[:, :, :H // 3] = rng.standard_normal((H // 3, W))
    # everywhere; the upper rows first, whole units of them; the coarse positions; the fine ones
    lists = [np.sort(rng.permutation(N)[:k]),
             np.sort(np.argsort(ref.haar_fwd(upper, levels).reshape(N) == 0, kind="stable")[:k]), np.arange(k), np.arange(N - k, N)]
    ctx = wcc.Context(0)
    ctx.ensure_workspace(d)
    yc = rng.standard_normal((B, C, k)).astype(np.float32)
    x = dev(rng.integers(-32, 33, (B, 8, H, W)).astype(np.float32) / 8)
    w = dev(rng.standard_normal((C, 8)).astype(np.float32))
    flat = torch.empty((B * C * N + 4096,), device="cuda")
    y = flat[:B * C * N].view(B, C, H, W)
    y16 = torch.empty((B, C, H, W), dtype=torch.bfloat16, device="cuda")
    for n in range(len(lists)):
        print(shape, "list", n, flush=True)
        idx = np.stack([lists[(n + b) % 4] for b in range(B)])
        flat.fill_(float("nan"))
        ctx.wcc_scatter_ihaar(d, dev(yc), dev(idx.astype(np.int32)), y)
        want = ref.haar_inv(ref.scatter(yc, idx, N), H, W, levels)
        got = y.cpu().numpy()
        for b in range(B):
            assert rel_l2(got[b], want[b]) <= 1e-6
        assert torch.isnan(flat[B * C * N:]).all()
        # both storage types through the layer: the same numbers, rounded once
        ctx.wcc_forward_fixed(d, x, w, None, 0.0, dev(idx.astype(np.int32)), y)
        ctx.wcc_forward_fixed(d16, x.bfloat16(), w, None, 0.0, dev(idx.astype(np.int32)), y16)
        assert torch.equal(y16, y.bfloat16())


@pytest.mark.parametrize("keep", [(1, 2), (1, 1), (1, 4)])
@pytest.mark.parametrize("shape", [(2, 16, 128, 128), (1, 19, 72, 264)], ids=lambda c: "x".join(map(str, c)))
def test_with_skip_connection(shape, keep):
    """The block's second layer on its own adds nothing to the planes: with x added afterwards it is the block, bit for bit."""
    B, C, H, W = shape
    rng = np.random.default_rng(synth.SEED_BASE + 0x1700 + C)
    x = torch.from_numpy(rng.integers(-32, 33, (B, C, H, W)).astype(np.float32) / 8).cuda()
    w1, w3 = (dev(rng.standard_normal(s).astype(np.float32)) for s in ((2 * C, C), (C, 2 * C)))
    w_dw = dev(rng.standard_normal((2 * C, 3, 3)).astype(np.float32))
    d = wcc.make_block_desc(B, C, 2, H, W, 3, *keep, wcc.F32, 0)
    ctx = wcc.Context(0)
    ctx.ensure_workspace(d)
    t1, t2 = (torch.empty((B, 2 * C, H, W), device="cuda") for _ in range(2))
    y = torch.full_like(x, float("nan"))
    ctx.wcc_block_forward(d, x, w1, None, w_dw, w3, None, y, t1, t2)
    d3 = wcc.make_desc(B, 2 * C, C, H, W, 3, *keep, wcc.F32, 0)
    ctx3 = wcc.Context(0)
    ctx3.ensure_workspace(d3)
    branch = torch.full_like(x, float("nan"))
    ctx3.wcc_forward(d3, t2, w3, None, 0.0, branch)
    assert torch.equal(y, branch + x)


# levels, B, C, H, W, keep: shared at three levels, at four up to a quarter kept; last units that are not full
BLOCKS = [(3, 2, 16, 128, 128, (1, 2)), (3, 1, 20, 72, 264, (1, 1)), (3, 1, 32, 136, 96, (1, 5)),
          (4, 2, 16, 128, 128, (1, 4)), (4, 1, 20, 144, 272, (1, 8)), (4, 1, 32, 128, 128, (1, 2))]


@pytest.mark.parametrize("maps", [wcc.F32, wcc.BF16])
@pytest.mark.parametrize("shape", BLOCKS, ids=lambda c: "x".join(map(str, c)))
def test_skip_connection_against_oracle(ref, shape, maps):
    """The block's second layer in 64 bits from the first one's output as the call gives it and the call's own index set.
    fp32 maps: sums of 32 bits.  bf16 maps: each value is rounded once, by 2^-9 of it at most."""
    levels, B, C, H, W, keep = shape
    cfg = synth.BlockCfg("shared", B, C, 2, H, W, levels, *keep, synth.W_F32, 0, sigma=1.0,
                         seed=synth.SEED_BASE + 0x1780 + 16 * levels + C)
    print(cfg, maps, flush=True)
    x, w1, w_dw, w3 = synth.make_block_inputs(cfg)
    t = torch.bfloat16 if maps == wcc.BF16 else torch.float32
    xd = dev(x).to(t)
    d = wcc.make_block_desc(B, C, 2, H, W, levels, *keep, cfg.w_dtype, 0, maps)
    ctx = wcc.Context(0)
    ctx.ensure_workspace(d)
    flat = torch.full((x.size + 4096,), float("nan"), dtype=t, device="cuda")
    y = flat[:x.size].view(x.shape)
    t1 = torch.empty((B, 2 * C, H, W), dtype=t, device="cuda")
    idx3 = torch.empty((B, cfg.k), dtype=torch.int32, device="cuda")
    (w1d, _), (w3d, _) = upload_weights(w1), upload_weights(w3)
    ctx.wcc_block_forward(d, xd, w1d, None, dev(w_dw), w3d, None, y, t1, None, None, idx3)
    t2 = ref.depthwise3x3(t1.float().cpu().numpy().astype(np.float64), w_dw)
    branch, _ = layer_with_index_set(ref, cfg.layer(1), w3, t2, idx3.cpu().numpy().astype(np.int64))
    want = xd.float().cpu().numpy().astype(np.float64) + branch
    assert rel_l2(y.float().cpu().numpy(), want) <= (2.0 ** -9 + 1e-5 if maps == wcc.BF16 else 1e-5)
    assert torch.isnan(flat[x.size:].float()).all()
    ctx.close()
