"""The contraction of few channels (needs an MI355X): up to 32 channels into up to 32 rows of 8-bit codes take the fp32
matrix kernel where the signal is long, beyond that the 8-bit one; one, two and three stages of 16 channels; rows of the compressed
signal of whole words and not.  int8 weights bit for bit (every sum is an exact integer), bf16 within the
rounding of the additions."""
import numpy as np
import pytest
import torch

from paper_2205_12268_amd import wcc
from tests.util import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("wt", [wcc.I8, wcc.BF16])
@pytest.mark.parametrize("B,H,W", [(1, 2, 6), (2, 30, 34), (3, 64, 132), (16, 64, 132)])     # k = 3, 255, 2112 and, enough
# workgroups for the large tiles, 2112 again
@pytest.mark.parametrize("K,M", [(1, 1), (8, 8), (12, 32), (16, 33), (32, 32), (33, 32), (32, 33), (36, 20), (48, 130)])
def test_few_channels(ref, K, M, B, H, W, wt):
    k = -(-H * W // 4)
    rng = np.random.default_rng(K * 1000 + M + H)
    xc = rng.integers(-127, 128, size=(B, K, k), dtype=np.int8)
    alpha = np.float32(1.75)
    scale = None
    if wt == wcc.I8:
        w = rng.integers(-127, 128, size=(M, K), dtype=np.int8)
        scale = (rng.random(M) + 0.5).astype(np.float32)
        stored = dev(w)
    else:
        stored = torch.from_numpy(rng.standard_normal((M, K)).astype(np.float32)).bfloat16().cuda()
        w = stored.float().cpu().numpy()
    d = wcc.make_desc(B, K, M, H, W, 1, 1, 4, wt, 8)
    ctx = wcc.Context(0)
    flat = torch.full((B * M * k + 64,), float("nan"), device="cuda")
    ctx.wcc_pointwise(d, stored, None if scale is None else dev(scale), dev(xc), dev(np.array([alpha])),
                      flat[:B * M * k].view(B, M, k))
    torch.cuda.synchronize()
    assert bool(torch.isnan(flat[B * M * k:]).all())
    got = flat[:B * M * k].view(B, M, k).cpu().numpy()
    sx = alpha / np.float32(127.0)
    if wt == wcc.I8:
        acc = np.einsum("mc,bcj->bmj", w.astype(np.int64), xc.astype(np.int64)).astype(np.float32)
        np.testing.assert_array_equal(got, acc * (sx * scale)[None, :, None])
    else:
        want = ref.pointwise(w.astype(np.float64), np.full(M, float(sx)), xc.astype(np.float64))
        bound = ref.pointwise(np.abs(w).astype(np.float64), np.full(M, float(sx)), np.abs(xc.astype(np.float64)))
        assert np.all(np.abs(got - want) <= (K + 2) * 2.0 ** -24 * bound)
    ctx.close()
