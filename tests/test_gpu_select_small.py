"""The one-workgroup selection (N <= 16384) at the edges of its steps (needs an MI355X): keys that
one 13-bit field decides, that leave up to 512 keys in a bin (a list) or more (another pass), one and
several passes, equal keys, planes at and around its 4096 / 8192 / 16384 positions, k from 1 to N."""
import numpy as np
import pytest
import torch

from paper_2205_12268_amd import wcc

pytestmark = pytest.mark.gpu


def keys(kind, N, rng):
    if kind == "equal":
        return np.full(N, 0x40490FDB, np.uint32)
    if kind == "two":
        return np.where(rng.random(N) < 0.5, 0, 0x3F800000).astype(np.uint32)
    if kind == "field":                     # differences below 2^13: one field, no list
        return (0x3F800000 + rng.integers(0, 8192, N)).astype(np.uint32)
    if kind == "list":                      # about N / 8192 keys a bin of the first field
        return rng.integers(0x3F000000, 0x40000000, N).astype(np.uint32)
    if kind == "cluster":                   # one far key, the rest in one bin of the first two passes
        v = (0x3F800000 + rng.integers(0, 1 << 9, N)).astype(np.uint32)
        v[rng.integers(0, N)] = 0x7F000000
        return v
    if kind == "cluster_ties":              # the same with classes of equal keys
        v = (0x3F800000 + 64 * rng.integers(0, 6, N)).astype(np.uint32)
        v[rng.integers(0, N)] = 0
        return v
    return rng.integers(0, 0x7F800000, N).astype(np.uint32)   # any finite non-negative float


@pytest.mark.parametrize("kind", ["equal", "two", "field", "list", "cluster", "cluster_ties", "any"])
@pytest.mark.parametrize("H,W", [(2, 2), (2, 6), (32, 64), (64, 64), (2, 2050), (64, 128), (2, 4098), (128, 128), (130, 126)])
def test_small_selection(kind, H, W):
    N, B = H * W, 2
    rng = np.random.default_rng(N + sum(map(ord, kind)))
    key = np.stack([keys(kind, N, rng) for _ in range(B)])
    norm = torch.from_numpy(key.view(np.float32)).cuda()
    ctx = wcc.Context(0)
    for k in sorted({1, 2, N // 5 + 1, N // 2, N - 1, N}):
        d = wcc.make_desc(B, 1, 1, H, W, 1, k, N, wcc.F32, 0)
        assert wcc.k_of(d) == k
        ctx.ensure_workspace(d)
        idx = torch.full((B, k), -7, dtype=torch.int32, device="cuda")
        ctx.wcc_joint_topk(d, None, norm, idx)
        for b in range(B):
            order = np.lexsort((np.arange(N), -key[b].astype(np.int64)))[:k]
            np.testing.assert_array_equal(idx[b].cpu().numpy(), np.sort(order))
    ctx.close()
