"""The selection of planes above 16384 positions in two launches (needs an MI355X): its digits (zero alone, 64
steps an octave between 2^-32 and 2^32, the rest in the first and last step), digits whose keys fit in LDS (16384)
or are read from memory, classes of equal keys, one and several chunks of 4096, 8192 and 16384 positions, the
largest plane it takes and the next one, which the four launches take."""
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
    (1, 1024, 1024),    # 256 chunks, the largest plane
    (1, 1024, 1026),    # four launches
    (17, 512, 514),     # too many chunks: four launches
])
def test_two_launch_selection_chunks(B, H, W, kind):
    N = H * W
    check(B, H, W, kind, [1, N // 8 + 1, N // 2, N])
