"""How many planes of partial channel norms a layer's workspace holds, and with it which layers the
fixed array of wcc_forward_static takes.  The workspace's size is a pure host function; one case
runs on an MI355X."""
import pytest

from paper_2205_12268_amd import synth, wcc

F32, BF16, I8 = wcc.F32, wcc.BF16, wcc.I8

# Layers with one plane of partial norms (and of maxima, with 8-bit activations), all a little
# below the array's size: the strips alone give half a thousand waves, or there are too few channels to
# share.  B, C_in, C_out, H, W, levels, keep_num, keep_den, weights, act bits
FIT = [
    (8, 16, 96, 114, 480, 1, 3, 10, F32, 0),
    (2, 16, 96, 436, 576, 1, 1, 4, BF16, 8),
    (3, 26, 70, 156, 896, 1, 3, 8, F32, 0),
    (13, 16, 74, 562, 44, 1, 4, 8, I8, 8),
    (4, 5, 27, 96, 1172, 1, 4, 4, BF16, 0),
    (9, 5, 106, 62, 872, 1, 1, 4, BF16, 8),
    (11, 7, 9, 76, 1040, 2, 7, 8, BF16, 0),
    (13, 5, 41, 252, 96, 2, 2, 2, I8, 8),
    (2, 4, 10, 624, 696, 3, 2, 2, BF16, 0),
    (10, 5, 12, 544, 176, 3, 7, 10, F32, 8),
    (3, 5, 6, 512, 672, 4, 2, 2, F32, 0),
    (4, 6, 61, 448, 128, 4, 10, 10, BF16, 8),
]


def one_plane_bytes(B, Ci, Co, H, W, levels, num, den, wt, bits):
    """The workspace with one plane of partial norms: every buffer rounded up to 256 bytes."""
    N = H * W
    k = -(-num * N // den)
    ks = -(-k // 4) * 4
    chunk = next((c for c in (4096, 2048) if -(-N // c) * B >= 512), 1024)
    nblk = -(-N // chunk)
    q = bits == 8
    parts = [4 * B * N, 4 * B * N if q else 0, 4 * B * N, 4 * B * 3 * 2048, 32 * B, B * nblk * 2048, 4 * B * nblk,
             4 * B * N, 4 * B * k, 256, 4 * B * nblk if q else 0, 1024, 4 * B * Ci * ks, 4 * B * Co * ks]
    return sum(-(-p // 256) * 256 for p in parts)


@pytest.mark.parametrize("case", FIT, ids=lambda c: "x".join(map(str, c)))
def test_layers_that_fit_the_static_array_with_one_plane(case):
    assert one_plane_bytes(*case) <= wcc.STATIC_SCRATCH_BYTES      # what the case is about
    assert wcc.workspace_bytes(wcc.make_desc(*case)) <= wcc.STATIC_SCRATCH_BYTES


@pytest.mark.parametrize("levels", [1, 2, 3, 4])
@pytest.mark.parametrize("bits", [0, 8])
@pytest.mark.parametrize("C", [1, 4, 6, 7, 16, 31, 64])
def test_one_plane_where_strips_give_half_a_thousand_waves(levels, bits, C):
    """W = 256 columns are one wave (two at four levels), H / 2^levels of them a plane."""
    H = (512 << levels) // (2 if levels == 4 else 1)
    case = (1, C, 24, H, 256, levels, 1, 4, BF16, bits)
    assert wcc.workspace_bytes(wcc.make_desc(*case)) == one_plane_bytes(*case)


@pytest.mark.gpu
def test_static_entry_takes_such_a_layer():
    import torch

    from tests.util import dev, upload_weights
    cfg = synth.LayerCfg("planes", *FIT[1], sigma=1.5, seed=synth.SEED_BASE + 0x1300)
    x, w = synth.make_inputs(cfg)
    d = wcc.make_desc(*FIT[1])
    ctx = wcc.Context(0)
    ctx.ensure_workspace(d)
    wd, _ = upload_weights(w)
    ys = [torch.full((2, 96, 436, 576), float("nan"), device="cuda") for _ in range(2)]
    ctx.wcc_forward_static(d, dev(x), wd, None, 0.0, ys[0])
    ctx.wcc_forward(d, dev(x), wd, None, 0.0, ys[1])
    torch.cuda.synchronize()
    assert bool(torch.isfinite(ys[0]).all()) and torch.equal(ys[0], ys[1])
    ctx.close()
