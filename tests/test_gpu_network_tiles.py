"""The network's kernels at the edges of their tiles (32 x 4 or 8 voxels, a few
planes; 16 voxels and channels on the coarse levels), and their two tile sizes
against each other."""
import numpy as np
import pytest

from oracle import learned as OL

pytestmark = pytest.mark.gpu


# extents (z, y, x): one tile, x beyond one, few and many rows, a thin box.  Weights
# of 0 and +-1, about four to an output channel, and small whole inputs: every sum
# of the forward pass is exact in FP32 as in FP64, so the oracle rounds the same
# values to bfloat16 and no entry flips; the weight gradient's sums of up to 15 000
# terms are off by their own rounding, 15 000 times 2^-24 of the largest at worst.
@pytest.mark.parametrize("dims", [(8, 8, 8), (8, 8, 40), (40, 16, 8), (16, 8, 72), (24, 40, 16)])
def test_gradient_at_tile_edges(dims):
    from paper_1010_2832_amd import learned as L
    from paper_1010_2832_amd import vfstokes as V
    Z, Y, X = dims
    print(f"[network] {dims}", flush=True)
    rng = np.random.default_rng(4)
    offs = np.cumsum([0] + OL.layer_sizes())
    w = np.zeros(offs[-1], np.float32)
    for layer, (cin, cout) in enumerate(L.LAYERS):
        n = offs[layer + 1] - offs[layer]
        on = rng.random(n) < 4.0 / (27 * cin)
        w[offs[layer]:offs[layer + 1]] = on * rng.choice([-1.0, 1.0, 1.0], n)
    x = rng.integers(-2, 3, size=(Z, Y, X, 16)).astype(np.float32)
    gy = rng.integers(-2, 3, size=(Z, Y, X, 6)).astype(np.float32)
    net = V.Unet()
    net.vfs_unet_set_weights(w)
    y = net.vfs_unet_forward(x)
    y_o, cache = OL.forward(w.astype(np.float64), x.astype(np.float64), bf16_mode=True)
    assert np.abs(y_o).max() > 0
    assert np.array_equal(y, y_o.astype(np.float32))
    net.vfs_unet_backward(gy)
    g = net.vfs_unet_get_grad()
    g_o = OL.backward(cache, gy.astype(np.float64), bf16_mode=True)
    for layer in range(8):
        sl = slice(offs[layer], offs[layer + 1])
        scale = np.abs(g_o[sl]).max()
        err = np.abs(g[sl] - g_o[sl]).max() / scale
        print(f"[network] layer {layer}: gradient off by {err:.1e} of {scale:.3g}", flush=True)
        assert scale > 0 and err <= 15000 * 2.0**-24
    net.close()


def test_large_and_small_tiles_give_the_same_bits():
    """At 168^3 the middle levels run in large tiles, at 96^3 in small ones; away
    from the crop's border (a receptive field of 30 voxels, and 8 for the coarse
    cells) the outputs are equal."""
    from paper_1010_2832_amd import learned as L
    from paper_1010_2832_amd import vfstokes as V
    rng = np.random.default_rng(6)
    net = V.Unet()
    net.vfs_unet_set_weights(L.he_init(3, last_scale=1.0))
    x = rng.standard_normal(size=(168, 168, 168, 16), dtype=np.float32)
    big = net.vfs_unet_forward(x)[80:96, 80:96, 80:96].copy()
    small = net.vfs_unet_forward(np.ascontiguousarray(x[40:136, 40:136, 40:136]))[40:56, 40:56, 40:56]
    assert np.array_equal(big, small)
    net.close()
