"""FP32 weight gradients at the edges of their pixel tiles, against the FP64
oracle: several whole planes in a tile (1 to 10 texels wide, batches that do not
fill the last tile) and planes that choose the 32-wide tile.

A weight's gradient is a sum of at most n * R * R products in FP32, a layer's
within 1e-3 in norm (the tolerance of the other gradient tests)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2509_20198_amd as ls
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("res,pad,n", [(4, 0, 37), (2, 1, 19), (8, 0, 8), (6, 3, 5), (10, 1, 7), (20, 0, 7), (52, 0, 1),
                                       (48, 4, 2)])
def test_weight_gradients_of_small_and_wide_planes(res, pad, n):
    g = ls.Grid(res=res, pad=pad, tile_size=res * 1000)
    rng = np.random.default_rng(res)
    x = (rng.standard_normal((n, g.R, g.R, 8)) * 0.3).astype(np.float32)
    gy = rng.standard_normal((n, res, res, 4)).astype(np.float32)
    w = synth.unet_weights(2, head_std=0.05, bias_std=0.05).astype(np.float32)
    wt, xt, gt = (torch.from_numpy(a).cuda() for a in (w, x, gy))
    runs = []
    try:
        for c in range(-1, 3):  # numbers of partial sums
            for layer in range(len(synth.UNET_SHAPES)):
                ls.set_conv_config(layer, ls.FP32, 2, c)
            gw, _ = ls.refine_backward(wt, xt, gt, g, ls.FP32)
            runs.append(gw.cpu().numpy().astype(np.float64))
    finally:
        for layer in range(len(synth.UNET_SHAPES)):
            ls.set_conv_config(layer, ls.FP32, 2, -1)
    ref, _ = oracle.unet_backward(w.astype(np.float64), x.astype(np.float64), gy.astype(np.float64), res, pad)
    off = 0
    for name, ci, co in synth.UNET_SHAPES:
        sz = co * 9 * ci + co
        for gw in runs:
            assert np.linalg.norm(gw[off:off + sz] - ref[off:off + sz]) <= 1e-3 * np.linalg.norm(ref[off:off + sz]), name
        off += sz


def _us(fn):
    fn()
    ts = []
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        fn()
        b.record()
        torch.cuda.synchronize()
        ts.append(a.elapsed_time(b) * 1e3)
    return min(ts)


def test_tiny_planes_take_their_share_of_time():
    """2,000 tiles of 4 x 4 have the texels of 3.5 tiles of 96 x 96.  With a
    workgroup's tile for every plane their backward took eleven times as long;
    six times leaves room for the launches and the 1 x 1 planes."""
    w = torch.from_numpy(synth.unet_weights(2).astype(np.float32)).cuda()

    def backward(res, pad, n):
        g = ls.Grid(res=res, pad=pad, tile_size=res * 1000)
        x = torch.randn((n, g.R, g.R, 8), device="cuda")
        gy = torch.randn((n, res, res, 4), device="cuda")
        return lambda: ls.refine_backward(w, x, gy, g, ls.FP32)

    assert _us(backward(4, 0, 2000)) <= 6 * _us(backward(64, 16, 4))
