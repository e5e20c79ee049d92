"""FP32 network on planes that do not fill the conv kernels' pixel blocks
(8 x 4 and 8 x 8 per wave): odd and tiny grids, windows clipped by the plane,
the paper network's 40-, 24- and 4-channel layers, every tiling.

Against the FP64 oracle.  A forward output is a chain of at most 864 products
per layer over eleven layers, so 1e-5 of the largest output (about 170 FP32
roundoffs) bounds it; gradients per layer within 1e-3 in norm.  All tilings
sum in the same order: equal bits."""
import numpy as np
import pytest
import torch

import oracle
import paper_2509_20198_amd as ls
import synth
from paper_2509_20198_amd import autotune as AT

pytestmark = pytest.mark.gpu


def _case(res, pad, n, seed):
    g = ls.Grid(res=res, pad=pad, tile_size=res * 1000)
    rng = np.random.default_rng(seed)
    x = (rng.standard_normal((n, g.R, g.R, 8)) * 0.3).astype(np.float32)
    gy = rng.standard_normal((n, res, res, 4)).astype(np.float32)
    return g, x, gy


@pytest.mark.parametrize("res,pad,n", [(4, 0, 1), (12, 4, 2), (20, 2, 3), (34, 3, 1), (36, 0, 70)])
def test_unet_ragged_planes(res, pad, n):
    g, x, gy = _case(res, pad, n, 11 + res)
    w = synth.unet_weights(2, head_std=0.05, bias_std=0.05).astype(np.float32)
    wt, xt, gt = (torch.from_numpy(a).cuda() for a in (w, x, gy))
    runs = []
    try:
        for c in range(-1, 4):
            for layer in range(len(synth.UNET_SHAPES)):
                for p in (0, 1):
                    ls.set_conv_config(layer, ls.FP32, p, c)
            y, _ = ls.refine_tiles(wt, xt, None, g, ls.FP32, want_tex=False)
            act = torch.empty(ls.act_bytes(g, n, ls.FP32), dtype=torch.uint8, device="cuda")
            y2, _ = ls.refine_tiles(wt, xt, None, g, ls.FP32, want_tex=False, act_save=act)
            gw, gx = ls.refine_backward(wt, xt, gt, g, ls.FP32, act_save=act, want_grad_x=True)
            torch.cuda.synchronize()
            assert torch.equal(y, y2)  # windows of the decoder's last level against whole planes
            runs.append([t.cpu().numpy().astype(np.float64) for t in (y, gw, gx)])
    finally:
        AT.reset(ls.FP32, (0, 1))
    for r in runs[1:]:
        for a, b in zip(runs[0], r):
            assert np.array_equal(a, b)
    y, gw, gx = runs[0]
    w64, x64, gy64 = w.astype(np.float64), x.astype(np.float64), gy.astype(np.float64)
    y_ref = oracle.unet_forward(w64, x64, res, pad)
    gw_ref, gx_ref = oracle.unet_backward(w64, x64, gy64, res, pad, want_gx=True)
    assert np.abs(y - y_ref).max() <= 1e-5 * np.abs(y_ref).max()
    assert np.linalg.norm(gx - gx_ref) <= 1e-3 * np.linalg.norm(gx_ref)
    off = 0
    for name, ci, co in synth.UNET_SHAPES:
        sz = co * 9 * ci + co
        a, b = gw[off:off + sz], gw_ref[off:off + sz]
        assert np.linalg.norm(a - b) <= 1e-3 * np.linalg.norm(b), name
        off += sz


@pytest.mark.parametrize("res,pad,n", [(16, 0, 1), (20, 6, 2), (42, 3, 3)])
def test_paper_network_ragged_planes(res, pad, n):
    g, x, _ = _case(res, pad, n, 31 + res)
    w = synth.pnet_weights(4, R=g.R, final_std=0.05, bias_std=0.02).astype(np.float32)
    y, _ = ls.lsnet_refine_tiles(torch.from_numpy(w).cuda(), torch.from_numpy(x).cuda(), None, g, ls.FP32,
                                 want_tex=False)
    torch.cuda.synchronize()
    y_ref = oracle.pnet_forward(w.astype(np.float64), x.astype(np.float64), res, pad)
    assert np.abs(y.cpu().numpy() - y_ref).max() <= 1e-5 * np.abs(y_ref).max()
