"""FP32 network with infinite weights and inputs: only what a conv's taps reach
is affected.  A tap outside the plane, or outside the tensor that a wider plane
embeds, contributes nothing; neither does an input outside the window that the
head's weight gradient sums over."""
import numpy as np
import pytest
import torch

import oracle
import paper_2509_20198_amd as ls
import synth

pytestmark = pytest.mark.gpu

HEAD = 4 * 9 * 24 + 4  # the last layer's weights and biases


def _case(res, pad, seed):
    g = ls.Grid(res=res, pad=pad, tile_size=res * 1000)
    rng = np.random.default_rng(seed)
    x = (rng.standard_normal((2, g.R, g.R, 8)) * 0.3).astype(np.float32)
    gy = rng.standard_normal((2, res, res, 4)).astype(np.float32)
    w = synth.unet_weights(2, head_std=0.05, bias_std=0.05).astype(np.float32)
    return g, w, x, gy


def _same(a, ref, tol):
    """Equal infinities and NaNs, the rest within tol in norm."""
    assert np.array_equal(np.isnan(a), np.isnan(ref))
    fin = np.isfinite(ref)
    assert np.array_equal(np.isfinite(a), fin)
    inf = ~fin & ~np.isnan(ref)
    assert np.array_equal(a[inf], ref[inf])
    assert np.linalg.norm(a[fin] - ref[fin]) <= tol * np.linalg.norm(ref[fin])


@pytest.mark.parametrize("res,pad", [(20, 0), (34, 3), (12, 4)])
@pytest.mark.parametrize("tap", [0, 2, 5, 7, 8])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_taps_outside_the_plane(res, pad, tap, value):
    """One infinite weight of the head, on a skip channel (its inputs are nowhere
    zero): forward and input gradient, also with twice the pixels per wave."""
    g, w, x, gy = _case(res, pad, 3)
    w[-HEAD + (2 * 9 + tap) * 24 + 16 + 3] = value
    w64, x64 = w.astype(np.float64), x.astype(np.float64)
    y_ref = oracle.unet_forward(w64, x64, res, pad)
    _, gx_ref = oracle.unet_backward(w64, x64, gy.astype(np.float64), res, pad, want_gx=True)
    wt, xt, gt = (torch.from_numpy(a).cuda() for a in (w, x, gy))
    try:
        for c in (-1, 2):
            for p in (0, 1):
                ls.set_conv_config(10, ls.FP32, p, c)
            y, _ = ls.refine_tiles(wt, xt, None, g, ls.FP32, want_tex=False)
            _, gx = ls.refine_backward(wt, xt, gt, g, ls.FP32, want_grad_x=True)
            torch.cuda.synchronize()
            _same(y.cpu().numpy().astype(np.float64), y_ref, 1e-5)
            _same(gx.cpu().numpy().astype(np.float64), gx_ref, 1e-3)
    finally:
        for p in (0, 1):
            ls.set_conv_config(10, ls.FP32, p, -1)


@pytest.mark.parametrize("res,pad", [(20, 6), (22, 5), (4, 6)])
def test_inputs_outside_the_heads_window(res, pad):
    """Saved activations of finite inputs: the head's weight gradient does not
    see inputs beyond the one-texel ring of its window."""
    g, w, x, gy = _case(res, pad, 5)
    R = g.R
    wt, xt, gt = (torch.from_numpy(a).cuda() for a in (w, x, gy))
    act = torch.empty(ls.act_bytes(g, 2, ls.FP32), dtype=torch.uint8, device="cuda")
    ls.refine_tiles(wt, xt, None, g, ls.FP32, want_tex=False, act_save=act)
    want, _ = ls.refine_backward(wt, xt, gt, g, ls.FP32, act_save=act)
    far = torch.ones((R, R), dtype=torch.bool)
    far[pad - 1:pad + res + 1, pad - 1:pad + res + 1] = False
    xt[:, far.cuda()] = float("inf")
    got, _ = ls.refine_backward(wt, xt, gt, g, ls.FP32, act_save=act)
    torch.cuda.synchronize()
    assert torch.isfinite(want).all()
    assert torch.equal(got[-HEAD:], want[-HEAD:])
