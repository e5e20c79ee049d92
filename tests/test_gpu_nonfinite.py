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


def _planes(g, n, act):
    """The saved FP32 activations A1 .. A10 and the two pooled ones."""
    f = act.cpu().numpy().view(np.float32).astype(np.float64)
    shapes = {"A1": (16, 1), "A2": (16, 1), "P1": (16, 2), "A3": (32, 2), "A4": (32, 2), "P2": (32, 4), "A5": (64, 4),
              "A6": (64, 4), "A7": (32, 2), "A8": (32, 2), "A9": (16, 1), "A10": (16, 1)}
    out, at = {}, 0
    for k, (c, s) in shapes.items():
        m = n * (g.R // s) ** 2 * c
        out[k] = f[at:at + m].reshape(n, g.R // s, g.R // s, c)
        at += m
    return out


def _conv(x, w, b):
    """3x3 conv without the taps outside the plane, then max(., 0) with NaN to 0, as the kernels' fmaxf."""
    n, h, wd, cin = x.shape
    w = w.reshape(-1, 3, 3, cin)
    s = np.broadcast_to(b, (n, h, wd, len(b))).copy()
    for ky in range(3):
        for kx in range(3):
            oy, ox = slice(max(0, 1 - ky), min(h, h + 1 - ky)), slice(max(0, 1 - kx), min(wd, wd + 1 - kx))
            iy, ix = slice(max(0, ky - 1), min(h, h + ky - 1)), slice(max(0, kx - 1), min(wd, wd + kx - 1))
            with np.errstate(invalid="ignore"):
                s[:, oy, ox] += (x[:, iy, ix, None, :] * w[None, None, None, :, ky, kx, :]).sum(-1)
    return np.where(s > 0, s, 0.0)


@pytest.mark.parametrize("layer", range(10))
@pytest.mark.parametrize("value", [np.inf, -np.inf])
def test_every_layer_on_its_own_inputs(layer, value):
    """Infinite weights at three taps of one hidden layer; its saved output
    against a 64-bit conv of its saved inputs."""
    g, w, x, gy = _case(20, 0, 9)
    shapes = [(ci, co) for _, ci, co in synth.UNET_SHAPES]
    off = sum(co * 9 * ci + co for ci, co in shapes[:layer])
    ci, co = shapes[layer]
    wl = w[off:off + co * 9 * ci].reshape(co, 9, ci)
    wl[1, 0, 0] = wl[co - 1, 5, ci - 1] = wl[co // 2, 7, ci // 2] = value
    act = torch.empty(ls.act_bytes(g, 2, ls.FP32), dtype=torch.uint8, device="cuda")
    ls.refine_tiles(torch.from_numpy(w).cuda(), torch.from_numpy(x).cuda(), None, g, ls.FP32, want_tex=False, act_save=act)
    torch.cuda.synchronize()
    a = _planes(g, 2, act)
    up = lambda t: t.repeat(2, 1).repeat(2, 2)
    src = [x.astype(np.float64), a["A1"], a["P1"], a["A3"], a["P2"], a["A5"], np.concatenate([up(a["A6"]), a["A4"]], -1),
           a["A7"], np.concatenate([up(a["A8"]), a["A2"]], -1), a["A9"]][layer]
    got = a[["A1", "A2", "A3", "A4", "A5", "A6", "A7", "A8", "A9", "A10"][layer]]
    want = _conv(src, wl.astype(np.float64), w[off + co * 9 * ci:off + co * 9 * ci + co].astype(np.float64))
    assert (want == np.inf).any() or value < 0
    _same(got, want, 1e-5)
