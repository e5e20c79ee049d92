"""GPU: the BF16 fully connected layers of the paper's network where their loops
and tiles change: numbers of K steps that are no multiple of those in flight
(R = 16, 48 and 80), and the full chunk of 1,024 rows."""
import numpy as np
import pytest
import torch

import oracle
import paper_2509_20198_amd as ls
import synth
from test_gpu_lsnet import _inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("res,pad", [(16, 0), (16, 16), (64, 8)])
@pytest.mark.parametrize("tiles", [1, 5])
def test_bf16_k_remainders(res, pad, tiles):
    """Per-tile RMS of the normalised height against the oracle within the gate
    of the 96 x 96 grid (0.05 m of its 480 m)."""
    region, g, x, cz = _inputs(tiles, 1, 7 + res, pad=pad, res=res)
    w64 = synth.pnet_weights(2, R=g.R)
    y, _ = ls.lsnet_refine_tiles(torch.from_numpy(w64.astype(np.float32)).cuda(), x, cz, g, ls.BF16, want_tex=False)
    torch.cuda.synchronize()
    xs = x.cpu().numpy().astype(np.float64)
    ref = oracle.pnet_forward(w64, xs, res, pad)
    head = (ref - xs[:, pad:pad + res, pad:pad + res][..., [0, 2, 3, 4]])[..., 0]
    d = y.cpu().numpy()[..., 0].astype(np.float64) - ref[..., 0]
    rms = np.sqrt((d ** 2).reshape(tiles, -1).mean(1))
    assert rms.max() <= 0.05 / 480, rms
    assert np.sqrt((head ** 2).mean()) > 4 * 0.05 / 480  # the network's own part is well above the gate


@pytest.mark.parametrize("n", [1008, 1009, 1024, 1033])
def test_bf16_full_chunk_same_bits(n):
    region, g, x, cz = _inputs(3, 1, 11)
    w = torch.from_numpy(synth.pnet_weights(2, R=g.R, bias_std=0.02).astype(np.float32)).cuda()
    k = torch.arange(n, device="cuda") % 3
    y, _ = ls.lsnet_refine_tiles(w, x[k].contiguous(), cz[k].contiguous(), g, ls.BF16, want_tex=False)
    y3, _ = ls.lsnet_refine_tiles(w, x, cz, g, ls.BF16, want_tex=False)
    assert torch.equal(y, y3[k])
