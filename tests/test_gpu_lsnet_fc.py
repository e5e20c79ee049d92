"""GPU: the fully connected layers of the paper's network in BF16 at batch sizes
around their row and column tiles: the sums run over K in order whatever the
tiling, so a tile's result has the same bits in every batch."""
import numpy as np
import pytest
import torch

import paper_2509_20198_amd as ls
import synth
from test_gpu_lsnet import _inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [15, 17, 65, 224, 225])
def test_bf16_batch_sizes_same_bits(n):
    region, g, x, cz = _inputs(3, 1, 11)
    w = torch.from_numpy(synth.pnet_weights(2, R=g.R, bias_std=0.02).astype(np.float32)).cuda()
    xb = x[torch.arange(n, device="cuda") % 3].contiguous()
    cb = cz[torch.arange(n, device="cuda") % 3].contiguous()
    y, tex = ls.lsnet_refine_tiles(w, xb, cb, g, ls.BF16)
    for i in (0, n // 2, n - 1):
        y1, tex1 = ls.lsnet_refine_tiles(w, xb[i : i + 1].contiguous(), cb[i : i + 1].contiguous(), g, ls.BF16)
        assert torch.equal(y[i], y1[0])
        assert torch.equal(tex[i], tex1[0])
