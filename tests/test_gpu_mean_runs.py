"""GPU: mean splat of Morton-ordered points in runs of equal texels, as long as
a lane, a quad of lanes and a row of sixteen hold and one more or less: the
integer sums against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_2509_20198_amd as ls
import synth
from gpu_helpers import arrays_to_dev

pytestmark = pytest.mark.gpu


def _compact(c):
    return sum(((c >> (2 * i)) & 1) << i for i in range(16))


@pytest.mark.parametrize("run", [7, 8, 31, 32, 33, 127, 128, 129, 1100])
def test_runs_of_equal_texels(run):
    region = synth.Region(tiles_x=1, tiles_y=1)
    rng = np.random.default_rng(run)
    n = 3 * 2048 + 77
    code = 40 + np.arange(n) // run
    x = (_compact(code) * 1000 + rng.integers(0, 1000, n)).astype(np.int32)
    y = (_compact(code >> 1) * 1000 + rng.integers(0, 1000, n)).astype(np.int32)
    x[rng.integers(0, n, 20)] = -5  # outside: dropped
    z = rng.integers(-(2**31), 2**31, n, dtype=np.int64).astype(np.int32)
    z[: n // 2] = -(2**31)
    rgb = rng.integers(65000, 65536, (n, 3)).astype(np.uint16)
    ts = np.zeros(1, np.int32)
    want, wd = oracle.splat_mean(region, x, y, z, rgb, ts, 1)
    xt, yt, zt, rt = arrays_to_dev(x, y, z, rgb)
    acc, nd = ls.splat_mean(ls.Grid.of(region), xt, yt, zt, rt, torch.from_numpy(ts).cuda(), 1)
    torch.cuda.synchronize()
    assert np.array_equal(acc.cpu().numpy(), want)
    assert int(nd.item()) == wd
