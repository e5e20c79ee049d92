"""GPU: windows with many points at few positions, against the FP64 oracle (the
largest (z, R, G, B) of a position counts), and the time they take."""
import numpy as np
import pytest
import torch

import paper_2509_20198_amd as ls
import synth
from gpu_helpers import arrays_to_dev
from test_gpu_recon import _compare

pytestmark = pytest.mark.gpu

H = 48000  # padded half window, raw units


def _repeated(n, positions, levels, seed):
    """n points on `positions` positions; heights and colours of few levels tie."""
    rng = np.random.default_rng(seed)
    u, v = rng.integers(-H, H, positions), rng.integers(-H, H, positions)
    k = rng.integers(0, positions, n)
    z = (rng.integers(0, levels, n) * 700 - 900).astype(np.int32)
    rgb = (65535 - rng.integers(0, levels, (n, 3)) * 9000).astype(np.uint16)
    return (u[k] + 32000).astype(np.int32), (v[k] + 32000).astype(np.int32), z, rgb


# windows up to 2,644 points sort in LDS, larger ones in global memory
@pytest.mark.parametrize("n,positions", [(600, 10), (2, 1), (900, 1), (500, 499), (2640, 40), (2700, 40), (6000, 4000)])
@pytest.mark.parametrize("levels", [2, 7])
def test_repeated_positions(n, positions, levels):
    _compare(synth.Region(), _repeated(n, positions, levels, n + positions), np.zeros(1, np.int32))


def test_extreme_heights_and_colours():
    n = 300
    x, y, z, rgb = _repeated(n, 12, 3, 8)
    z[:] = np.where(np.arange(n) % 3 == 0, -(2**31), np.where(np.arange(n) % 3 == 1, 2**31 - 1, 0))
    z[x == x[0]] = -(2**31)
    rgb[x == x[0]] = 0
    region = synth.Region()
    xt, yt, zt, rt = arrays_to_dev(x, y, z, rgb)
    got, cz, _ = ls.recon_tiles(ls.Grid.of(region), xt, yt, zt, rt, torch.zeros(1, dtype=torch.int32, device="cuda"))
    # the same window with each position's largest point alone
    keep = {}
    for i in range(n):
        p = (int(x[i]), int(y[i]))
        if p not in keep or (z[i], *rgb[i]) > (z[keep[p]], *rgb[keep[p]]):
            keep[p] = i
    k = np.array(sorted(keep.values()))
    assert len(k) == 12
    xt, yt, zt, rt = arrays_to_dev(x[k], y[k], z[k], rgb[k])
    want, cz1, _ = ls.recon_tiles(ls.Grid.of(region), xt, yt, zt, rt, torch.zeros(1, dtype=torch.int32, device="cuda"))
    torch.cuda.synchronize()
    assert torch.equal(got, want) and torch.equal(cz, cz1)


def test_time_of_repeated_positions():
    """1,000 points at one position take no more than five times as long as 1,000
    spread over the window (340 times with a sort by one lane that reads heights
    and colours at every comparison)."""
    rng = np.random.default_rng(3)
    region = synth.Region()
    tl = torch.zeros(1, dtype=torch.int32, device="cuda")

    def us(u, v):
        n = len(u)
        p = arrays_to_dev(u, v, rng.integers(0, 5000, n), rng.integers(0, 65536, (n, 3)))
        ts = []
        for _ in range(4):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            ls.recon_tiles(ls.Grid.of(region), *p, tl)
            b.record()
            torch.cuda.synchronize()
            ts.append(a.elapsed_time(b) * 1e3)
        return min(ts)

    spread = us(rng.integers(0, 64000, 1000), rng.integers(0, 64000, 1000))
    one = us(np.full(1000, 30500), np.full(1000, 30500))
    print(f"1,000 points spread {spread:.0f} us, at one position {one:.0f} us")
    assert one <= 5 * spread
