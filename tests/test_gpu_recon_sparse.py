"""GPU: tile lists in which most windows hold fewer than three points, or none:
these come last, without face maps.  Against the FP64 oracle, and the time of a
nearly empty list."""
import numpy as np
import pytest
import torch

import oracle
import paper_2509_20198_amd as ls
import synth
from gpu_helpers import R_M, arrays_to_dev

pytestmark = pytest.mark.gpu

S = 64000


def _counts(tx, ty, rng, of):
    """Points well inside their tiles (one window each): of(t) of them in tile t."""
    x, y = [], []
    for t in range(tx * ty):
        n = of(t)
        x.append((t % tx) * S + rng.integers(20000, 44000, n))
        y.append((t // tx) * S + rng.integers(20000, 44000, n))
    x, y = np.concatenate(x), np.concatenate(y)
    z = rng.integers(0, 5000, len(x)).astype(np.int32)
    rgb = rng.integers(0, 65536, (len(x), 3)).astype(np.uint16)
    return x.astype(np.int32), y.astype(np.int32), z, rgb


@pytest.mark.parametrize("order", [ls.ORDER_LIST, ls.ORDER_LONGEST_FIRST])
@pytest.mark.parametrize("tx,ty,every,most", [(40, 40, 3, 5), (33, 32, 1, 3), (40, 40, 400, 700), (7, 3, 2, 2)])
def test_windows_of_few_points(tx, ty, every, most, order):
    """Every few tiles hold up to `most` points; with a caller's CSR, several
    launches of face maps and the rest without, in the library's scratch and in
    a workspace."""
    rng = np.random.default_rng(tx + every + most)
    region = synth.Region(tiles_x=tx, tiles_y=ty)
    g = ls.Grid.of(region)
    ps = _counts(tx, ty, rng, lambda t: int(rng.integers(0, most + 1)) if t % every == 0 else 0)
    tl = rng.permutation(tx * ty).astype(np.int32)
    tl[-2:] = tl[0], tx * ty + 5  # listed twice, outside
    dev = arrays_to_dev(*ps)
    tt = torch.from_numpy(tl).cuda()
    runs = []
    for fn in (ls.recon_tiles, ls.recon_tiles_noalloc):
        off = torch.empty(len(tl) + 1, dtype=torch.int32, device="cuda")
        idx = torch.empty(4 * len(ps[0]), dtype=torch.int32, device="cuda")
        x, cz, st = fn(g, *dev, tt, order=order, bin_off=off, bin_idx=idx)
        torch.cuda.synchronize()
        o = off.cpu().numpy()
        runs.append([a.cpu().numpy() for a in (x, cz, st)] + [o, idx.cpu().numpy()[:o[-1]]])
    for a, b in zip(*runs):
        assert np.array_equal(a, b)
    x, cz, st, off, idx = runs[0]
    want_off, want_idx = oracle.bin_points(region, *ps[:2], tl[:-2])
    assert np.array_equal(off[:-2], want_off) and np.array_equal(idx, want_idx)
    assert np.all(st[-2:] & ls.TILE_BADID) and np.all(x[-2:] == 0)
    k = np.concatenate([np.flatnonzero(np.diff(want_off) >= 3)[:40], np.flatnonzero(np.diff(want_off) == 2)[:20],
                        np.flatnonzero(np.diff(want_off) == 1)[:20], np.flatnonzero(np.diff(want_off) == 0)[:5]])
    xo, czo, sto = oracle.recon_tiles(region, *ps, tl[k])
    assert np.array_equal(st[k] & 3, sto)
    assert np.abs(x[k, ..., 0] - xo[..., 0]).max() * R_M <= 1e-4
    assert np.abs(x[k, ..., 1] - xo[..., 1]).max() * R_M <= 1e-5
    np.testing.assert_allclose(cz[k], czo, atol=1e-9)
    empty = np.flatnonzero(np.diff(want_off) == 0)
    assert np.all(x[empty] == 0) and np.all(st[empty] & ls.TILE_EMPTY)


def test_time_of_a_nearly_empty_list():
    """16,384 tiles with 1,000 points in all: little more than writing the maps
    (1.6 times that; 2.7 times with launches for face maps over every tile)."""
    rng = np.random.default_rng(2)
    g = ls.Grid.of(synth.Region(tiles_x=128, tiles_y=128))
    n = 1000
    p = arrays_to_dev(rng.integers(0, 128 * S, n), rng.integers(0, 128 * S, n), rng.integers(0, 5000, n),
                      rng.integers(0, 65536, (n, 3)))
    tl = torch.arange(128 * 128, dtype=torch.int32, device="cuda")
    x = torch.empty((128 * 128, g.R, g.R, 8), device="cuda")

    def us(fn):
        ts = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            fn()
            b.record()
            torch.cuda.synchronize()
            ts.append(a.elapsed_time(b) * 1e3)
        return min(ts)

    fill = us(x.zero_)
    recon = us(lambda: ls.recon_tiles(g, *p, tl, x_out=x))
    print(f"fill {fill:.0f} us, reconstruction {recon:.0f} us")
    assert recon <= 2 * fill
