"""GPU: points with more Delaunay neighbours than a star's lanes hold as
candidates (64), and stars that own more triangles than a wave collects (96),
one alone and several of one wave together, against the FP64 oracle."""
import numpy as np
import pytest

import oracle
import paper_2509_20198_amd as ls
import synth
from test_gpu_recon import _compare, _window_points

pytestmark = pytest.mark.gpu

H = 48000  # padded half window, raw units


def _owned(u, v):
    """Triangles of every point of which it is the lowest vertex, by (v, u), and neighbours."""
    pts = oracle.canon(oracle.make_points(u, v, np.zeros(len(u), np.int32), np.zeros((len(u), 3), np.uint16)))
    tri = oracle.delaunay(pts)
    low = [min(t, key=lambda i: (pts["v"][i], pts["u"][i])) for t in tri]
    return np.bincount(low, minlength=len(pts)), np.bincount(tri.ravel(), minlength=len(pts))


def _check(u, v, seed):
    rng = np.random.default_rng(seed)
    for mirror in (False, True):
        gpu, _ = _compare(synth.Region(), _window_points(-u - 1 if mirror else u, v, rng), np.zeros(1, np.int32))
        assert not np.any(gpu["status"] & ls.TILE_DEGENERATE)


def _arc(cx, cy, r, k, first, last):
    t = np.linspace(first, last, k)
    return np.rint(cx + r * np.cos(t)).astype(np.int64), np.rint(cy + r * np.sin(t)).astype(np.int64)


@pytest.mark.parametrize("k", [98, 150, 300])
def test_lowest_point_under_an_arc(k):
    """One star owns the whole fan."""
    u, v = _arc(0, -47000, 66000, k, np.pi / 4, 3 * np.pi / 4)
    u, v = np.concatenate([u, [0]]), np.concatenate([v, [-47000]])
    assert _owned(u, v)[0].max() > 96
    _check(u, v, k)


@pytest.mark.parametrize("hubs,k", [(3, 330), (5, 600), (8, 640)])
def test_neighbouring_fans(hubs, k):
    """Hubs on a small arc: each is the outermost in a part of the directions, so
    the large arc falls to them in parts, all stars of one wave."""
    u, v = _arc(137, -47000, 66000, k, np.pi / 4, 3 * np.pi / 4)
    hu, hv = _arc(0, -47500, 400, hubs, np.pi / 4, 3 * np.pi / 4)
    u, v = np.concatenate([u, hu]), np.concatenate([v, hv])
    own = np.sort(_owned(u, v)[0])[::-1]
    assert own[:hubs].sum() > 2 * 96 and own[1] > 96 // 3
    _check(u, v, k)


@pytest.mark.parametrize("k", [65, 110, 200])
def test_rings_of_more_neighbours_than_candidates(k):
    """Hubs inside rings, with other points around."""
    rng = np.random.default_rng(k)
    u, v = [], []
    hubs = [(-20000, -18000), (21000, -15000), (1000, 22000)]
    for x, y in hubs:
        ru, rv = _arc(x, y, 15000, k, 0.1, 0.1 + 2 * np.pi * (k - 1) / k)
        u += [x, *ru]
        v += [y, *rv]
    bu, bv = rng.integers(-H, H, 400), rng.integers(-H, H, 400)
    far = np.min([np.hypot(bu - x, bv - y) for x, y in hubs], axis=0) > 17000
    u, v = np.concatenate([u, bu[far]]), np.concatenate([v, bv[far]])
    assert np.sort(_owned(u, v)[1])[-3] > 64 - 8 * (k == 65)
    _check(u, v, k)
