"""GPU: the star walks of the reconstruction at the edges of their groups, work
items and candidate lists, against the FP64 oracle (tolerances of
test_gpu_recon); several launches per call against one."""
import numpy as np
import pytest
import torch

import oracle
import paper_2509_20198_amd as ls
import synth
from delaunay_check import check_linear_valid
from gpu_helpers import R_M
from test_gpu_recon import TOL_M, _compare, _gpu_recon, _window_points

pytestmark = pytest.mark.gpu

H = 48000  # padded half window, raw units


@pytest.mark.parametrize("m", [3, 4, 7, 8, 9, 16, 17, 33])
def test_point_counts_around_groups_and_items(m):
    rng = np.random.default_rng(m)
    u, v = rng.integers(-H, H, m), rng.integers(-H, H, m)
    _compare(synth.Region(), _window_points(u, v, rng), np.zeros(1, np.int32))


@pytest.mark.parametrize("clump,side", [(70, 40), (400, 60), (900, 3000)])
def test_density_jumps(clump, side):
    """More points in a bucket than a candidate list holds, beside nearly empty ones."""
    rng = np.random.default_rng(clump)
    cu, cv = rng.integers(-H + side, H - side, 2)
    u = np.concatenate([rng.integers(-H, H, 60), cu + rng.integers(0, side, clump)])
    v = np.concatenate([rng.integers(-H, H, 60), cv + rng.integers(0, side, clump)])
    _compare(synth.Region(), _window_points(u, v, rng), np.zeros(1, np.int32))


def test_lattice_clump_ties():
    """Cocircular points everywhere, too many for the candidate lists in one
    place: the linear map of a valid Delaunay triangulation (several are
    correct), the oracle's nearest points."""
    rng = np.random.default_rng(5)
    a, b = np.meshgrid(np.arange(-H, H, 6000), np.arange(-H, H, 6000))
    c, d = np.meshgrid(np.arange(0, 600, 30), np.arange(0, 600, 30))
    u = np.concatenate([a.ravel(), c.ravel() + 1000])
    v = np.concatenate([b.ravel(), d.ravel() - 2000])
    region, ps, tl = synth.Region(), _window_points(u, v, rng), np.zeros(1, np.int32)
    gpu = _gpu_recon(region, ps, tl, want_csr=False)
    xo, _, _ = oracle.recon_tiles(region, *ps, tl)
    assert np.abs(gpu["x"][0, ..., 1] - xo[0, ..., 1]).max() * R_M <= 1e-5
    qx, qy = np.meshgrid(-H + 500 + 1000 * np.arange(96), -H + 500 + 1000 * np.arange(96))
    h = gpu["x"][0] * R_M + gpu["cz"][0]
    check_linear_valid(np.stack([u, v], 1), ps[2] * 0.01, qx, qy, h[..., 0], h[..., 1], TOL_M)


def test_several_launches_per_call():
    """More tiles than the fixed scratch holds face maps for."""
    tx, ty = 40, 25
    g = ls.Grid.of(synth.Region(tiles_x=tx, tiles_y=ty))
    rng = np.random.default_rng(3)
    n = 6000
    x = torch.from_numpy(rng.integers(0, tx * 64000, n).astype(np.int32)).cuda()
    y = torch.from_numpy(rng.integers(0, ty * 64000, n).astype(np.int32)).cuda()
    z = torch.from_numpy(rng.integers(0, 5000, n).astype(np.int32)).cuda()
    rgb = torch.from_numpy(rng.integers(0, 65536, (n, 3)).astype(np.uint16)).cuda()
    tl = torch.arange(tx * ty, dtype=torch.int32, device="cuda")
    want = ls.recon_tiles(g, x, y, z, rgb, tl)
    got = ls.recon_tiles_noalloc(g, x, y, z, rgb, tl)
    torch.cuda.synchronize()
    for a, b in zip(want, got):
        assert torch.equal(a, b)
