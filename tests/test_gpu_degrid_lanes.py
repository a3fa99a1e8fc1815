"""Degridding by groups of lanes: every support (4, 8 and 16 lanes a group), rows
that lie exactly on cells (both ends of the stencil then carry weight), row
counts around the blocks, grids narrower than the stencil, and plane counts
around the transform's batches, against the oracle's gridding."""
import numpy as np
import pytest

from oracle import degrid as od

from .gpu_util import dev, host, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    return require_gpu()


@pytest.mark.parametrize("W", list(range(2, 17)))
def test_supports_and_aligned_rows(env, W):
    torch, swv = env
    rng = np.random.default_rng(W)
    nx, ny, cell = 24, 18, 2.0 ** -7
    n = 2 * 256 // (4 if W <= 4 else 8 if W <= 8 else 16) + 5
    u, v, w = (rng.uniform(-300, 300, n) for _ in range(3))
    # u Nx cell = u 3/8, v Ny cell = v 9/32: whole and half cells in either or both
    u[3], v[3] = 8.0 * 5, 0.1
    u[4], v[4] = 0.3, 32.0
    u[5], v[5] = -8.0 * 11, -64.0
    u[6], v[6] = 4.0, 16.0
    w[7] = w.min()                     # the first plane of the range
    u[8] = 8.0
    img = rng.uniform(-0.3, 1.0, (ny, nx)) * (rng.uniform(size=(ny, nx)) < 0.1)
    got = host(swv.predict_degrid(torch.as_tensor(img, device="cuda"), dev(u, torch), dev(v, torch),
                                  dev(w, torch), cell, W)[0])
    ref = od.predict_degrid(img, cell, u, v, w, W, -1)
    assert np.abs(got - ref).max() <= 1e-12 * np.abs(img).sum()


@pytest.mark.parametrize("nx,ny,W,wmax", [(1, 1, 16, 5.0), (2, 3, 12, 40.0), (5, 1, 16, 300.0),
                                          (33, 20, 8, 0.0), (33, 20, 9, 900.0), (300, 220, 6, 80.0)])
def test_narrow_grids_and_plane_counts(env, nx, ny, W, wmax):
    torch, swv = env
    rng = np.random.default_rng(nx + 7 * ny + W)
    n, cell = 70, 0.6 / max(nx, ny, 4)
    u, v = rng.uniform(-200, 200, n), rng.uniform(-200, 200, n)
    w = rng.uniform(-wmax, wmax, n)
    img = rng.uniform(0.1, 1.0, (ny, nx)) * (rng.uniform(size=(ny, nx)) < max(0.05, 2.0 / (nx * ny)))
    img[ny // 2, nx // 2] = 1.0
    got = host(swv.predict_degrid(torch.as_tensor(img, device="cuda"), dev(u, torch), dev(v, torch),
                                  dev(w, torch), cell, W)[0])
    ref = od.predict_degrid(img, cell, u, v, w, W, -1)
    assert np.abs(got - ref).max() <= 1e-12 * np.abs(img).sum()
