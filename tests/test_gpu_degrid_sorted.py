"""Degridding of rows sorted by tile (supports above 6, from 65,536 rows, planes
beyond 4 MB): each row has the bits that it has among few rows, whatever its tile
and slab."""
import numpy as np
import pytest

from .gpu_util import dev, host, note, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    return require_gpu()


@pytest.mark.parametrize("n,nx,ny,W", [
    (65536, 200, 150, 9), (65539, 300, 220, 10),   # the latter: a last workgroup of 3 rows
    (70001, 5000, 1, 16), (2 ** 21 + 5, 200, 160, 7)])   # one row of tiles; two slabs
def test_bits_of_few_rows(env, n, nx, ny, W):
    torch, swv = env
    rng = np.random.default_rng(n + W)
    cell = 0.3 / max(nx, ny)
    u, v, w = rng.uniform(-300, 300, n), rng.uniform(-300, 300, n), rng.uniform(-9, 9, n)
    u[:n // 2] = rng.normal(40.0, 3.0, n // 2)     # half of them in a few tiles
    v[:n // 2] = rng.normal(-25.0, 3.0, n // 2)
    w[0], w[1] = -10.0, 10.0                       # the range of every part below
    u[5], u[6], v[7], u[n - 1], v[n - 2] = np.nan, 2.0 ** 70, -np.inf, 2.0 ** 60, 0.0
    img = torch.as_tensor(rng.uniform(-0.3, 1.0, (ny, nx)), device="cuda")
    note(f"degrid sorted n={n} {nx}x{ny} W={W}")
    got = host(swv.predict_degrid(img, dev(u, torch), dev(v, torch), dev(w, torch), cell, W)[0])
    starts = [0, n // 2 - 30000, n - 60000]
    for s in starts:
        k = np.concatenate([[0, 1], np.arange(s, s + 60000)])
        few = host(swv.predict_degrid(img, *(dev(a[k], torch) for a in (u, v, w)), cell, W)[0])
        assert np.array_equal(got[k], few, equal_nan=True)
    assert np.isnan(got[[5, 6, 7, n - 1]]).all() and np.isfinite(got[[0, 1, n - 2]]).all()
