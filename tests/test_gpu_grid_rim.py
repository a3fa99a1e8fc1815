"""Dirty images whose corners, and pixels between others, lie off the unit disk: zero
there, and on it the oracle's values (FP64) or the adjoint's real parts
(FP32-compensated), by quads that straddle the rim, octets and the general route."""
import numpy as np
import pytest

from oracle import clean as oc

from .gpu_util import dev, dev_c, fp64_row_bound, host, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    return require_gpu()


@pytest.mark.parametrize("nx,ny,cx,cy,cell,unit", [
    (90, 90, 0, 0, 1.0 / 90, False), (64, 64, None, None, 1.6 / 64, False),
    (129, 70, 40, 69, 1.1 / 89, True), (256, 256, None, None, 2.4 / 256, False),
    (300, 280, 150, 100, 1.9 / 300, True)])
@pytest.mark.parametrize("prec", ["fp64", "f32c"])
def test_pixels_on_and_off_the_disk(env, nx, ny, cx, cy, cell, unit, prec):
    torch, swv = env
    n = 333
    rng = np.random.default_rng(nx + ny)
    u, v, w = (rng.uniform(-300, 300, n) for _ in range(3))
    y = np.ones(n, complex) if unit else rng.normal(size=n) + 1j * rng.normal(size=n)
    U, V, W, Y = dev(u, torch), dev(v, torch), dev(w, torch), dev_c(y, torch)
    img = host(swv.dirty_image(U, V, W, None if unit else Y, nx, ny, cell, cx, cy, -1, prec)).ravel()
    x0, y0 = nx // 2 if cx is None else cx, ny // 2 if cy is None else cy
    iy, ix = np.divmod(np.arange(nx * ny), nx)
    on = ((ix - x0) * cell) ** 2 + ((iy - y0) * cell) ** 2 < 1.0
    assert 0 < on.sum() < on.size
    assert np.all(img[~on] == 0.0)
    l, m, nm1, _ = oc.image_grid(nx, ny, cell, x0, y0)
    if prec == "fp64":
        p = np.flatnonzero(on)
        ref = oc.dirty_image(u, v, w, y, l[p], m[p], nm1[p])
        bound = fp64_row_bound(l[p], m[p], nm1[p], u, v, w, np.abs(y)) / n
        assert np.all(np.abs(img[p] - ref) <= bound)
    else:
        L, M, N = swv.image_grid(nx, ny, cell, cx, cy)
        adj = host(swv.adjoint(U, V, W, Y, L, M, N, prec="f32c")).real / n
        # the same FP32 sums but for the order in which chunks are added
        assert np.all(np.abs(img - adj)[on] <= 64 * 2.0 ** -53 * np.abs(y).mean())
