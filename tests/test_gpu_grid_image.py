"""Dirty images by axis phasors: the borders of the cover (lane tiles, strips
with the axes exchanged, step remainders), centres off the middle, row counts
around the chunks, unit visibilities, both signs, and rows whose w phase is
beyond the table's direct reach."""
from fractions import Fraction

import numpy as np
import pytest

from oracle import clean as oc

from .gpu_util import dev, dev_c, host, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    return require_gpu()


def _rows(n, seed, scale=300.0):
    rng = np.random.default_rng(seed)
    u, v, w = (rng.uniform(-scale, scale, n) for _ in range(3))
    return u, v, w, rng.standard_normal(n) + 1j * rng.standard_normal(n)


def _bound(u, v, w, y, l, m, nm1):
    """Phase roundings of the oracle (2 pi 2^-52 of the terms' magnitudes), a few
    2^-53 per phasor and product, and the running sum."""
    ph = np.abs(u).max() * np.abs(l) + np.abs(v).max() * np.abs(m) + np.abs(w).max() * np.abs(nm1)
    return np.abs(y).mean() * (2 * np.pi * 2.0 ** -52 * ph + (40 + np.sqrt(u.size)) * 2.0 ** -52)


@pytest.mark.parametrize("nx,ny,cx,cy,n,sign,unit", [
    (64, 64, None, None, 63, -1, False), (129, 129, None, None, 300, 1, False),
    (128, 128, 64, 64, 65, -1, True), (200, 40, None, None, 129, -1, False),
    (41, 201, None, None, 1000, 1, True), (130, 66, 70, 30, 500, -1, False),
    (255, 257, 127, 128, 70, 1, False), (100, 100, 20, 50, 64, -1, False),
    (127, 300, 63, 149, 1, -1, False), (90, 90, 0, 0, 50, -1, False),
    (96, 96, -5, 130, 50, 1, False)])
def test_images_against_oracle(env, nx, ny, cx, cy, n, sign, unit):
    torch, swv = env
    u, v, w, y = _rows(n, nx + 3 * ny + n)
    if unit:
        y = np.ones(n, np.complex128)
    cell = 0.9 / max(nx, ny)
    got = host(swv.dirty_image(dev(u, torch), dev(v, torch), dev(w, torch),
                               None if unit else dev_c(y, torch), nx, ny, cell, cx, cy, sign))
    c = (nx // 2 if cx is None else cx, ny // 2 if cy is None else cy)
    l, m, nm1, inside = oc.image_grid(nx, ny, cell, *c)
    l, m, nm1 = (np.where(inside, a, 0.0) for a in (l, m, nm1))
    ref = oc.dirty_image(u, v, w, y, l, m, nm1, sign)
    err = np.abs(got.ravel() - np.where(inside, ref, 0.0))
    assert np.all(err <= _bound(u, v, w, y, l, m, nm1))
    assert np.all(got.ravel()[~inside] == 0.0)


def test_w_phases_beyond_the_cells(env):
    """Rows with |w| up to 2^60 beside ordinary ones, against exact phases."""
    torch, swv = env
    u, v, w, y = _rows(40, 9)
    w[7], w[21], w[30] = 2.0 ** 45 + 0.375, -2.0 ** 52 - 3.0, 2.0 ** 60
    nx = 65
    cell = 0.01
    got = host(swv.dirty_image(dev(u, torch), dev(v, torch), dev(w, torch), dev_c(y, torch), nx, nx,
                               cell))
    l, m, nm1 = (host(t).ravel() for t in swv.image_grid(nx, nx, cell))
    for p in (0, 64, 32 * nx + 32, 40 * nx + 3, nx * nx - 1):
        x = 0.0
        for j in range(u.size):
            ph = (Fraction(u[j]) * Fraction(l[p]) + Fraction(v[j]) * Fraction(m[p]) +
                  Fraction(w[j]) * Fraction(nm1[p]))
            x += (np.exp(2j * np.pi * float(ph - round(ph))) * y[j]).real
        assert abs(got.ravel()[p] - x / u.size) <= 60 * 2.0 ** -52 * np.abs(y).mean(), p


def test_non_finite_rows_reach_every_pixel(env):
    torch, swv = env
    for k in range(4):
        r = list(_rows(200, 11))
        r[k][5] = np.nan if k != 2 else np.inf
        args = [dev(a, torch) for a in r[:3]] + [dev_c(r[3], torch)]
        assert not np.isfinite(host(swv.dirty_image(*args, 70, 66, 0.001))).any()


@pytest.mark.parametrize("nx,ny,cx,cy,sign", [(255, 255, None, None, -1), (256, 383, None, None, 1),
                                              (391, 259, 195, 129, -1), (300, 300, 128, 170, -1)])
def test_octets_against_oracle(env, nx, ny, cx, cy, sign):
    """Images with two and three whole 64-position blocks to the square, beside
    longer axes and centres off the middle: pixels from every region."""
    torch, swv = env
    u, v, w, y = _rows(90, nx + ny)
    cell = 0.5 / max(nx, ny)
    got = host(swv.dirty_image(dev(u, torch), dev(v, torch), dev(w, torch), dev_c(y, torch), nx, ny,
                               cell, cx, cy, sign))
    c = (nx // 2 if cx is None else cx, ny // 2 if cy is None else cy)
    l, m, nm1, _ = oc.image_grid(nx, ny, cell, *c)
    ref = oc.dirty_image(u, v, w, y, l, m, nm1, sign)
    assert np.all(np.abs(got.ravel() - ref) <= _bound(u, v, w, y, l, m, nm1))


@pytest.mark.parametrize("nx,ny,cx,cy,n,sign,unit", [
    (64, 64, None, None, 63, -1, False), (129, 128, None, None, 301, 1, False),
    (40, 200, None, None, 1000, -1, True), (130, 66, 70, 30, 500, 1, False),
    (255, 257, None, None, 4097, -1, False), (6, 7, None, None, 50, -1, False)])
def test_f32c_images_are_the_adjoints_real_parts(env, nx, ny, cx, cy, n, sign, unit):
    """The FP32-compensated image of four mirrored pixels at a time takes the
    adjoint's FP32 steps on the adjoint's chunks: its values are the adjoint's real
    parts but for the order in which the chunks' FP64 sums are added."""
    torch, swv = env
    u, v, w, y = _rows(n, 5 * nx + ny)
    if unit:
        y = np.ones(n, np.complex128)
    cell = 0.9 / max(nx, ny)
    U, V, W, Y = dev(u, torch), dev(v, torch), dev(w, torch), dev_c(y, torch)
    img = host(swv.dirty_image(U, V, W, None if unit else Y, nx, ny, cell, cx, cy, sign, "f32c"))
    l, m, nm1 = swv.image_grid(nx, ny, cell, cx, cy)
    adj = host(swv.adjoint(U, V, W, Y, l, m, nm1, sign=sign, prec="f32c")).real / n
    inside = host(l) ** 2 + host(m) ** 2 < 1.0
    c = (nx // 2 if cx is None else cx, ny // 2 if cy is None else cy)
    centre = np.zeros(nx * ny, bool)
    centre[c[1] * nx + c[0]] = True
    off = (host(l) == 0) & (host(m) == 0) & ~centre
    tol = 64 * 2.0 ** -53 * np.abs(y).mean()
    assert np.all(np.abs(img.ravel() - adj)[~off] <= tol) and np.all(img.ravel()[off] == 0.0)
    assert inside.all()
