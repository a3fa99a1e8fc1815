"""Gradients with the table phasor: component counts around the 64-component
groups and columns, row counts around the chunks and steps, and rows beyond the
cells' direct reach."""
import numpy as np
import pytest

from oracle import visibility as ov

from .gpu_util import dev, dev_c, host, require_gpu
from .test_gpu_image import _grad_scales

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    return require_gpu()


def _run(env, u, v, w, y, l, m, f, sign=-1):
    torch, swv = env
    return [host(g) for g in swv.grad_direct(*(dev(a, torch) for a in (u, v, w)), dev_c(y, torch),
                                             *(dev(a, torch) for a in (l, m, f)), sign=sign,
                                             alpha=-2.0)]


@pytest.mark.parametrize("n,k,sign", [
    (1, 1, -1), (33, 64, 1), (64, 65, -1), (511, 128, 1), (513, 193, -1), (2047, 257, 1),
    (100003, 3, -1), (30001, 321, 1), (1027, 2049, -1),
    (1501, 577, 1), (2300, 1100, -1), (1027, 2048, 1)])   # 4, 8 and 8 columns of a workgroup
def test_edges_against_oracle(env, n, k, sign):
    rng = np.random.default_rng(n + 3 * k)
    u, v, w = (rng.uniform(-5e4, 5e4, n) for _ in range(3))
    y = rng.standard_normal(n) + 1j * rng.standard_normal(n)
    l, m, f = rng.uniform(-0.03, 0.03, k), rng.uniform(-0.03, 0.03, k), rng.lognormal(-3, 1, k)
    got = _run(env, u, v, w, y, l, m, f, sign)
    q = np.unique(np.linspace(0, k - 1, min(k, 60)).astype(int))
    ref = ov.grad_direct(u, v, w, y, l[q], m[q], f[q], sign=sign, alpha=-2.0)
    for g, r, sc in zip(got, ref, _grad_scales(u, v, w, l[q], m[q], f[q], y)):
        assert np.all(np.abs(g[q] - r) <= 2.0 * sc)


def test_rows_beyond_the_cells(env):
    """A row whose phases are whole turns far above 2^39 for every component adds
    its visibility's plain terms to the others'."""
    rng = np.random.default_rng(8)
    n, k = 300, 70
    u, v, w = (rng.uniform(-50, 50, n) for _ in range(3))
    y = rng.standard_normal(n) + 1j * rng.standard_normal(n)
    l, m, f = np.full(k, 0.25), rng.uniform(-0.03, 0.03, k), np.ones(k)
    rest = _run(env, np.delete(u, 7), np.delete(v, 7), np.delete(w, 7), np.delete(y, 7), l, m, f)
    u[7], v[7], w[7] = 2.0 ** 44, 0.0, 0.0
    got = _run(env, u, v, w, y, l, m, f)
    # e = 1: z = conj(y), so Z0 gains Re y and Zu gains -u Im y
    assert np.all(np.abs(got[0] - rest[0] + 2.0 * y[7].real) <= 1e-11)
    gain = 2.0 * f * -1 * 2 * np.pi * (-u[7] * y[7].imag)
    assert np.allclose(got[1] - rest[1], gain, rtol=1e-9)
    u[7] = np.nan
    assert np.isnan(np.concatenate(_run(env, u, v, w, y, l, m, f))).all()
