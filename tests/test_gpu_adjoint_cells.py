"""FP64 adjoint with the table phasor: pixel counts around its 64-pixel groups
and columns, row counts around its chunks and steps, and the inputs that take
its WIDE form (far pixels, rows beyond the cells, non-finite rows)."""
import numpy as np
import pytest

from oracle import visibility as ov

from .gpu_util import dev, dev_c, fp64_row_bound, host, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    return require_gpu()


def _case(n, p, seed, scale=3e4):
    rng = np.random.default_rng(seed)
    u, v, w = (rng.uniform(-scale, scale, n) for _ in range(3))
    l, m = rng.uniform(-0.05, 0.05, p), rng.uniform(-0.05, 0.05, p)
    return u, v, w, rng.standard_normal(n) + 1j * rng.standard_normal(n), l, m, ov.n_minus_1(l, m)


def _run(env, u, v, w, y, l, m, nm1, sign=-1):
    torch, swv = env
    return host(swv.adjoint(*(dev(a, torch) for a in (u, v, w)), dev_c(y, torch),
                            *(dev(a, torch) for a in (l, m, nm1)), sign=sign))


@pytest.mark.parametrize("n,p,sign", [
    (1, 1, -1), (31, 64, 1), (33, 65, -1), (64, 129, 1), (511, 193, -1), (512, 255, 1),
    (513, 257, -1), (2047, 321, 1), (70001, 5, -1), (300003, 130, 1), (1027, 2049, -1),
    (1501, 577, 1), (2300, 1100, -1), (1027, 2048, 1),   # 4, 8 and 8 columns of a workgroup
    (9000, 4095, 1), (9000, 4097, -1)])                  # the chunk sums' two widths
def test_edges_against_oracle(env, n, p, sign):
    u, v, w, y, l, m, nm1 = _case(n, p, n + 5 * p)
    got = _run(env, u, v, w, y, l, m, nm1, sign)
    k = np.unique(np.linspace(0, p - 1, min(p, 60)).astype(int))
    ref = ov.adjoint(u, v, w, y, l[k], m[k], nm1[k], sign)
    assert np.all(np.abs(got[k] - ref) <= fp64_row_bound(l[k], m[k], nm1[k], u, v, w, np.abs(y)))


def test_far_pixels_and_rows(env):
    """Pixel coordinates beyond 2, rows beyond the cells' direct reach with exact
    phases, and a row that is not finite: only what they touch changes."""
    u, v, w, y, l, m, nm1 = _case(500, 130, 3, scale=64.0)
    clean = _run(env, u, v, w, y, l, m, nm1)
    l2 = l.copy()
    l2[70] = 2.0 ** 40 + 0.5          # with u a multiple of 2: whole turns
    u2 = np.round(u / 2.0) * 2.0
    got = _run(env, u2, 0 * v, 0 * w, y, l2, m, nm1)
    assert abs(got[70] - y.sum()) <= 1e-12 * np.abs(y).sum()
    ref = _run(env, u2, 0 * v, 0 * w, y, l, m, nm1)
    keep = np.arange(130) != 70
    assert np.array_equal(got[keep], ref[keep])
    u3, v3, w3 = u.copy(), v.copy(), w.copy()
    u3[9], v3[9], w3[9] = 2.0 ** 44, 0.0, 0.0
    l3 = np.full(130, 0.25)           # 2^42 turns: y[9] enters as it is
    base = _run(env, np.delete(u, 9), np.delete(v, 9), np.delete(w, 9), np.delete(y, 9), l3, m, nm1)
    got = _run(env, u3, v3, w3, y, l3, m, nm1)
    assert np.all(np.abs(got - base - y[9]) <= 1e-12 * np.abs(y).sum())
    u3[9] = np.inf
    assert np.isnan(_run(env, u3, v3, w3, y, l, m, nm1)).all()
    l4 = l.copy()
    l4[5] = np.nan
    got = _run(env, u, v, w, y, l4, m, nm1)
    keep = np.arange(130) != 5
    assert np.isnan(got[5]) and np.array_equal(got[keep], clean[keep])
