"""The FP32-compensated direct sum's reduced phase: leaves on either side of the
phase centre's horizon over baselines from a few to millions of wavelengths (n - 1
reaches -2 there, so a phase may be twice the baseline), and phases near zero of
both signs, whose sine keeps FP32's relative accuracy."""
import numpy as np
import pytest

from .gpu_util import dev, fp64_row_bound, host, require_gpu

pytestmark = pytest.mark.gpu

# per component: the reduced phase rounded to FP32 (2 pi 2^-25 turns at most), the
# hardware sine and cosine (2.5e-7 at most), a few 2^-24 of a product's rounding
PER_TERM = 2 * np.pi * 2.0 ** -25 + 2.5e-7 + 8 * 2.0 ** -24


@pytest.fixture(scope="module")
def env():
    return require_gpu()


@pytest.mark.parametrize("n_vis,n_leaf,J,sign", [(700, 3, 6, -1), (700, 40, 3, 1), (9000, 300, 8, -1),
                                                 (90, 5000, 9, -1), (300000, 5, 1, 1)])
def test_leaves_all_over_the_sphere(env, n_vis, n_leaf, J, sign):
    torch, swv = env
    rng = np.random.default_rng(n_vis + n_leaf)
    n_pix = 12 * 4 ** (J - 1)
    pix = np.sort(rng.choice(n_pix, min(n_leaf, n_pix), replace=False))
    t = swv.Tree.from_pixels(J, 1.0, 0.5, pix, rng.lognormal(-3, 1, pix.size))
    lf = t.leaves()
    assert lf["nm1"].min() < -1.2
    # lengths around every power of two and of its root, mostly along w, where the
    # leaves behind the horizon have their longest phases
    b = 2.0 ** (np.arange(n_vis) % 20 + 5 + rng.choice([0.0, 0.1, 0.4, 0.49], n_vis))
    a = rng.normal(size=(3, n_vis)) * np.array([[0.2], [0.2], [1.0]])
    u, v, w = a / np.linalg.norm(a, axis=0) * b
    got = host(t.predict_leaves(*(dev(x, torch) for x in (u, v, w)), sign=sign, prec="f32c"))
    swv.synchronize()
    rows = np.unique(np.linspace(0, n_vis - 1, min(n_vis, 200)).astype(int))
    u, v, w = u[rows], v[rows], w[rows]
    ld = np.longdouble
    ph = (u[:, None].astype(ld) * lf["l"] + v[:, None].astype(ld) * lf["m"] +
          w[:, None].astype(ld) * lf["nm1"])
    ref = (np.exp(2j * np.pi * sign * (ph - np.rint(ph)).astype(np.float64)) * lf["flux"]).sum(1)
    bound = PER_TERM * lf["flux"].sum() + fp64_row_bound(u, v, w, lf["l"], lf["m"], lf["nm1"],
                                                         lf["flux"])
    assert np.all(np.abs(got[rows] - ref) <= bound)
    t.close()


@pytest.mark.parametrize("n_comp", [1, 6])
def test_phases_near_zero_keep_their_sine(env, n_comp):
    """Phases of 1e-9 to 1e-3 turns, all of a row's with one sign.  Rounded to FP32
    they are good to 2^-25 of themselves, and so is the hardware sine to a few
    2^-22; held to a fixed 2^-33 turns the smallest would be off by a tenth."""
    torch, swv = env
    n = 500
    rng = np.random.default_rng(n_comp)
    ph = 10.0 ** rng.uniform(-9, -3, n) * rng.choice([-1, 1], n)
    l, f = rng.uniform(0.5, 1.0, n_comp) * 2.0 ** -20, rng.lognormal(-3, 1, n_comp)
    u, z = ph * 2.0 ** 20, np.zeros(n)
    got = host(swv.predict_direct(*(dev(x, torch) for x in (u, z, z, l, np.zeros(n_comp), f)),
                                  sign=1, prec="f32c"))
    ref = (f * np.sin(2 * np.pi * u[:, None] * l)).sum(1)
    assert np.all(np.abs(got.imag - ref) <= 1e-5 * np.abs(ref))
