"""FP32-compensated direct sum: component counts around its fours, ranges and
sub-ranges, row counts around the layouts that share components between waves
and workgroups (the batched kernel, which gives a row to one wave, has the same
bits), and rows beyond the reach of the phase that starts at a magic number."""
import numpy as np
import pytest

from oracle import visibility as ov

from .gpu_util import dev, host, require_gpu

pytestmark = pytest.mark.gpu

# per component: the reduced phase rounded to FP32 (2 pi 2^-25 turns at most), the
# hardware sine and cosine (2.5e-7 at most), a few 2^-24 of a product's rounding
PER_TERM = 2 * np.pi * 2.0 ** -25 + 2.5e-7 + 8 * 2.0 ** -24


@pytest.fixture(scope="module")
def env():
    return require_gpu()


@pytest.mark.parametrize("n_vis,n_comp", [
    (1, 1), (63, 3), (65, 31), (511, 32), (513, 63), (64, 130), (1025, 1025), (351, 4096),
    (100, 20000), (9000, 2049), (140001, 37), (300001, 18)])
def test_layouts_against_oracle_and_batched(env, n_vis, n_comp):
    torch, swv = env
    rng = np.random.default_rng(n_vis + 11 * n_comp)
    u, v, w = (rng.uniform(-1e5, 1e5, n_vis) for _ in range(3))
    l, m = rng.uniform(-0.03, 0.03, n_comp), rng.uniform(-0.03, 0.03, n_comp)
    f = rng.lognormal(-3, 1, n_comp)
    d = [dev(a, torch) for a in (u, v, w, l, m, f)]
    got = swv.predict_direct(*d, prec="f32c")
    out = torch.empty(n_vis, dtype=torch.complex64, device="cuda")
    plan = swv.BatchPlan([dict(zip(("u", "v", "w", "l", "m", "flux"), d), route="direct",
                               prec="f32c", out=out)])
    plan.run()
    swv.synchronize()
    assert torch.equal(got, out)
    rows = np.unique(np.linspace(0, n_vis - 1, min(n_vis, 200)).astype(int))
    ref = ov.predict_direct(u[rows], v[rows], w[rows], l, m, f)
    assert np.abs(host(got)[rows] - ref).max() <= PER_TERM * f.sum()
    plan.close()


def test_rows_beyond_the_magic_number(env):
    """Rows from 2^17 to 2^40 wavelengths, whose phases are multiples of 1/8 turn,
    and rows that are not finite: each row against its exact value."""
    torch, swv = env
    n, k = 400, 21
    rng = np.random.default_rng(4)
    u = np.round(rng.uniform(-1, 1, n) * 2.0 ** rng.uniform(5, 40, n)) / 4.0
    v, w = np.zeros(n), np.zeros(n)
    l, m, f = np.full(k, 0.5), np.zeros(k), np.ones(k)
    got = host(swv.predict_direct(*(dev(a, torch) for a in (u, v, w, l, m, f)), prec="f32c"))
    swv.synchronize()
    ref = k * np.exp(-2j * np.pi * ((u * 0.5) % 1.0))
    assert np.abs(got - ref).max() <= PER_TERM * k
    bad = u.copy()
    bad[70], bad[300] = np.nan, -np.inf
    x = host(swv.predict_direct(*(dev(a, torch) for a in (bad, v, w, l, m, f)), prec="f32c"))
    with pytest.raises(swv.SwvError):
        swv.synchronize()
    keep = ~np.isin(np.arange(n), (70, 300))
    assert np.isnan(x[~keep]).all() and np.abs(x[keep] - ref[keep]).max() <= PER_TERM * k


def test_a_row_keeps_its_bits_beside_far_rows(env):
    torch, swv = env
    rng = np.random.default_rng(6)
    u, v, w = (rng.uniform(-5e4, 5e4, 300) for _ in range(3))
    l, m, f = rng.uniform(-0.03, 0.03, 50), rng.uniform(-0.03, 0.03, 50), rng.lognormal(-3, 1, 50)
    run = lambda a: host(swv.predict_direct(*(dev(x, torch) for x in (a, v, w, l, m, f)), prec="f32c"))
    alone = run(u)
    u2 = u.copy()
    u2[[0, 130, 299]] = 4e5, 3e7, -2e6
    keep = ~np.isin(np.arange(300), (0, 130, 299))
    assert np.array_equal(run(u2)[keep], alone[keep])
