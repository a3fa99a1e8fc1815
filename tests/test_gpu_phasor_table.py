"""FP64 direct sum with the table phasor: the borders of its dispatch and of its
summation order (component counts around the shortest list, ranges and
sub-ranges; row counts around its tiles and layouts), every layout the same
bits, and phases beyond the table's direct reach."""
import numpy as np
import pytest

from oracle import visibility as ov

from .gpu_util import dev, fp64_row_bound, host, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    return require_gpu()


def _case(rng, n_vis, n_comp, scale=2e5):
    u, v, w = (rng.uniform(-scale, scale, n_vis) for _ in range(3))
    l, m = rng.uniform(-0.03, 0.03, n_comp), rng.uniform(-0.03, 0.03, n_comp)
    return u, v, w, l, m, rng.lognormal(-3, 1, n_comp)


def _run(env, u, v, w, l, m, f, sign=-1):
    torch, swv = env
    out = swv.predict_direct(*(dev(a, torch) for a in (u, v, w, l, m, f)), sign=sign)
    swv.synchronize()
    return host(out)


@pytest.mark.parametrize("n_vis,n_comp", [
    (1, 15), (1, 16), (65, 17), (511, 31), (513, 255), (1025, 256), (63, 257), (351, 2049),
    (64, 4097), (20001, 33), (70001, 129), (140001, 64)])
def test_edges_against_oracle_and_batched(env, n_vis, n_comp):
    """Layouts chosen from one row to many (components shared by workgroups,
    by waves, or whole rows per wave) against the oracle; the batched kernel,
    which gives every row to one wave, has the same bits."""
    torch, swv = env
    u, v, w, l, m, f = _case(np.random.default_rng(n_vis + 7 * n_comp), n_vis, n_comp)
    got = _run(env, u, v, w, l, m, f)
    rows = np.unique(np.linspace(0, n_vis - 1, min(n_vis, 300)).astype(int))
    ref = ov.predict_direct(u[rows], v[rows], w[rows], l, m, f)
    bound = fp64_row_bound(u[rows], v[rows], w[rows], l, m, ov.n_minus_1(l, m), f)
    assert np.all(np.abs(got[rows] - ref) <= bound)
    out = torch.empty(n_vis, dtype=torch.complex128, device="cuda")
    d = {k: dev(a, torch) for k, a in zip(("u", "v", "w", "l", "m", "flux"), (u, v, w, l, m, f))}
    plan = swv.BatchPlan([{"route": "direct", "out": out, "sign": -1, **d}])
    plan.run()
    swv.synchronize()
    assert np.array_equal(host(out), got)


def test_phases_beyond_the_cells(env):
    """Rows whose phases are whole turns or quarters far above 2^39 (exact in
    FP64) beside ordinary ones: the exact values, and the ordinary rows keep
    the bits they have alone."""
    rng = np.random.default_rng(5)
    n, k = 200, 20
    u = rng.uniform(-1e4, 1e4, n)
    v, w = np.zeros(n), np.zeros(n)
    l, m, f = np.full(k, 0.5), np.zeros(k), np.ones(k)
    alone = _run(env, u, v, w, l, m, f)
    u2 = u.copy()
    u2[17] = 2.0 ** 45 + 2.0        # half of it: a whole number of turns
    u2[40] = 2.0 ** 45 + 0.5        # a quarter turn more
    u2[41] = -2.0 ** 45 - 0.5
    got = _run(env, u2, v, w, l, m, f)
    ref = {17: 1.0, 40: -1j, 41: 1j}
    for j, x in ref.items():
        assert abs(got[j] - k * x) <= k * 1e-15, j
    keep = [j for j in range(n) if j not in ref]
    assert np.array_equal(got[keep], alone[keep])


def test_non_finite_rows_stay_apart(env):
    torch, swv = env
    u, v, w, l, m, f = _case(np.random.default_rng(6), 130, 40)
    clean = _run(env, u, v, w, l, m, f)
    u[3], v[70] = np.nan, np.inf
    out = swv.predict_direct(*(dev(a, torch) for a in (u, v, w, l, m, f)))
    with pytest.raises(swv.SwvError):
        swv.synchronize()
    got = host(out)
    assert np.isnan(got[3]) and np.isnan(got[70])
    keep = [j for j in range(130) if j not in (3, 70)]
    assert np.array_equal(got[keep], clean[keep])
