"""FP64 direct sums of fluxes near the top of FP64's range: a power of two times the
fluxes gives that power times the visibilities, bit for bit, as long as these stay
finite, in lists on either side of the table kernels' shortest one and in the
layouts that share components."""
import numpy as np
import pytest

from .gpu_util import dev, host, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    return require_gpu()


@pytest.mark.parametrize("n_vis,n_comp", [(100, 7), (351, 16), (351, 5000), (20001, 900),
                                          (300001, 600), (1100001, 17)])
def test_sums_scale_with_the_flux(env, n_vis, n_comp):
    torch, swv = env
    rng = np.random.default_rng(n_vis + n_comp)
    u, v, w = (rng.uniform(-1e4, 1e4, n_vis) for _ in range(3))
    u[0] = v[0] = w[0] = 0.0   # phases on the cells' nodes
    l, m = rng.uniform(-0.3, 0.3, n_comp), rng.uniform(-0.3, 0.3, n_comp)
    f = rng.lognormal(-3, 1, n_comp) * 2.0 ** -20
    f[:7] = rng.uniform(1, 2, 7) * rng.choice([-1, 1], 7)
    rows, L, M = [dev(a, torch) for a in (u, v, w)], dev(l, torch), dev(m, torch)
    scale = 2.0 ** 1019
    out = torch.empty(n_vis, dtype=torch.complex128, device="cuda")
    plan = swv.BatchPlan([dict(zip(("u", "v", "w"), rows), route="direct", l=L, m=M,
                               flux=dev(f * scale, torch), out=out)])
    plan.run()
    got = host(swv.predict_direct(*rows, L, M, dev(f * scale, torch)))
    swv.synchronize()
    plan.close()
    ref = host(swv.predict_direct(*rows, L, M, dev(f, torch)))
    assert np.isfinite(got).all() and np.array_equal(got, host(out))
    assert np.array_equal(got.view(np.float64), ref.view(np.float64) * scale)
