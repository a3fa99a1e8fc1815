"""Short component lists around 3 x 2^20 rows, where a lane takes a second row: each row
is the same as in a call of its own part, for components and for a tree's leaves."""
import numpy as np
import pytest

from .gpu_util import dev, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    return require_gpu()


@pytest.mark.parametrize("n_comp", [1, 15])
@pytest.mark.parametrize("extra", [-1, 0, 1, 256, 257])
def test_rows_do_not_depend_on_the_rows_per_lane(env, n_comp, extra):
    torch, swv = env
    n = 3 * 2**20 + extra
    rng = np.random.default_rng(n_comp)
    r = [dev(rng.uniform(-1e4, 1e4, n), torch) for _ in range(3)]
    l, m, flux = (rng.uniform(-0.3, 0.3, n_comp), rng.uniform(-0.3, 0.3, n_comp),
                  rng.uniform(0.1, 1.0, n_comp))
    lmf = [dev(x, torch) for x in (l, m, flux)]
    tree = swv.Tree(20, 1.0, 0.4, l, m, flux)
    for call in (lambda *x: swv.predict_direct(*x, *lmf), tree.predict):
        whole = torch.view_as_real(call(*r))
        for a, b in ((0, 1000), (n // 2 - 500, n // 2 + 500), (n - 1000, n)):
            part = torch.view_as_real(call(*(x[a:b].contiguous() for x in r)))
            assert torch.equal(whole[a:b], part)
    tree.close()
