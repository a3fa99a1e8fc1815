"""Calls whose kernels need 2^32 threads or more in all, which no single launch
takes: layouts that give a row several threads, at row counts past that border."""
import numpy as np
import pytest

from oracle import visibility as ov

from .gpu_util import fp64_row_bound, host, note, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch, swv = require_gpu()
    yield torch, swv
    torch.cuda.empty_cache()


def _room(torch, need):
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    free, _ = torch.cuda.mem_get_info()
    if free < need + (8 << 30):
        pytest.skip(f"needs {need / 2**30:.0f} GiB of free device memory")


def _rows(rng, n, border):
    """Sampled rows, those around the border and the last ones among them."""
    return np.unique(np.concatenate([rng.integers(0, n, 300), np.arange(n - 300, n),
                                     np.arange(border - 20, min(border + 20, n))]))


def _track(torch, n):
    """One coordinate for all three axes (8 bytes a row), from the row index."""
    return torch.arange(n, dtype=torch.float64, device="cuda").mul_(3.7e-7).add_(0.1).sin_().mul_(2e4)


def test_direct_sum_of_long_lists_past_2_31_rows(env):
    """600 components: four rows a lane over eight waves, two threads a row."""
    torch, swv = env
    n, k = (1 << 31) + 300, 600
    _room(torch, 24 * n)
    note(f"direct sum, {n} rows x {k} components")
    rng = np.random.default_rng(3)
    l, m, f = rng.uniform(-0.02, 0.02, k), rng.uniform(-0.02, 0.02, k), rng.lognormal(-3, 1, k)
    L, M, F = (torch.as_tensor(a, device="cuda") for a in (l, m, f))
    x = _track(torch, n)
    out = torch.empty(n, dtype=torch.complex128, device="cuda")
    swv.predict_direct(x, x, x, L, M, F, out=out)
    swv.synchronize()
    rows = _rows(rng, n, 1 << 31)
    idx = torch.as_tensor(rows, device="cuda")
    xs = host(x[idx])
    ref = ov.predict_direct(xs, xs, xs, l, m, f)
    bound = fp64_row_bound(xs, xs, xs, l, m, ov.n_minus_1(l, m), f)
    assert np.all(np.abs(host(out[idx]) - ref) <= bound)


def test_batched_plan_past_2_31_rows(env):
    """512 threads to every 256 rows; the same bits as the single call."""
    torch, swv = env
    n, k = (1 << 31) + 300, 500
    _room(torch, (8 + 16 + 24) * n)
    note(f"batched plan, {n} rows x {k} components")
    rng = np.random.default_rng(4)
    l, m, f = rng.uniform(-0.02, 0.02, k), rng.uniform(-0.02, 0.02, k), rng.lognormal(-3, 1, k)
    L, M, F = (torch.as_tensor(a, device="cuda") for a in (l, m, f))
    x = _track(torch, n)
    out = torch.empty(n, dtype=torch.complex128, device="cuda")
    plan = swv.BatchPlan([dict(route="direct", u=x, v=x, w=x, l=L, m=M, flux=F, out=out)])
    plan.run()
    swv.synchronize()
    plan.close()
    idx = torch.as_tensor(_rows(rng, n, 1 << 31), device="cuda")
    xs = x[idx]
    assert torch.equal(out[idx], swv.predict_direct(xs, xs, xs, L, M, F))


def test_degridding_of_2_28_rows(env):
    """16 lanes a row at support 9; planes small enough that rows stay unsorted."""
    torch, swv = env
    n, nx = (1 << 28) + 40, 12
    _room(torch, 40 * n)
    note(f"degridding, {n} rows, support 9")
    rng = np.random.default_rng(5)
    img = torch.as_tensor(rng.lognormal(-1, 1, (nx, nx)), device="cuda")
    x = _track(torch, n).mul_(0.01)
    out, st = swv.predict_degrid(img, x, x, x, 0.003, support=9)
    assert st["plane_bytes"] <= 4 << 20
    rows = torch.as_tensor(_rows(rng, n, 1 << 28), device="cuda")
    # the same w range, so the same planes, by way of its ends
    ends = torch.stack([x.argmin(), x.argmax()])
    rows = torch.cat([rows, ends])
    xs = x[rows]
    assert torch.equal(out[rows], swv.predict_degrid(img, xs, xs, xs, 0.003, support=9)[0])
