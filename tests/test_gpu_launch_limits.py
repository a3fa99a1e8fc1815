"""Calls whose kernels need 2^32 threads or more in all, which no single launch
takes: layouts that give a row, a pixel or a component several threads, past that
border."""
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


def test_image_sums_past_2_26_pixels_and_gradients_past_2_25_components(env):
    """Adding up chunks at 64 threads a pixel and 128 a component would take 2^32."""
    torch, swv = env
    rng = np.random.default_rng(6)
    u, v, w = (rng.uniform(-3e3, 3e3, 2) for _ in range(3))
    y = rng.normal(size=2) + 1j * rng.normal(size=2)
    rows = [torch.as_tensor(a, device="cuda") for a in (u, v, w, y)]
    n = (1 << 26) + 5
    note(f"adjoint, {n} pixels")
    l = torch.arange(n, dtype=torch.float64, device="cuda").mul_(1.3 / n).sub_(0.65)
    m = l.flip(0).mul_(0.3)
    nm1 = -(l * l + m * m) / (1 + torch.sqrt(1 - l * l - m * m))
    img = swv.adjoint(*rows, l, m, nm1)
    idx = torch.as_tensor(_rows(rng, n, 1 << 26), device="cuda")
    lp, mp, np_ = (host(a[idx]) for a in (l, m, nm1))
    ref = ov.adjoint(u, v, w, y, lp, mp, np_)
    # the same bound as a direct sum's, rows and pixels exchanged
    bound = fp64_row_bound(lp, mp, np_, u, v, w, np.abs(y))
    assert np.all(np.abs(host(img[idx]) - ref) <= bound)
    del img, nm1
    k = (1 << 25) + 3
    note(f"gradients, {k} components")
    f = torch.ones(k, dtype=torch.float64, device="cuda")
    g = swv.grad_direct(*rows, l[:k], m[:k], f)
    idx = torch.as_tensor(_rows(rng, k, 1 << 25), device="cuda")
    lp, mp = host(l[idx]), host(m[idx])
    gr = ov.grad_direct(u, v, w, y, lp, mp, np.ones(lp.size))
    nm1 = ov.n_minus_1(lp, mp)
    err = fp64_row_bound(lp, mp, nm1, u, v, w, np.abs(y))
    wide = 4 * np.pi * np.abs([u, v, w]).max(axis=1).sum() / (1 + nm1)   # |d phi / dl|, |d phi / dm|
    for a, b, s in zip(g, gr, (1.0, wide, wide)):
        assert np.all(np.abs(host(a[idx]) - b) <= s * err)
    swv.synchronize()


def test_dirty_image_of_2_26_pixels_about_its_corner(env):
    torch, swv = env
    rng = np.random.default_rng(7)
    u, v, w = (rng.uniform(-300, 300, 3) for _ in range(3))
    y = rng.normal(size=3) + 1j * rng.normal(size=3)
    n, cell = 8192, 0.7 / 8192
    note(f"dirty image, {n} x {n} pixels about the corner")
    img = swv.dirty_image(*(torch.as_tensor(a, device="cuda") for a in (u, v, w, y)), n, n, cell, 0, 0)
    p = np.unique(np.concatenate([rng.integers(0, n * n, 500), np.arange(n * n - 300, n * n)]))
    got = host(img.reshape(-1)[torch.as_tensor(p, device="cuda")])
    l, m = (p % n) * cell, (p // n) * cell
    nm1 = ov.n_minus_1(l, m)
    ref = ov.adjoint(u, v, w, y, l, m, nm1).real / 3
    bound = fp64_row_bound(l, m, nm1, u, v, w, np.abs(y)) / 3
    assert np.all(np.abs(got - ref) <= bound)
