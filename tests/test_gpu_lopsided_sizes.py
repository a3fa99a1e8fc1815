"""Calls with one dimension tiny and the other large take about the time of their
bytes: within five times a copy of what their kernels read and write."""
import numpy as np
import pytest

from .gpu_util import dev, note, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    return require_gpu()


def best_us(torch, call, least_ms=30.0, runs=20):
    """Least time of a call, in runs of four after least_ms of them (the clock settles)."""
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    best, spent, done = float("inf"), 0.0, 0
    while done < runs:
        a.record()
        for _ in range(4):
            call()
        b.record()
        b.synchronize()
        t = a.elapsed_time(b)
        spent += t
        if spent > least_ms:
            best, done = min(best, 250.0 * t), done + 1
    return best


def copy_us(torch, n_bytes):
    x = torch.zeros(n_bytes // 16, dtype=torch.float64, device="cuda")   # read and written
    y = torch.empty_like(x)
    return best_us(torch, lambda: y.copy_(x))


@pytest.mark.parametrize("prec", ["fp64", "f32c"])
def test_adjoint_of_one_row(env, prec):
    torch, swv = env
    n = 6_000_000
    r = [dev(np.array([x]), torch) for x in (10.0, -20.0, 3.0)]
    y = torch.ones(1, dtype=torch.complex128, device="cuda")
    l = torch.linspace(-0.3, 0.3, n, dtype=torch.float64, device="cuda")
    t = best_us(torch, lambda: swv.adjoint(*r, y, l, l, l, prec=prec))
    least = copy_us(torch, (24 + 16 + 32) * n)   # directions, image, one set of partial sums
    note(f"adjoint {prec}, 1 row x {n} pixels: {t:.0f} us, a copy of its bytes {least:.0f}")
    assert t <= 5 * least


def test_gradients_of_one_row(env):
    torch, swv = env
    n = 1_000_000
    r = [dev(np.array([x]), torch) for x in (10.0, -20.0, 3.0)]
    y = torch.ones(1, dtype=torch.complex128, device="cuda")
    l = torch.linspace(-0.3, 0.3, n, dtype=torch.float64, device="cuda")
    t = best_us(torch, lambda: swv.grad_direct(*r, y, l, l, l))
    # components, packed (read twice), sums written and read, gradients
    least = copy_us(torch, (24 + 96 + 64 + 24) * n)
    note(f"gradients, 1 row x {n} components: {t:.0f} us, a copy of its bytes {least:.0f}")
    assert t <= 5 * least


@pytest.mark.parametrize("rows,pixels", [(100, 10_000), (64, 30_000), (300, 3_000)])
def test_small_adjoint(env, rows, pixels):
    """Little work for the chip: about the time of the same pixels' ten rows (the
    call's own), not a few waves' chain of many pixels each."""
    torch, swv = env
    rng = np.random.default_rng(1)
    r = [dev(rng.uniform(-1e4, 1e4, rows), torch) for _ in range(3)]
    y = torch.ones(rows, dtype=torch.complex128, device="cuda")
    l = dev(rng.uniform(-0.3, 0.3, pixels), torch)
    n = -0.5 * l * l
    t = best_us(torch, lambda: swv.adjoint(*r, y, l, l, n))
    ten = best_us(torch, lambda: swv.adjoint(*(a[:10] for a in r), y[:10], l, l, n))
    note(f"adjoint, {rows} rows x {pixels} pixels: {t:.1f} us, ten rows {ten:.1f}")
    assert t <= 1.4 * ten


@pytest.mark.parametrize("rows,comps", [(10_000_000, 5), (10_000_000, 16), (1_000_000, 32)])
def test_f32c_sum_of_a_short_list(env, rows, comps):
    """A term costs about what it does in a long list, beside the rows' own bytes."""
    torch, swv = env
    rng = np.random.default_rng(2)
    r = [dev(rng.uniform(-1e4, 1e4, rows), torch) for _ in range(3)]
    c = [dev(rng.uniform(-0.3, 0.3, 1000), torch) for _ in range(3)]
    out = torch.empty(rows, dtype=torch.complex64, device="cuda")
    call = lambda k: swv.predict_direct(*r, *(a[:k] for a in c), prec="f32c", out=out)
    t, full = best_us(torch, lambda: call(comps)), best_us(torch, lambda: call(1000))
    least = max(full * comps / 1000, copy_us(torch, 32 * rows))
    note(f"f32c, {rows} rows x {comps} components: {t:.1f} us; share of 1000 or bytes {least:.1f}")
    assert t <= 1.4 * least + 5.0   # 5 us: the packing's launch and the rest of the call


def _image_rows(torch, n):
    rng = np.random.default_rng(3)
    r = [dev(rng.uniform(-1e4, 1e4, n), torch) for _ in range(3)]
    return r, torch.ones(n, dtype=torch.complex128, device="cuda")


@pytest.mark.parametrize("nx,ny", [(64, 64), (100, 60)])
def test_image_of_few_rows(env, nx, ny):
    """About the time of ten rows, the call's own."""
    torch, swv = env
    r, y = _image_rows(torch, 100)
    call = lambda n: swv.dirty_image(*(a[:n] for a in r), y[:n], nx, ny, 0.0005)
    t, ten = best_us(torch, lambda: call(100)), best_us(torch, lambda: call(10))
    note(f"image {nx} x {ny}, 100 rows: {t:.1f} us, ten rows {ten:.1f}")
    assert t <= 1.5 * ten


@pytest.mark.parametrize("prec,rows,nx,ny", [("fp64", 100_000, 1, 300), ("fp64", 10_000, 300, 2),
                                             ("f32c", 1000, 256, 256), ("f32c", 1000, 128, 128)])
def test_image_against_the_adjoint_of_its_pixels(env, prec, rows, nx, ny):
    """No slower than the general route, whose half is thrown away."""
    torch, swv = env
    r, y = _image_rows(torch, rows)
    lmn = swv.image_grid(nx, ny, 0.0005)
    t = best_us(torch, lambda: swv.dirty_image(*r, y, nx, ny, 0.0005, prec=prec))
    adj = best_us(torch, lambda: swv.adjoint(*r, y, *lmn, prec=prec))
    note(f"image {prec} {nx} x {ny}, {rows} rows: {t:.1f} us, adjoint {adj:.1f}")
    # 8 us: the general FP64 route has two more launches
    assert t <= 1.1 * adj + (8.0 if prec == "fp64" else 0.0)
