"""The autotuner leaves no call slower than the defaults do."""
import numpy as np
import pytest

from .gpu_util import dev, note, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    return require_gpu()


def _best_ms(torch, call):
    """Least time of a call in 30 runs of four, after 50 ms of them (the clock settles)."""
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    best, spent = float("inf"), 0.0
    runs = 0
    while runs < 30:
        a.record()
        for _ in range(4):
            call()
        b.record()
        b.synchronize()
        t = a.elapsed_time(b)
        spent += t
        if spent > 50.0:
            best = min(best, t / 4)
            runs += 1
    return best


def _tuned_and_default(torch, swv, family, call):
    """Times of the call as tuned and with the family's default shapes, in turn."""
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    tuned = default = float("inf")
    with torch.cuda.stream(s):
        swv.api._CONTEXTS.pop((0, s.cuda_stream), None)
        ctx = swv.context()
        shapes = [[ctx.tune_get(family, c) for c in (0, 1)]]
        ctx.autotune()
        shapes.append([ctx.tune_get(family, c) for c in (0, 1)])
        for _ in range(2):
            for k in (0, 1):
                for c in (0, 1):
                    ctx.tune_set(family, c, *shapes[k][c])
                t = _best_ms(torch, call)
                tuned, default = (tuned, min(t, default)) if k == 0 else (min(t, tuned), default)
    note(f"family {family}: default {shapes[0]} {default:.4f} ms, tuned {shapes[1]} {tuned:.4f} ms")
    return tuned, default


@pytest.mark.parametrize("rows,comps", [(1 << 18, 2048), (1_000_000, 1000)])
def test_direct_sum_keeps_its_layouts(env, rows, comps):
    """Tuned by whole rows per wave alone, these calls took a tenth longer."""
    torch, swv = env
    rng = np.random.default_rng(1)
    r = [dev(rng.uniform(-1e4, 1e4, rows), torch) for _ in range(3)]
    c = [dev(rng.uniform(-0.03, 0.03, comps), torch) for _ in range(3)]
    out = torch.empty(rows, dtype=torch.complex128, device="cuda")
    tuned, default = _tuned_and_default(torch, swv, 0, lambda: swv.predict_direct(*r, *c, out=out))
    assert tuned <= 1.04 * default
