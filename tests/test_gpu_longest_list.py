"""The longest component list, 2^31 - 1: a border of the summation order is an
index that 32 bits hold only just.  Unit sources in the phase centre's direction:
the sum is their number, exactly in FP64."""
import pytest

from .gpu_util import note, require_gpu

pytestmark = pytest.mark.gpu


def test_two_to_the_31_less_one_components():
    torch, swv = require_gpu()
    n = (1 << 31) - 1
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    free, _ = torch.cuda.mem_get_info()
    need = n * (16 + 80) + (8 << 30)   # two arrays, the packed list with its headroom
    if free < need:
        pytest.skip(f"needs {need / 2**30:.0f} GiB of free device memory")
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        swv.api._CONTEXTS.pop((0, s.cuda_stream), None)   # a context to be closed below
        zero = torch.zeros(n, dtype=torch.float64, device="cuda")
        one = torch.ones(n, dtype=torch.float64, device="cuda")
        u = torch.linspace(-1e3, 1e3, 64, dtype=torch.float64, device="cuda")
        for prec in ("fp64", "f32c"):
            note(f"direct {prec}, 64 rows x {n} components")
            got = swv.predict_direct(u, u, u, zero, zero, one, prec=prec)
            if prec == "fp64":
                assert torch.equal(got, torch.full_like(got, float(n)))
            else:
                assert float((got - n).abs().max()) <= 2.0 ** -23 * n
        swv.synchronize()
        ctx = swv.api._CONTEXTS.pop((0, s.cuda_stream))
        ctx.close()
        del zero, one, got
    torch.cuda.empty_cache()
