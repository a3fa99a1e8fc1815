"""The wavelet route as a sum over the leaves with the weights its coefficients
give: leaf counts around the summation order's ranges (one leaf to thousands,
fewer than the direct sum's table takes among them), row counts around the
layouts, both precisions, alone and batched, exact and thresholded, against
the oracle's traversal."""
import numpy as np
import pytest

from oracle import threshold as oth
from oracle import tree as ot

from .gpu_util import dev, fp64_row_bound, host, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    return require_gpu()


@pytest.mark.parametrize("J,k,n,frac", [
    (1, 1, 1, None), (2, 15, 65, None), (5, 16, 513, 0.3), (9, 17, 1025, 0.0), (12, 33, 351, 0.1),
    (8, 255, 20001, None), (10, 257, 63, 0.5), (11, 900, 140001, None), (16, 3, 70001, 0.7),
    (25, 5, 1300003, None), (14, 4100, 351, None)])
def test_edges_against_the_traversal(env, J, k, n, frac):
    torch, swv = env
    rng = np.random.default_rng(100 * J + k + n)
    u, v, w = (rng.uniform(-2e4, 2e4, n) for _ in range(3))
    half = 0.4 if J < 5 else 0.04
    l, m, f = rng.uniform(-half, half, k), rng.uniform(-half, half, k), rng.lognormal(-3, 1, k)
    t, rt = swv.Tree(J, 1.1, 0.4, l, m, f), ot.build_tree(J, 1.1, 0.4, l, m, f)
    if frac is not None:
        keep = oth.retained(rt, frac)
        t = t.prune(keep)
    U, V, W = dev(u, torch), dev(v, torch), dev(w, torch)
    got, got32 = t.predict(U, V, W), t.predict(U, V, W, prec="f32c")
    outs = [torch.empty(n, dtype=d, device="cuda") for d in (torch.complex128, torch.complex64)]
    plan = swv.BatchPlan([dict(route="tree", prec=p, tree=t, u=U, v=V, w=W, out=o)
                          for p, o in zip(("fp64", "f32c"), outs)])
    plan.run()
    swv.synchronize()
    assert torch.equal(got, outs[0]) and torch.equal(got32, outs[1])
    assert torch.equal(got32, got.to(torch.complex64))
    rows = np.unique(np.linspace(0, n - 1, min(n, 200)).astype(int))
    args = (u[rows], v[rows], w[rows])
    ref = ot.predict_tree(rt, *args) if frac is None else oth.predict_thresholded(rt, keep, *args)
    # the leaves' phase roundings (a thresholded tree's are fewer and nearer the
    # centre of theirs: the bound of the whole set, with the flux in one place,
    # covers them), and J + 2 roundings of the weights
    bound = fp64_row_bound(*args, rt.leaf_l, rt.leaf_m, rt.leaf_nm1, rt.leaf_flux)
    if frac is not None:
        far = np.argmax(rt.leaf_l ** 2 + rt.leaf_m ** 2)
        one = np.array([far])
        bound = bound + 4 * fp64_row_bound(*args, rt.leaf_l[one], rt.leaf_m[one], rt.leaf_nm1[one],
                                           np.array([np.abs(f).sum()]))
    assert np.all(np.abs(host(got)[rows] - ref) <= bound + (J + 2) * 4e-16 * np.abs(f).sum())
    plan.close()
