"""Small predictions with long lists, whose workgroups share components by way of
partial sums in memory, inside a caller's graph: captured after a call of many rows
only, so that the partial sums' buffer would have to be made during the capture, and
replayed after other calls have grown the context's workspaces."""
import numpy as np
import pytest

from .gpu_util import dev, dev_c, host, note, require_gpu

pytestmark = pytest.mark.gpu
K, N, MANY = 5000, 351, 200_001


@pytest.fixture(scope="module")
def env():
    return require_gpu()


@pytest.mark.parametrize("warm", [False, True])
@pytest.mark.parametrize("route,prec", [("direct", "fp64"), ("direct", "f32c"), ("tree", "fp64"),
                                        ("tree", "f32c"), ("leaves", "f32c")])
def test_captured_small_call(env, route, prec, warm):
    torch, swv = env
    rng = np.random.default_rng(9)
    u, v, w = (rng.uniform(-1e4, 1e4, MANY) for _ in range(3))
    l, m, f = rng.uniform(-0.4, 0.4, K), rng.uniform(-0.4, 0.4, K), rng.lognormal(-3, 1, K)
    U, V, W, L, M, F = (dev(a, torch) for a in (u, v, w, l, m, f))
    small = [a[:N].contiguous() for a in (U, V, W)]
    t = swv.Tree(9, 1.1, 0.4, l, m, f)
    assert t.stats()["n_leaves"] > 4200
    call = {"direct": lambda *r, out=None: swv.predict_direct(*r, L, M, F, prec=prec, out=out),
            "tree": lambda *r, out=None: t.predict(*r, prec=prec, out=out),
            "leaves": lambda *r, out=None: t.predict_leaves(*r, prec=prec, out=out)}[route]
    out = torch.zeros(N, dtype=torch.complex128 if prec == "fp64" else torch.complex64,
                      device="cuda")
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    note(f"captured small call: {route} {prec}, after {'the same' if warm else 'a large one only'}")
    with torch.cuda.stream(s):
        ctx = swv.context(U.device)
        call(U, V, W)
        if warm:
            call(*small)
        s.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        call(*small, out=out)
    with torch.cuda.stream(s):
        ref = call(*small)
        for n in (500, 60_000):   # workspaces grow between the replays
            out.zero_()
            y = dev_c(np.ones(MANY), torch)
            swv.adjoint(U, V, W, y, *(torch.zeros(n, dtype=torch.float64, device="cuda"),) * 3)
            swv.dirty_image(U, V, W, y, 100, 90, 0.001)
            scribble = torch.full((1 << 22,), 7.0, dtype=torch.float64, device="cuda")
            s.synchronize()
            g.replay()
            s.synchronize()
            assert torch.equal(out, ref)
            assert float(scribble.min()) == float(scribble.max()) == 7.0
        ctx.synchronize()
    assert np.isfinite(host(out)).all()
    t.close()


@pytest.mark.parametrize("k", [7, 16, 4000])
@pytest.mark.parametrize("warm,captured", [("f32c", "fp64"), ("fp64", "f32c"), ("grad", "fp64"),
                                           ("fp64", "grad")])
def test_a_call_of_another_kind_is_warm_up_enough(env, k, warm, captured):
    """Calls that pack the same list: the captured one finds its buffer made."""
    torch, swv = env
    rng = np.random.default_rng(k)
    u, v, w = (rng.uniform(-1e4, 1e4, 20000) for _ in range(3))
    l, m, f = rng.uniform(-0.4, 0.4, k), rng.uniform(-0.4, 0.4, k), rng.lognormal(-3, 1, k)
    rows, comps = [dev(a, torch) for a in (u, v, w)], [dev(a, torch) for a in (l, m, f)]
    y = dev_c(np.ones(u.size), torch)

    def call(kind):
        if kind == "grad":
            return torch.stack(swv.grad_direct(*rows, y, *comps))
        return swv.predict_direct(*rows, *comps, prec=kind)

    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    note(f"captured {captured} after {warm}, {k} components")
    with torch.cuda.stream(s):
        swv.api._CONTEXTS.pop((0, s.cuda_stream), None)   # a context of its own
        call(warm)
        # the adjoint of the components' directions has the gradients' other workspace
        z = torch.zeros(3 * k, dtype=torch.float64, device="cuda")
        swv.adjoint(*rows, y, z, z, z)
        s.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        out = call(captured)
    with torch.cuda.stream(s):
        ref = call(captured)
        for _ in range(3):
            out.zero_()
            g.replay()
            s.synchronize()
            assert torch.equal(out, ref)
        swv.context(rows[0].device).synchronize()
