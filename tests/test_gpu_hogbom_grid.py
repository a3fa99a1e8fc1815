"""Hogbom cycle over many workgroups: the sizes where the split changes, bit for
bit against the oracle, and a captured call on a size that would run grid-wide."""
import numpy as np
import pytest

from oracle import clean as oc

from .gpu_util import host, note, require_gpu
from .test_gpu_clean import _beam_like, _hogbom_gpu, _image_like


@pytest.fixture(scope="module")
def env():
    return require_gpu()


@pytest.mark.gpu
@pytest.mark.parametrize("ny,nx", [(71, 72), (64, 80), (1, 5121), (5632, 1), (363, 361),
                                   (363, 363), (520, 530)])
def test_sizes_bitwise(env, ny, nx):
    """One below and at the smallest grid-wide size, one pixel in the last
    workgroup, and more pixels than 256 workgroups hold at two per thread."""
    torch, swv = env
    rng = np.random.default_rng(ny + 5 * nx)
    beam = _beam_like(rng, ny, nx, quantum=1 / 64)
    img = _image_like(rng, ny, nx, beam, n_src=5, quantum=1 / 16)
    for gain, thr, k, absolute in ((0.2, 0.0, 60, False), (0.5, 0.1, 90, True)):
        note(f"hogbom {ny}x{nx} gain={gain} k={k} abs={absolute}")
        got = _hogbom_gpu(torch, swv, img, beam, gain, thr, k, absolute)
        ref = oc.hogbom(img, beam, gain, thr, k, absolute)
        for g, r in zip(got, ref):
            assert np.array_equal(g, r)


@pytest.mark.gpu
def test_captured_call(env):
    torch, swv = env
    from paper_1909_03956_amd.api import _ptr, check, context, lib
    ny, nx, k = 80, 81, 50
    rng = np.random.default_rng(4)
    beam = _beam_like(rng, ny, nx)
    img = _image_like(rng, ny, nx, beam)
    t_beam = torch.as_tensor(beam, device="cuda")
    t_img = torch.as_tensor(img, device="cuda")
    pix = torch.empty(k, dtype=torch.int64, device="cuda")
    val = torch.empty(k, dtype=torch.float64, device="cuda")
    n = torch.zeros(1, dtype=torch.int64, device="cuda")
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    note("captured hogbom 80x81")
    with torch.cuda.stream(s):
        ctx = context(t_img.device)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        check(lib().swv_hogbom(ctx.handle, nx, ny, _ptr(t_img), _ptr(t_beam), 0.1, 0.0, k, 0,
                               _ptr(pix), _ptr(val), _ptr(n)))
    ref = oc.hogbom(img, beam, 0.1, 0.0, k, False)
    for _ in range(3):
        t_img.copy_(torch.as_tensor(img))
        g.replay()
        torch.cuda.synchronize()
        found = int(n.item())
        for a, r in zip((host(t_img), host(pix)[:found], host(val)[:found]), ref):
            assert np.array_equal(a, r)
