"""Calls of one context issued in turn on two streams give the results of one stream."""
import pytest

from paper_1504_06570_amd.scene import configs as C

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def phx():
    from paper_1504_06570_amd import phx
    return phx


def test_gradients_of_moments(phx):
    """Each call's cotangent coefficients, which the context holds, are those its own adjoint reads."""
    import torch
    scene = C.gradients(scale=2e-3, screen_n=128)      # 25 sources of 2e4 photons
    tr = phx.Tracer(scene)
    flags = int(scene.physics) | phx.F_CULL
    words = tr.new_moments()
    tr.trace(flags=flags, moments=words)
    g = torch.Generator(device="cuda").manual_seed(1)
    dmom = [torch.randn((25, 5), generator=g, device="cuda", dtype=torch.float64) for _ in range(8)]
    want = [tr.adjoint_moments(words, d, flags=flags) for d in dmom]
    got = [torch.zeros_like(w) for w in want]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for k, d in enumerate(dmom):
        tr.adjoint_moments(words, d, flags=flags, grad=got[k], stream=streams[k % 2])
    torch.cuda.synchronize()
    for w, v in zip(want, got):
        assert w.abs().sum() > 0 and torch.equal(w, v)
    tr.close()
