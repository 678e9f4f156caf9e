"""Calls of one context issued in turn on two streams give the results of one stream."""
import numpy as np
import pytest

from paper_1504_06570_amd.scene import configs as C
from paper_1504_06570_amd.scene.readout import Readout

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


def test_readouts_between_traces(phx):
    """The context's readout scratch (its lists, counters and thresholds) serves one call at a time."""
    import torch
    scene = C.telescope(scale=2e-3)
    tr = phx.Tracer(scene)
    rng = np.random.default_rng(2)
    images, params = [], []
    for k in range(6):
        img = rng.poisson(30.0, (512, 512)).astype(np.int32)
        img[rng.integers(0, 512, 40), rng.integers(0, 512, 40)] = 200000
        images.append(torch.from_numpy(img).cuda())
        params.append(Readout(seed=k, amp_nx=2, amp_ny=2, cte_parallel=1 - 10.0 ** -(3 + k % 3)))
    want = [tr.readout(i, p) for i, p in zip(images, params)]
    ref = tr.trace(seed=5)[0]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    traced = [tr.new_image() for _ in images]
    got = []
    torch.cuda.synchronize()
    for k, (i, p) in enumerate(zip(images, params)):
        with torch.cuda.stream(streams[k % 2]):
            got.append(tr.readout(i, p))
        tr.trace(traced[k], seed=5, stream=streams[(k + 1) % 2])
    torch.cuda.synchronize()
    for w, v, t in zip(want, got, traced):
        assert torch.equal(w, v) and torch.equal(t, ref)
    tr.close()
