"""GPU readout chain (phx_readout, through the C ABI) against the CPU oracle: the electrons after
bleeding and defects, after the parallel and after the serial transfers bit for bit, and the
digitised ADU value for value (values whose digitiser floors sit within 1e-9 of an integer in the
oracle may differ by the rounding of the two implementations)."""
import numpy as np
import pytest

import oracle as O
from paper_1504_06570_amd.scene import configs as C
from paper_1504_06570_amd.scene.readout import Readout

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def phx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1504_06570_amd import phx as P
    return P


def _image(ny=256, nx=256, seed=0):
    rng = np.random.default_rng(seed)
    img = rng.poisson(40.0, (ny, nx)).astype(np.uint32)
    # bright spots that saturate and bleed, one near the implant
    for (fy, fx, n) in ((0.16, 0.12, 900000), (0.78, 0.5 - 1.0 / nx, 2500000),
                        (0.47, 0.78, 150000), (0.04, 0.98, 99999)):
        img[int(fy * ny), int(fx * nx)] = n
    return img


def run_both(P, img, rp):
    import torch
    tr = P.Tracer(C.tiny(scale=1e-4))
    dev = torch.from_numpy(img.view(np.int32)).cuda()
    out, work, par, ser = tr.readout(dev, rp, stages=True)
    torch.cuda.synchronize()
    g = [t.cpu().numpy() for t in (out, work, par, ser)]
    tr.close()
    o_out, margin, o_work, o_par, o_ser = O.readout(rp, img)
    return g, (o_out, margin, o_work, o_par, o_ser)


def check(g, o):
    g_out, g_work, g_par, g_ser = g
    o_out, margin, o_work, o_par, o_ser = o
    assert np.array_equal(g_work.view(np.uint32), o_work)
    assert np.array_equal(g_par.view(np.uint32), o_par)
    assert np.array_equal(g_ser.view(np.uint32), o_ser)
    ga = g_out.view(np.uint16)
    diff = ga != o_out
    assert not (diff & (margin >= 1e-9)).any(), np.argwhere(diff & (margin >= 1e-9))[:5]
    return int(diff.sum())


@pytest.mark.parametrize("layout", [(4, 2, 8, 6), (1, 1, 0, 0), (8, 2, 3, 5)])
def test_readout_parity(phx, layout):
    """Bleeding, dark current, hot/dead pixels, hot columns, transfer trails (inefficiencies raised
    to 1e-4 / 5e-5 so that many electrons are delayed), read noise, non-linearity and bit errors
    on a 256 x 256 image with saturating spots, for several amplifier layouts."""
    ax, ay, ox, oy = layout
    rp = Readout(amp_nx=ax, amp_ny=ay, over_x=ox, over_y=oy, hot_fraction=2e-3,
                 dead_fraction=2e-3, hot_column_fraction=2e-4, cte_parallel=1 - 1e-4,
                 cte_serial=1 - 5e-5, dark_rate=1.0)
    g, o = run_both(phx, _image(), rp)
    assert check(g, o) <= 2
    # the spots bled: a full well plateau around each
    assert (o[2] == rp.full_well).sum() > 30


def test_readout_of_a_traced_image(phx):
    """The trace's image of the telescope field read out on the device equals the oracle's readout
    of the same image."""
    import torch
    s = C.telescope(scale=0.02)
    tr = phx.Tracer(s)
    img, _, _, _ = tr.trace()
    rp = Readout(seed=7)
    out, work, par, ser = tr.readout(img, rp, stages=True)
    torch.cuda.synchronize()
    host = img.cpu().numpy().view(np.uint32)
    g = [t.cpu().numpy() for t in (out, work, par, ser)]
    tr.close()
    o = O.readout(rp, host)
    assert host.sum() > 0
    assert check(g, o) <= 2


def test_readout_repeats_and_scratch_buffers(phx):
    """Two calls give the same ADU, with caller buffers or the context's scratch."""
    import torch
    img = torch.from_numpy(_image(128, 128, seed=3).view(np.int32)).cuda()
    rp = Readout(amp_nx=2, amp_ny=2, cte_parallel=1 - 1e-4)
    tr = phx.Tracer(C.tiny(scale=1e-4))
    a = tr.readout(img, rp)
    b = tr.readout(img, rp)
    c, _, _, _ = tr.readout(img, rp, stages=True)
    torch.cuda.synchronize()
    assert torch.equal(a, b) and torch.equal(a, c)
    tr.close()


def test_readout_error_paths(phx):
    """Bad layouts and parameters are refused before any launch."""
    import torch
    img = torch.zeros((64, 64), dtype=torch.int32, device="cuda")
    tr = phx.Tracer(C.tiny(scale=1e-4))
    for bad in (dict(amp_nx=3), dict(amp_ny=3), dict(cte_parallel=0.0), dict(gain=(0.0,) * 32),
                dict(hot_fraction=0.7, dead_fraction=0.7), dict(full_well=0.0),
                dict(full_well=2e7), dict(dark_rate=1e5, exposure=15.0)):
        with pytest.raises(phx.PhxError):
            tr.readout(img, Readout(amp_nx=2, amp_ny=2).replace(**bad))
    tr.close()


@pytest.mark.parametrize("shape,over", [
    ((3, 130), dict(amp_nx=1, amp_ny=1)),                                      # less than a workgroup
    ((66, 514), dict(amp_nx=2, amp_ny=2, over_x=1, over_y=65)),
    ((4, 8200), dict(amp_nx=4, amp_ny=2)),                                     # half-rows beyond LDS
    ((128, 128), dict(cte_parallel=0.5, cte_serial=0.6)),                      # no word is kept
    ((64, 256), dict(cte_parallel=1.0, cte_serial=1.0)),
    ((64, 256), dict(nonlinearity=3.0, read_noise=(4000.0,) * 32)),            # bounds do not hold
    ((64, 256), dict(bit_sigma=(0.3,) * 16, read_noise=(0.0,) * 32)),
    ((64, 256), dict(bit_sigma=(0.0,) * 15 + (0.01,), bias=(-50.0,) * 32)),    # clamped values
    ((2, 64), dict(dark_rate=1e3, full_well=1e7, hot_fraction=0.0, hot_column_fraction=0.0)),
])
def test_readout_at_the_edges_of_its_kernels(phx, shape, over):
    """Packets at the limits of the light and heavy transfers (64 electrons) and of a wavefront's draw
    blocks (256), ragged sizes, transfer probabilities that leave no word or every word, and values for
    which the deviates in 32 bits decide nothing: the electrons of every stage and the converted
    values are the oracle's."""
    rp = Readout(**{**dict(amp_nx=4, amp_ny=2, over_x=3, over_y=2, hot_fraction=1e-3,
                           dead_fraction=1e-3, hot_column_fraction=1e-3, cte_parallel=1 - 1e-4,
                           cte_serial=1 - 5e-5), **over})
    img = _image(*shape)
    edge = np.array([0, 1, 3, 4, 5, 63, 64, 65, 255, 256, 257, 1023, 1024, 1025, 100000, 100001],
                    np.uint32)
    img[:2, 8:24] = edge
    g, o = run_both(phx, img, rp)
    assert check(g, o) <= 2


def test_digitised_values_of_large_cancelling_terms(phx):
    """Gains so small and biases so large that the two forms of the quotient, e / (g (1 + a e / W)) and
    e / (g (1 + (a / W) e)), differ by more than any fixed margin: per amplifier the bias puts the
    first form's value on a whole number that the second form's misses from below."""
    n_amp, W, a = 16, 1e5, 0.01
    rng = np.random.default_rng(0)
    img = np.zeros((64, 128), np.uint32)
    gain, bias, want = [], [], []
    while len(gain) < n_amp:
        ne, g = float(rng.integers(1000, 90000)), 10.0 ** rng.uniform(-9, -5)
        q1, q2 = ne / (g * (1.0 + a * ne / W)), ne / (g * (1.0 + (a / W) * ne))
        k = float(rng.integers(100, 60000))
        b = k - q1
        if q2 + b < k == q1 + b:
            amp = len(gain)
            img[32 * (amp // 8):, 16 * (amp % 8):16 * (amp % 8) + 16] = int(ne)
            gain.append(g)
            bias.append(b)
            want.append(int(k))
    rp = Readout(amp_nx=8, amp_ny=2, over_x=0, over_y=0, hot_fraction=0.0, dead_fraction=0.0,
                 hot_column_fraction=0.0, cte_parallel=1.0, cte_serial=1.0, dark_rate=0.0,
                 full_well=W, nonlinearity=a, gain=tuple(gain + [1.0] * 16),
                 bias=tuple(bias + [0.0] * 16), read_noise=(0.0,) * 32, bit_sigma=(0.0,) * 16)
    g, o = run_both(phx, img, rp)
    assert np.array_equal(o[0], np.array(want, np.uint16)[:, None, None] + np.zeros_like(o[0]))
    assert np.array_equal(g[0].view(np.uint16), o[0])


@pytest.mark.parametrize("shape", [(1024, 1024), (1024, 1028), (2056, 4096)])
def test_readout_where_the_packets_per_workgroup_change(phx, shape):
    """256 packets per workgroup, 512, and a part of a second batch of loads (2304): sparse spots at the
    limits of the transfers on an empty image, stage by stage against the oracle."""
    rng = np.random.default_rng(4)
    img = np.zeros(shape, np.uint32)
    n = 3000
    img[rng.integers(0, shape[0], n), rng.integers(0, shape[1], n)] = rng.choice(
        [1, 4, 63, 64, 65, 257, 3000], n)
    rp = Readout(amp_nx=4, amp_ny=2, dark_rate=0.0, hot_column_fraction=0.0, cte_parallel=1 - 1e-5,
                 cte_serial=1 - 1e-5)
    g, o = run_both(phx, img, rp)
    assert check(g, o) <= 2


def _time(phx, images):
    """Median seconds of a readout of each image, taken in turn."""
    import time
    import torch
    tr = phx.Tracer(C.tiny(scale=1e-4))
    dev = [torch.from_numpy(i.astype(np.int32)).cuda() for i in images]
    rp = Readout(amp_nx=4, amp_ny=2)
    t = [[] for _ in dev]
    for k in range(25):
        for j, d in enumerate(dev):
            torch.cuda.synchronize()
            a = time.perf_counter()
            tr.readout(d, rp)
            torch.cuda.synchronize()
            t[j].append(time.perf_counter() - a)
    tr.close()
    return [float(np.median(v[5:])) for v in t]


def test_a_small_image_is_spread_over_the_compute_units(phx):
    """64 x 64 pixels: their electrons cost little beside the launches (1.9 times an empty image's time
    when one workgroup held them all, 1.1 now)."""
    empty, full = _time(phx, [np.zeros((64, 64)), np.full((64, 64), 60)])
    assert full < 1.5 * empty


def test_a_background_is_not_handed_out_packet_by_packet(phx):
    """Pixels that all hold 300 electrons: 2.4 times the time of 10 (11.5 when every packet above 64 was
    handed to whole wavefronts)."""
    rng = np.random.default_rng(6)
    dark, bright = _time(phx, [rng.poisson(10.0, (1024, 1024)), rng.poisson(300.0, (1024, 1024))])
    assert bright < 5.0 * dark


@pytest.mark.parametrize("shape,layout", [((128, 256), (4, 2)), ((3, 130), (1, 1))])
def test_readout_at_the_limits_a_wavefront_chooses(phx, shape, layout):
    """Wavefronts with 0 to 64 packets at and beside each limit between the two transfer kernels (64 to
    2048 electrons by doubling), alone and among others above it: every stage against the oracle."""
    rng = np.random.default_rng(8)
    edges = np.array([63, 64, 65, 127, 128, 129, 256, 257, 512, 513, 1024, 1025, 2047, 2048, 2049,
                      5000])
    img = rng.poisson(20.0, shape).astype(np.uint32)
    flat = img.reshape(-1)
    for w in range(flat.size // 64):
        k = int(rng.integers(0, 65))
        at = 64 * w + rng.permutation(64)[:k]
        flat[at] = rng.choice(edges[:int(rng.integers(1, edges.size + 1))], k)
    rp = Readout(amp_nx=layout[0], amp_ny=layout[1], dark_rate=0.0, cte_parallel=1 - 1e-4,
                 cte_serial=1 - 5e-5)
    g, o = run_both(phx, img, rp)
    assert check(g, o) <= 2
