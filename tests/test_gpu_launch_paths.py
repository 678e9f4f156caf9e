"""Kernels and launch rules at the sizes where they can go wrong."""
import numpy as np
import pytest

from tests import moments_ref as R

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def phx():
    from paper_1504_06570_amd import phx
    return phx


EDGE = (1 << 127) - 1


@pytest.mark.parametrize("n_src", [1, 8, 9, 441])
def test_moments_at_the_edges_of_their_words(phx, n_src):
    """Counts of one and of 64 bits, sums of zero, of one bit, of full range and either sign, exact
    halves, against rational arithmetic (equal: each result is one rounding of an exact ratio)."""
    import torch
    from paper_1504_06570_amd.scene import configs as C
    rng = np.random.default_rng(n_src)
    edge = [(1, 1, -1, 1, 0, -1), ((1 << 64) - 1, EDGE, -EDGE - 1, -EDGE - 1, EDGE, 1),
            (0, 5, 5, 5, 5, 5), (2, (1 << 54) + 1, -((1 << 54) + 1), 1, 1, 1),
            (3, EDGE, EDGE, EDGE, 1 << 126, -(1 << 126))]
    sums = edge[:n_src]
    while len(sums) < n_src:
        n = int(rng.integers(1, 10 ** 7))
        x, y = (int(v) for v in rng.normal(0.0, 3e-2, 2) * 2.0 ** 44)
        d = [int(v) for v in rng.integers(-n, n, 2)]
        sums.append((n, n * x + d[0], n * y + d[1], n * (x * x + 10 ** 17), n * (y * y + 10 ** 17),
                     n * (x * y + 10 ** 15)))
    tr = phx.Tracer(C.tiny(scale=0.01))
    w = torch.from_numpy(R.words_of(sums)).cuda()
    got = tr.moments(w).cpu().numpy()
    np.testing.assert_array_equal(got, R.moments_from_sums(sums))


def test_launches_of_one_context_on_two_streams_wait_for_each_other(phx):
    """One-chunk launches stay on the caller's stream; two streams used in turn must not meet in the
    context's workspace: the images add up to those of one stream."""
    import torch
    from paper_1504_06570_amd.scene import configs as C
    scene = C.full(scale=2e-4, screen_n=128)
    tr = phx.Tracer(scene)
    flags = int(scene.physics) | phx.F_CULL
    want = tr.trace(flags=flags)[0]
    for k in range(5):
        tr.trace(want, flags=flags, seed=100 + k)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    images = [tr.new_image(), tr.new_image()]
    torch.cuda.synchronize()
    tr.trace(images[0], flags=flags, stream=streams[0])
    for k in range(5):
        tr.trace(images[(k + 1) % 2], flags=flags, seed=100 + k, stream=streams[(k + 1) % 2])
    torch.cuda.synchronize()
    assert torch.equal(images[0] + images[1], want)
    tr.close()


@pytest.mark.parametrize("photons", [1, 255, 256, 257, 4097, (1 << 19) - 1, (1 << 19) + 1,
                                     (1 << 20) + 63, (1 << 21) + 1, (1 << 22) + 5])
@pytest.mark.parametrize("cull", [True, False])
def test_lists_hold_every_photon_at_the_edges_of_ranges_and_of_the_sort(phx, photons, cull):
    """The lists of photons to trace (unsorted and sorted, with the pre-roll and without, ranges of 256,
    1024 and 4096) against phx_trace_noalloc, which never sorts and cuts chunks of 2^19: the same image,
    and every photon in one place of the statistics."""
    import torch
    from paper_1504_06570_amd.scene import configs as C
    scene = C.full(scale=1e-6, screen_n=64)
    tr = phx.Tracer(scene)
    flags = int(scene.physics) | (phx.F_CULL if cull else 0)
    got, st, _, _ = tr.trace(flags=flags, stats=tr.new_stats(), photon_count=photons)
    want, st2, _, _ = tr.trace(flags=flags, stats=tr.new_stats(), photon_count=photons, noalloc=True)
    torch.cuda.synchronize()
    assert torch.equal(got, want) and torch.equal(st, st2)
    assert int(phx.stats_table(st).sum()) == photons
    tr.close()


def test_lists_of_many_sources_without_an_atmosphere(phx):
    """A chunk of several sources above the sort's limit, classed only: the same image and moment words as
    one launch per source (below the limit, unsorted)."""
    import torch
    from paper_1504_06570_amd.scene import configs as C
    scene = C.telescope(scale=0.2)      # 441 sources, 2e6 photons
    tr = phx.Tracer(scene)
    m = tr.new_moments()
    img = tr.trace(moments=m)[0]
    ref, mr = tr.new_image(), tr.new_moments()
    for s in range(0, 441, 63):
        tr.trace(ref, moments=mr, src_begin=s, src_end=s + 63)
    torch.cuda.synchronize()
    assert torch.equal(img, ref) and torch.equal(m, mr)
    tr.close()


def _ghosts(phx):
    from paper_1504_06570_amd.scene import coatings as cm
    from paper_1504_06570_amd.scene import configs as C
    scene = C.full(scale=1e-6, screen_n=64)
    scene.reflectance = cm.standard_reflectance()
    return phx.Tracer(scene), int(scene.physics) | phx.F_GHOSTS


@pytest.mark.parametrize("photons,shape", [
    (1, {}), (65, {}), (1000003, dict(back_blocks_per_cu=1)),   # blocks of the list reserved, or not
    (20000003, dict(chunk_log2=18)),                            # branches claimed, or dealt out
    (20000003, dict(chunk_log2=20, dynamic_tiles=1)),
])
def test_ghost_lists_of_every_size_hold_the_same_starts(phx, photons, shape):
    """The ghost list reserved by blocks and entry by entry, its branches from a counter and in turn:
    the same image, and every photon in one place of the statistics."""
    import torch
    tr, flags = _ghosts(phx)
    want, st, _, _ = tr.trace(flags=flags, stats=tr.new_stats(), photon_count=photons)
    tr.set_launch_config(**shape)
    got, st2, _, _ = tr.trace(flags=flags, stats=tr.new_stats(), photon_count=photons)
    torch.cuda.synchronize()
    assert torch.equal(got, want) and torch.equal(st, st2)
    assert int(phx.stats_table(st).sum()) == photons
    tr.close()


def test_a_short_ghost_list_takes_few_wavefronts(phx):
    """1e4 photons: the branch pass is launched for the entries there can be, however wide the launch
    shape is (a counter's atomic for each wavefront of the widest took 20 times the rest)."""
    import time
    import torch
    tr, flags = _ghosts(phx)
    img, t = tr.new_image(), {}
    for width in (2, 64):
        tr.set_launch_config(back_blocks_per_cu=width)
        v = []
        for _ in range(15):
            torch.cuda.synchronize()
            a = time.perf_counter()
            tr.trace(img, flags=flags, photon_count=10000)
            torch.cuda.synchronize()
            v.append(time.perf_counter() - a)
        t[width] = float(np.median(v[5:]))
    tr.close()
    assert t[64] < 3.0 * t[2], t


def test_the_dynamic_schedule_launches_the_workgroups_asked_for(phx):
    """Its wavefronts claim their work from one counter, each at least once: the widest shape takes 1.5
    times as long as the default one (2.6 times when it launched four times as many workgroups)."""
    import time
    import torch
    from paper_1504_06570_amd.scene import configs as C
    scene = C.full(scale=1e-6, screen_n=64)
    tr = phx.Tracer(scene)
    flags, img, t = int(scene.physics) | phx.F_CULL, tr.new_image(), {}
    tr.set_launch_config(dynamic_tiles=1, pipeline=0)
    for width in ((48, 2), (64, 64)):
        tr.set_launch_config(front_blocks_per_cu=width[0], back_blocks_per_cu=width[1])
        v = []
        for _ in range(9):
            torch.cuda.synchronize()
            a = time.perf_counter()
            tr.trace(img, flags=flags, photon_count=30000000)
            torch.cuda.synchronize()
            v.append(time.perf_counter() - a)
        t[width] = float(np.median(v[3:]))
    tr.close()
    assert t[64, 64] < 2.1 * t[48, 2], t
