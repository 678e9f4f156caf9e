"""The rules that choose launch sizes (phx_internal.h) at the edges of their ranges, on the CPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r"""
#include <cstdio>
#include "%s/paper_1504_06570_amd/csrc/phx_internal.h"
using namespace phx;
int main() {
    LaunchConfig d, dyn;
    dyn.dynamic = 1;
    printf("%%d %%d %%d\n", stage_groups(d, 2), stage_groups(dyn, 2), stage_groups(dyn, 64));
    for (unsigned long long tiles : {1, 511, 512, 1023, 1024, 1025, 2048, 4095, 4096, 8192, 1 << 18}) {
        const unsigned long long len = 256 * (tiles - 1) + 1;
        printf("%%llu %%llu %%llu\n", tiles, (unsigned long long)optics_groups(d, 256, len),
               (unsigned long long)optics_groups(dyn, 256, len));
    }
    // room for a start per photon and the unused end of every wavefront's block, at any width
    int bad = 0;
    for (int per_cu = 1; per_cu <= 64; ++per_cu)
        for (int lg = 10; lg <= 27; ++lg)
            for (int dynamic = 0; dynamic < 2; ++dynamic) {
                LaunchConfig c;
                c.back_per_cu = per_cu;
                c.dynamic = dynamic;
                const unsigned long long len = 1ull << lg;
                const unsigned long long waves = optics_groups(c, 256, len) * (kThreads / 64);
                bad += ghost_entries(len, 256, per_cu) < len + kGhostReserve * waves;
            }
    printf("%%d\n", bad);
}
"""


@pytest.fixture(scope="module")
def lines(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "r.cpp").write_text(SRC % ROOT)
    exe = str(d / "r")
    subprocess.check_call(["g++", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-o", exe, str(d / "r.cpp")])
    return [[int(x) for x in line.split()]
            for line in subprocess.check_output([exe], text=True).splitlines()]


def test_the_dynamic_schedule_takes_its_width_as_it_is(lines):
    assert lines[0] == [8, 2, 64]


def test_optics_workgroups(lines):
    """256 compute units, two in fours: 2048 workgroups from two tiles each on, half of them below, never more
    than tiles; 512 with the dynamic schedule."""
    for tiles, static, dynamic in lines[1:-1]:
        assert static == min(tiles, 2048 if tiles >= 4096 else 1024)
        assert dynamic == min(tiles, 512)


def test_the_ghost_list_has_room_for_every_wavefront(lines):
    assert lines[-1] == [0]
