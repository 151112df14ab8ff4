"""Shapes of the team relaxation kernels, on the host: every shape that the
dispatch takes fits a workgroup's LDS, and the wavefront counts that it takes
leave no hole.  The dispatch's source is compiled on its own."""
import ctypes
import os
import subprocess

import pytest

from paper_1403_0555_amd import build

LDS = 160 * 1024
PROBE = """
#include "gc_team.hip"
extern "C" void probe(int d, int K, int V, long *out)
{
    const GcTeamShape s = gc_team_shape(d, K, V);
    out[0] = s.cls;
    out[1] = s.waves;
    out[2] = s.cls ? (long)gc_team_lds_bytes(d, K, s, V, false) : 0;
    out[3] = s.cls ? gc_team_class(d, K, s.cls).spt : 0;
    out[4] = s.cls ? gc_team_class(d, K, s.cls).maxw : 0;
}
"""


@pytest.fixture(scope="module")
def shape(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("team")
    src, out = str(tmp / "probe.cpp"), str(tmp / "probe.so")
    with open(src, "w") as f:
        f.write(PROBE)
    subprocess.run([build.HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-shared", "-fPIC", "-I", build.CSRC, src, "-o", out], check=True)
    # the kernels' entry points stay unresolved: bound when called, and never called
    fn = ctypes.CDLL(out, mode=os.RTLD_LAZY).probe

    def at(d, K, V):
        v = (ctypes.c_long * 5)()
        fn(d, K, V, v)
        return tuple(v)
    return at


@pytest.mark.parametrize("d", [1, 2, 3, 4])
@pytest.mark.parametrize("K", [2, 3, 5, 7])
def test_team_shapes_fit_and_leave_no_hole(shape, d, K):
    taken = []
    for sites in range(1, 4096 // K + 1):
        cls, waves, lds, spt, maxw = shape(d, K, K * sites)
        if cls:
            assert 64 * waves * spt >= sites and waves <= maxw
            assert lds <= LDS - 1024, (d, K, sites, lds)   # 1 KiB for what the kernel holds beside
            taken.append(sites)
    assert taken == list(range(taken[0], taken[-1] + 1)) if taken else d == 1 or (d, K) == (4, 7)
    if K == 2:
        assert (taken[0], taken[-1]) == (65, 1024)
