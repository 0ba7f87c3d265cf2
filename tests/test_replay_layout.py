"""The replay's workspace layout, compiled for the host as it stands (cr_replay_layout.h): every
region holds what the kernels index it with, and no two overlap, over request counts from none to
the largest, few and many candidates and destinations, and slot budgets alone and in groups."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2608_19677_amd", "csrc")

HARNESS = r"""
#include "cr_replay_layout.h"
using namespace cr;

// Work items of a call whose requests go to the destinations evenly, or all but a few to one.
static uint64_t items(uint64_t n, uint32_t P, uint32_t R, uint32_t W, uint32_t G, int skew)
{
    WArg wa;
    seg_rule(n, P, &wa);
    const uint64_t S = seg_len(W, wa, G);
    uint64_t it = 0;
    for (uint32_t d = 0; d < R; ++d) {
        uint64_t cnt = skew ? (d ? (n > R ? 1 : 0) : n - (n > R ? R - 1 : 0)) : n / R + (d < n % R ? 1 : 0);
        it += cnt ? (cnt + S - 1) / S : 1;
    }
    return it * P;
}

// 0, or which region fails: 1 .. 6 a region runs into the next, 7 the marks past the workspace.
extern "C" int check(uint64_t n, uint32_t P, uint32_t R, uint32_t W, uint32_t J, int grouped, int skew)
{
    const ReplayWs w = replay_layout(nullptr, n, P, R);
    const PartGeom g = part_geom(n, P);
    auto at = [](const void* p) { return (uint64_t)(uintptr_t)p; };
    if (at(w.rec) + 8 * n * P > at(w.tcnt)) return 1;
    if (at(w.tcnt) + 4ull * P * R * g.ntiles > at(w.dtot)) return 2;
    if (at(w.dtot) + 4ull * P * R > at(w.grp_off)) return 3;
    if (at(w.grp_off) + 4ull * P * (R + 1) > at(w.item_off)) return 4;
    if (at(w.item_off) + 4ull * (P * R + 1) > at(w.gwave_off)) return 5;
    const uint64_t m0 = at(w.aborted), m1 = m0 + items(n, P, R, W, grouped ? grp_of(W, J) : 1u, skew);
    const uint64_t gw0 = at(w.gwave_off), gw1 = gw0 + 4ull * (P + 1);
    // the marks, written by the replay: clear of what the replay reads
    if (m0 < at(w.tcnt) || (m0 < gw1 && m1 > at(w.grp_off))) return 6;
    return m1 + 255 > w.bytes ? 7 : 0;  // the base is rounded up to 256 bytes
}
extern "C" uint64_t bytes(uint64_t n, uint32_t P, uint32_t R) { return replay_layout(nullptr, n, P, R).bytes; }
"""


@pytest.fixture(scope="module")
def layout(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("layout")
    src, lib = d / "layout.cpp", d / "layout.so"
    src.write_text(HARNESS)
    subprocess.run([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-I" + CSRC, str(src), "-o", str(lib)], check=True)
    so = ctypes.CDLL(str(lib))
    so.check.argtypes = [ctypes.c_uint64, ctypes.c_uint32, ctypes.c_uint32, ctypes.c_uint32, ctypes.c_uint32, ctypes.c_int, ctypes.c_int]
    so.bytes.restype = ctypes.c_uint64
    so.bytes.argtypes = [ctypes.c_uint64, ctypes.c_uint32, ctypes.c_uint32]
    return so


N = [0, 1, 2, 255, 256, 257, 1023, 1025, 4096, 30_011, 100_000, 999_999, 1_250_000, 1_600_000, 2_000_000, 2_250_000, 4_194_303,
     4_194_304, 10_000_000, 17_000_000, 20_000_000, 25_000_000, 70_000_000, 100_000_000, 10**9, 4 * 10**9, 2**32 - 2]


def test_marks_fit_and_regions_are_disjoint(layout):
    bad = []
    for n in N:
        for P in (1, 2, 3, 8, 9, 32, 63, 64, 65, 200, 255, 256):
            for R in (1, 2, 3, 4, 7, 8, 11, 16, 64, 65, 1024):
                for W, J, grouped in ((1, 1, 1), (8, 1, 1), (9, 1, 1), (16, 1, 1), (1, 1, 0), (8, 24, 0), (64, 24, 0), (512, 1, 0)):
                    for skew in (0, 1):
                        r = layout.check(n, P, R, W, J, grouped, skew)
                        if r:
                            bad.append((n, P, R, W, J, grouped, skew, r))
    assert not bad, (len(bad), bad[:10])


def test_layout_is_the_one_the_library_was_built_with(layout):
    from paper_2608_19677_amd import binding as B
    for n, P, R in ((0, 1, 1), (30_011, 2, 65), (20_000_000, 8, 2), (100_000_000, 64, 1024), (2**32 - 2, 1, 1)):
        assert layout.bytes(n, P, R) == B.cr_replay_workspace_bytes(n, P, R)
