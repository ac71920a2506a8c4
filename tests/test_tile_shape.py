"""The tile kernel's weight addresses, checked on the CPU with the header that the kernel itself uses: no load leaves the
weights, and a real channel's fragment is where it is stored."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2012_13846_amd", "csrc")
HARNESS = r"""
#include "sp_tile_shape.h"
using namespace sp;
// 0: every load of this layer is inside the weights and right; 1: outside; 2: a real channel's fragment is elsewhere
extern "C" int check(int cc, int co, int kvol, int f32, int big, int in_place) {
    const int elt = f32 ? 4 : 2;
    const TileShape t = tile_shape(cc, co, f32 != 0, big != 0);
    if (in_place ? !tile_in_place_ok(t, cc) || (uint64_t)kvol * cc * co * elt >> 32 : tile_copy_bytes(t, kvol, elt) >> 32) return 0;
    const TileWeights w = in_place ? tile_weights_in_place(t, kvol, cc, co, elt) : tile_weights_copied(t, kvol, elt);
    const int groups = t.kc * elt / 64;
    for (int y = 0; y < t.ny; ++y)
        for (int cs = 0; cs < t.ncs; ++cs)
            for (int lane = 0; lane < 64; ++lane) {
                uint32_t u, l;
                tile_weight_at(w, t.ncs, y, cs, lane & 15, lane >> 4, &u, &l);
                const int c = (y * t.ncs + cs) * 16 + (lane & 15);
                const int ks[2] = {0, kvol - 1}, sls[2] = {0, t.nsl - 1}, ss[2] = {0, groups - 1};
                for (int i = 0; i < 8; ++i) {
                    const int k = ks[i & 1], sl = sls[i >> 1 & 1], s = ss[i >> 2];
                    const uint64_t at = (uint64_t)k * w.k + (uint64_t)sl * w.slice + (uint64_t)s * w.s + u + l;
                    if (at + 16 > w.bytes) return 1;
                    const uint64_t cc0 = (uint64_t)(sl * groups + s) * (64 / elt) + (lane >> 4) * (16 / elt);
                    const uint64_t want = in_place ? (((uint64_t)k * co + c) * cc + cc0) * elt
                        : (((((uint64_t)k * t.ny + y) * t.ncs + cs) * t.nsl + sl) * groups + s) * 1024 + lane * 16;
                    if (c < co && at != want) return 2;
                }
            }
    return 0;
}
"""


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    d = tmp_path_factory.mktemp("tile_shape")
    (d / "harness.cpp").write_text(HARNESS)
    so = str(d / "harness.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(d / "harness.cpp"), "-o", so])
    return ctypes.CDLL(so).check


@pytest.mark.parametrize("f32", [0, 1])
@pytest.mark.parametrize("in_place", [0, 1])
def test_weight_loads_stay_inside_the_weights(check, f32, in_place):
    ccs = [1, 3, 15, 16, 17, 31, 32, 33, 48, 64, 65, 80, 96, 112, 128, 144, 192, 256, 300, 320, 512, 1024, 4096]
    cos = list(range(1, 130)) + [144, 200, 208, 255, 256, 257, 300, 400, 512, 1000, 4095, 4096]
    bad = [(cc, co, kvol, big, r) for cc in ccs for co in cos for kvol in (1, 27, 125) for big in (0, 1)
           if (r := check(cc, co, kvol, f32, big, in_place))]
    assert not bad, bad[:5]
