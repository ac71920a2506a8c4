"""How the fp32 layers on the bf16 matrix cores are cut (csrc/sp_split_shape.h), checked on the CPU with the header that the library
itself uses: every cut has a kernel, its LDS is there, and the heights and steps change where the measured launches say."""
import ctypes
import functools
import os
import re
import subprocess
import tempfile

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2012_13846_amd", "csrc")
HARNESS = r"""
#include "sp_split_shape.h"
using namespace sp;
extern "C" void cut(int cc, int co, int64_t n_rows, int kvol, int64_t links, int* out) {
    const SplitShape t = split_shape(cc, co);
    const SplitTile x = split_tile(t, n_rows, kvol, links);
    const int v[] = {x.halves, x.g, t.cc, t.nsl, t.cot, t.ny, split_lds(t.cc, t.cot / 16, x.g, x.halves, kvol)};
    for (int i = 0; i < 7; ++i) out[i] = v[i];
}
extern "C" int waves_of_a_simd(int cc, int nw, int g) { return split_simd_waves(cc, nw, g); }
"""
KERNELS = {(64, 128, 2), (64, 128, 3), (64, 64, 2), (64, 64, 3), (64, 48, 3), (64, 32, 2), (32, 128, 2), (32, 64, 2), (32, 48, 3), (32, 32, 2)}


@functools.lru_cache(maxsize=None)
def _lib():
    with tempfile.TemporaryDirectory() as d:
        src, so = os.path.join(d, "harness.cpp"), os.path.join(d, "harness.so")
        with open(src, "w") as f:
            f.write(HARNESS)
        subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, src, "-o", so])
        lib = ctypes.CDLL(so)
    lib.cut.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_int64, ctypes.c_int, ctypes.c_int64, ctypes.POINTER(ctypes.c_int)]
    return lib


def cut(cc, co, n_rows, kvol, links):
    """(halves of 32 rows, blocks of 16 links a step, slice, slices, channel tile, channel tiles, LDS bytes)"""
    out = (ctypes.c_int * 7)()
    _lib().cut(cc, co, n_rows, kvol, links, out)
    return tuple(out)


def waves_of_a_simd(cc, nw, g):
    return _lib().waves_of_a_simd(cc, nw, g)


def test_every_cut_has_a_kernel_and_fits():
    most = 0
    for cc in (20, 24, 32, 40, 48, 64, 80, 96, 100, 128, 192, 256, 512):
        for co in (20, 24, 32, 40, 48, 64, 72, 80, 96, 100, 128, 192, 256, 384):
            for kvol in (1, 8, 27, 64, 125):
                for n in (1, 31, 1000, 4097, 16384, 16385, 50000, 131073, 613402, 5000000):
                    for per in (0.2, 1.0, 5.0, 12.0, 33.0, 63.9, 64.0, 128.0):
                        h, g, c, nsl, cot, ny, lds = cut(cc, co, n, kvol, int(n * kvol * per / 128))
                        assert 2 <= h <= 7 and (c, cot, g) in KERNELS
                        assert c * nsl >= cc and cot * ny >= co
                        assert lds <= 163840 - 256        # static LDS beside it: a few words
                        most = max(most, lds)
    assert most == 161048 == cut(64, 128, 98337, 125, 8250000)[6]


@pytest.mark.parametrize("cc,co,n,kvol,per,want", [
    (64, 64, 613402, 27, 38.6, (3, 2)), (64, 64, 96000, 27, 15.7, (6, 2)), (128, 64, 144584, 27, 37.9, (3, 2)), (64, 64, 50598, 27, 49.4, (4, 3)),
    (64, 192, 48725, 27, 49.8, (3, 2)), (80, 48, 75486, 27, 38.8, (3, 3)), (24, 40, 75486, 27, 38.8, (3, 3)), (128, 32, 180627, 27, 29.5, (3, 2)),
    (64, 128, 96000, 27, 89.3, (6, 3)), (128, 128, 96000, 27, 15.7, (6, 2)), (128, 128, 95723, 27, 30.3, (6, 2)), (32, 64, 95723, 27, 30.3, (3, 2)),
    (64, 64, 85693, 27, 26.5, (3, 2)), (64, 128, 1000, 27, 40.0, (2, 2)), (64, 64, 16000, 27, 20.0, (2, 2))])
def test_measured_choices(cc, co, n, kvol, per, want):
    """Launches whose times stand at split_tile, or that a rule which counts an offset's weights once a tile made 5 to 36 % slower."""
    assert cut(cc, co, n, kvol, round(n * kvol * per / 128))[:2] == want



def test_registers_leave_the_workgroups_that_the_rule_counts_on():
    """The built kernels' vector registers (512 a SIMD lane, handed out in eights) and spills, from the metadata of their object file."""
    obj = os.path.join(os.path.dirname(CSRC), "_build", "sp_conv_split.o")
    llvm = "/opt/rocm/llvm/bin/"
    if not os.path.exists(obj) or not os.path.exists(llvm + "llvm-readelf"):
        pytest.skip("needs the object file of the build and ROCm's binary tools")
    with tempfile.TemporaryDirectory() as d:
        fat, code = os.path.join(d, "fat"), os.path.join(d, "code")
        subprocess.check_call([llvm + "llvm-objcopy", "--dump-section", ".hip_fatbin=" + fat, obj, os.path.join(d, "copy")])
        subprocess.check_call([llvm + "clang-offload-bundler", "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950",
                               "--input=" + fat, "--output=" + code])
        notes = subprocess.check_output([llvm + "llvm-readelf", "--notes", code], text=True)
    seen = set()
    for kernel in notes.split(".agpr_count:")[1:]:
        m = re.search(r"gather_split_kernelILi(\d+)ELi(\d+)ELi(\d+)E", kernel)
        if not m:
            continue
        cc, nw, g = map(int, m.groups())
        seen.add((cc, 16 * nw, g))
        regs = int(kernel.split()[0]) + int(re.search(r"\.vgpr_count: +(\d+)", kernel).group(1))
        waves = waves_of_a_simd(cc, nw, g)
        assert (regs + 7) // 8 * 8 * waves <= 512, (cc, nw, g, regs, waves)
        assert re.search(r"\.vgpr_spill_count: +0\b", kernel)
    assert seen == KERNELS
