"""Tiles of every height of the fp32 layers on the bf16 matrix cores (csrc/sp_conv_split.hip): 64 to 224 rows by channel tile, rows and
links, steps of 32 and 48 links, with last tiles of one row and of a few sub-tiles, one and several channel tiles.  Against
fp64: as far off as fp32 sums of up to 27 * 192 products may be (1.4e-7 of the rms measured, 3e-7 allowed), for 125 offsets as much
more as the square root of the links that are added."""
import pytest
import torch

from test_gpu_parity import sp  # noqa: F401  (the binding fixture)
from test_gpu_split import cloud, fwd64
from test_split_shape import cut

pytestmark = pytest.mark.gpu


def near(got, want, kvol=27):
    err, rms = got.double() - want, want.square().mean().sqrt()
    return float(err.square().mean().sqrt() / rms) <= 3e-7 * max(1.0, kvol / 27.0) ** 0.5 and float(err.abs().max() / rms) <= 1e-5


# (voxels, bits, halves of 32 rows, blocks of 16 links a step)
HEIGHTS = {
    (64, 128): [(12033, 5, 2, 2), (16417, 5, 3, 2), (114721, 5, 3, 3), (24577, 5, 4, 2), (32801, 5, 5, 2), (69761, 5, 5, 3), (41089, 5, 6, 2),
                (81985, 5, 6, 3), (49281, 5, 7, 2), (98337, 5, 7, 3)],
    (64, 192): [(16321, 5, 2, 2), (12001, 5, 3, 2), (16385, 5, 4, 2), (40961, 5, 4, 3), (24641, 5, 5, 2), (13633, 6, 6, 2)],
    (20, 128): [(1473, 4, 2, 2), (16417, 5, 3, 2), (24577, 6, 4, 2), (32801, 6, 5, 2), (41089, 6, 6, 2), (49281, 5, 7, 2)],
    (64, 64): [(34049, 5, 2, 2), (65569, 5, 3, 2), (49153, 6, 4, 2), (49153, 5, 4, 3), (34081, 6, 5, 2), (41089, 6, 6, 2), (49281, 7, 7, 2)],
    (32, 64): [(34049, 5, 2, 2), (65569, 5, 3, 2), (49153, 6, 4, 2)],
    (128, 32): [(49153, 5, 2, 2), (65569, 5, 3, 2), (49153, 6, 4, 2), (98401, 6, 5, 2)],
    (48, 48): [(98305, 5, 3, 3), (49153, 5, 4, 3), (65601, 5, 5, 3), (81985, 5, 6, 3)],
    (24, 40): [(65569, 5, 3, 3), (98401, 5, 5, 3)],
    (96, 96): [(65569, 5, 3, 3), (169441, 6, 5, 3)]}


@pytest.mark.parametrize("cin,cout,n,bits,halves,g", [k + v for k, vs in HEIGHTS.items() for v in vs])
def test_heights(sp, cin, cout, n, bits, halves, g):  # noqa: F811
    c, km, gen = cloud(sp, n, bits, n + cin)
    assert sp.sp_conv_kernel_name(km, cin, cout, torch.float32) == "gather_split_kernel"
    assert cut(cin, cout, n, 27, km.total)[:2] == (halves, g)
    x, w = torch.randn((n, cin), device="cuda", generator=gen), torch.randn((27, cout, cin), device="cuda", generator=gen)
    assert near(sp.sp_conv_fwd(km, x, w), fwd64(km, x, w))
    assert near(sp.sp_conv_bwd_data(km, x, w.transpose(1, 2).contiguous()), fwd64(km, x, w.flip(0)))


@pytest.mark.parametrize("n,bits,K,stride,cin,cout,direction", [(50000, 5, 5, 1, 64, 128, 0), (98337, 5, 5, 1, 64, 128, 0), (100000, 6, 5, 1, 64, 128, 0), (96000, 6, 2, 1, 64, 128, 0),
    (90000, 6, 4, 1, 128, 128, 0), (90000, 6, 4, 2, 64, 64, 1), (100000, 6, 3, 2, 128, 128, 0), (100000, 6, 3, 2, 64, 64, 1), (160000, 7, 2, 2, 128, 128, 1)])
def test_tall_tiles_of_other_maps(sp, n, bits, K, stride, cin, cout, direction):  # noqa: F811
    """160 rows and more with 8, 64 and 125 offsets (the second case: 161 048 bytes of LDS, the most there are) and on both sides of strided maps; a row with an infinity makes the tiles it reaches
    compute theirs again."""
    c, _, gen = cloud(sp, n, bits, n + K)
    km, _ = sp.sp_kmap_build(c, K, stride, 1)
    src, dst = (km.n_in, km.n_out) if direction == 0 else (km.n_out, km.n_in)
    assert sp.sp_conv_kernel_name(km, *((cin, cout) if direction == 0 else (cout, cin)), torch.float32, direction) == "gather_split_kernel"
    assert cut(cin, cout, dst, K ** 3, km.total)[0] >= 5
    x, w = torch.randn((src, cin), device="cuda", generator=gen), torch.randn((K ** 3, cout, cin), device="cuda", generator=gen)
    pin, pout = km.pairs_strided()
    a, b = (pin, pout) if direction == 0 else (pout, pin)

    def run(x):
        return sp.sp_conv_fwd(km, x, w) if direction == 0 else sp.sp_conv_bwd_data(km, x, w.transpose(1, 2).contiguous())

    want = torch.zeros((dst, cout), device="cuda", dtype=torch.float64)
    reached = torch.zeros(dst, device="cuda", dtype=torch.bool)
    for k in range(K ** 3):
        m = int(km.counts[k])
        want.index_add_(0, b[k, :m].long(), x[a[k, :m].long()].double() @ w[k].double().T)
        reached[b[k, :m][a[k, :m] == src - 1].long()] = True
    assert near(run(x), want, K ** 3)
    x[src - 1, 3] = float("inf")
    got = run(x)
    assert bool(reached.any()) and torch.equal(~torch.isfinite(got).all(1), reached)
    # (fp32 matrix cores: a longer chain of roundings; 2.3e-7 of the rms measured for 27 links of 128 channels)
    err, rms = (got.double() - want)[~reached], want.square().mean().sqrt()
    assert float(err.square().mean().sqrt() / rms) <= 6e-7 * max(1.0, K ** 3 / 27.0) ** 0.5


@pytest.mark.parametrize("n,bits,cin,cout,kernel", [(49151, 5, 48, 48, "tile"), (49152, 5, 48, 48, "split"), (56000, 5, 24, 40, "tile"),
                                                    (60000, 5, 40, 24, "tile"), (50000, 5, 128, 32, "split"), (100000, 6, 48, 48, "tile"),
                                                    (200000, 6, 48, 48, "split"), (49152, 6, 48, 128, "split"), (60000, 6, 36, 100, "split"),
                                                    (65535, 6, 40, 256, "split"), (65536, 6, 48, 128, "tile"), (49151, 5, 48, 80, "tile"),
                                                    (49152, 5, 48, 80, "split"), (60000, 6, 48, 80, "tile"), (65536, 5, 48, 80, "split")])
def test_lines(sp, n, bits, cin, cout, kernel):  # noqa: F811
    """Both sides of the lines between this kernel and the tile kernel: rows, and links of an offset a tile (16 and 27); layers that it
    pads, of one and two channel tiles and of tiles of 128 channels, which have the line of 64 k rows."""
    c, km, g = cloud(sp, n, bits, n)
    assert sp.sp_conv_kernel_name(km, cin, cout, torch.float32) == "gather_%s_kernel" % kernel
    x, w = torch.randn((n, cin), device="cuda", generator=g), torch.randn((27, cout, cin), device="cuda", generator=g)
    want = fwd64(km, x, w)
    err, rms = sp.sp_conv_fwd(km, x, w).double() - want, want.square().mean().sqrt()
    assert float(err.square().mean().sqrt() / rms) <= 3e-7
