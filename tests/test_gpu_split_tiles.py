"""Tiles of every height of the fp32 layers on the bf16 matrix cores (csrc/sp_conv_split.hip): 64 to 224 rows by channel tile, rows and
links, with last tiles of one row and of a few sub-tiles, one and several channel tiles.  Against fp64: as far off
as fp32 sums of up to 27 * 192 products may be (1.4e-7 of the rms measured, 3e-7 allowed)."""
import pytest
import torch

from test_gpu_parity import sp  # noqa: F401  (the binding fixture)
from test_gpu_split import cloud, fwd64

pytestmark = pytest.mark.gpu


# in the order of the heights: 2 .. 7 halves of 32 rows
@pytest.mark.parametrize("cin,cout,n,bits", [(64, 128, n, 5) for n in (8193, 21825, 60065, 73729, 90113, 100033)] +                # 2 .. 7
                         [(64, 256, 31393, 5), (64, 192, 72865, 5), (64, 192, 41377, 6)] +                                         # 4, 3, 6: channel tiles
                         [(20, 128, 14657, 5), (20, 128, 65025, 5), (32, 128, 24577, 5), (32, 128, 75425, 5),
                          (32, 128, 81921, 6), (32, 128, 56833, 5)] +                                                              # 2 .. 7
                         [(64, 64, 26305, 5), (64, 64, 66721, 5), (64, 64, 60065, 5), (128, 64, 73729, 5), (64, 64, 81921, 6)] +   # 2 .. 6
                         [(32, 64, 73729, 5), (32, 64, 66721, 5), (32, 64, 65505, 6)] +                                             # 2, 3, 4
                         [(128, 32, 87393, 5), (128, 32, 58465, 6), (128, 32, 74081, 6)] +                                         # 3, 4, 5
                         [(48, 48, n, 5) for n in (62785, 100033, 92833)] + [(24, 40, 85761, 5), (96, 96, 100545, 5)])  # 4, 5, 6; 3; 5
def test_heights(sp, cin, cout, n, bits):  # noqa: F811
    c, km, g = cloud(sp, n, bits, n + cin)
    assert sp.sp_conv_kernel_name(km, cin, cout, torch.float32) == "gather_split_kernel"
    x, w = torch.randn((n, cin), device="cuda", generator=g), torch.randn((27, cout, cin), device="cuda", generator=g)
    for got, want in ((sp.sp_conv_fwd(km, x, w), fwd64(km, x, w)),
                      (sp.sp_conv_bwd_data(km, x, w.transpose(1, 2).contiguous()), fwd64(km, x, w.flip(0)))):
        err, rms = got.double() - want, want.square().mean().sqrt()
        assert float(err.square().mean().sqrt() / rms) <= 3e-7
        assert float(err.abs().max() / rms) <= 1e-5


@pytest.mark.parametrize("n,bits,cin,cout,kernel", [(49151, 5, 48, 48, "tile"), (49152, 5, 48, 48, "split"), (56000, 5, 24, 40, "tile"),
                                                    (60000, 5, 40, 24, "tile"), (50000, 5, 128, 32, "split"), (100000, 6, 48, 48, "tile"),
                                                    (200000, 6, 48, 48, "split"), (49152, 6, 48, 128, "split"), (60000, 6, 36, 100, "split"),
                                                    (65535, 6, 40, 256, "split"), (65536, 6, 48, 128, "tile"), (65535, 5, 48, 80, "tile"),
                                                    (65536, 5, 48, 80, "split")])
def test_lines(sp, n, bits, cin, cout, kernel):  # noqa: F811
    """Both sides of the lines between this kernel and the tile kernel: rows, and links of an offset a tile (16 and 27); layers that it
    pads, of one and two channel tiles and of tiles of 128 channels, which have the line of 64 k rows."""
    c, km, g = cloud(sp, n, bits, n)
    assert sp.sp_conv_kernel_name(km, cin, cout, torch.float32) == "gather_%s_kernel" % kernel
    x, w = torch.randn((n, cin), device="cuda", generator=g), torch.randn((27, cout, cin), device="cuda", generator=g)
    want = fwd64(km, x, w)
    err, rms = sp.sp_conv_fwd(km, x, w).double() - want, want.square().mean().sqrt()
    assert float(err.square().mean().sqrt() / rms) <= 3e-7
