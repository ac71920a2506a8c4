"""fp32 layers on the bf16 matrix cores (csrc/sp_conv_split.hip): few and many rows (tiles of every height are test_gpu_split_tiles.py), slices and
channel tiles that reach past the layer, values that bf16 cannot hold.  Against fp64: the parity bound, and no further off than
fp32 matrix cores are (measured 1.1e-7 to 2e-7 of the rms for up to 125 * 64 products; 3e-7 allowed)."""
import numpy as np
import pytest
import torch

from test_gpu_parity import conv_case, dev, full_cubes, sp  # noqa: F401  (sp: the binding fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cin,cout", [(128, 128), (100, 128), (64, 128), (128, 384), (192, 128)])
def test_small_layers(sp, cin, cout):  # noqa: F811
    """Against the oracle, all three passes; the forward pass on this kernel, and the data gradient of 100 and 128 channels."""
    raw = full_cubes(12, 5)
    km, _ = sp.sp_kmap_build(sp.sp_coords_build(dev(raw), 1), 3, 1, 1)
    assert sp.sp_conv_kernel_name(km, cin, cout, torch.float32) == "gather_split_kernel"
    conv_case(sp, raw, 1, 3, 1, 1, cin, cout, False, seed=7 * cin + cout)


@pytest.mark.parametrize("K,stride,dil,transposed", [(2, 1, 1, False), (2, 2, 1, False), (2, 2, 1, True), (3, 2, 1, False), (3, 2, 1, True),
                                                     (3, 1, 2, False), (4, 1, 1, False), (4, 2, 1, False), (4, 2, 1, True), (5, 1, 1, False), (5, 2, 1, True), (1, 1, 1, False)])
def test_other_maps(sp, K, stride, dil, transposed):  # noqa: F811
    """64, 27, 8 and 125 offsets (two rounds of 64 in a tile's first wavefront), strided and transposed maps, dilation, both directions;
    against fp64 (an error of sums in fp32: it grows with the square root of the links that are added)."""
    cin = cout = 128
    km, _ = sp.sp_kmap_build(sp.sp_coords_build(dev(full_cubes(26, 1)), 1), K, stride, dil)
    if transposed:
        km = sp.sp_kmap_transpose(km)
    assert [sp.sp_conv_kernel_name(km, cin, cout, torch.float32, d) for d in (0, 1)] == ["gather_split_kernel"] * 2
    g = torch.Generator(device="cuda").manual_seed(K)
    x, dy = torch.randn((km.n_in, cin), device="cuda", generator=g), torch.randn((km.n_out, cout), device="cuda", generator=g)
    w = torch.randn((K ** 3, cout, cin), device="cuda", generator=g)
    pin, pout = km.pairs()
    at = np.concatenate([[0], np.cumsum(km.counts)])
    y, dx = torch.zeros((km.n_out, cout), device="cuda", dtype=torch.float64), torch.zeros((km.n_in, cin), device="cuda", dtype=torch.float64)
    for k in range(K ** 3):
        i, o = pin[at[k]:at[k + 1]].long(), pout[at[k]:at[k + 1]].long()
        y.index_add_(0, o, x[i].double() @ w[k].double().T)
        dx.index_add_(0, i, dy[o].double() @ w[k].double())
    for got, want in ((sp.sp_conv_fwd(km, x, w), y), (sp.sp_conv_bwd_data(km, dy, w), dx)):
        err, rms = got.double() - want, want.square().mean().sqrt()
        assert float(err.square().mean().sqrt() / rms) <= 3e-7 * max(1.0, K ** 3 / 27.0) ** 0.5
        assert float(err.abs().max() / rms) <= 1e-5


def cloud(sp, n, bits, seed):  # noqa: F811
    """n voxels of 4 clouds of 2^bits cells per axis."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    i = torch.randperm(4 << 3 * bits, device="cuda", generator=g)[:n].to(torch.int32)
    m = (1 << bits) - 1
    c = sp.sp_coords_build(torch.stack([i >> 3 * bits, i >> 2 * bits & m, i >> bits & m, i & m], dim=1).contiguous(), 1)
    return c, sp.sp_kmap_build(c, 3, 1, 1)[0], g


def fwd64(km, x, w):
    pin, pout = km.pairs_strided()
    y = torch.zeros((km.n_out, w.shape[1]), device="cuda", dtype=torch.float64)
    for k in range(w.shape[0]):
        m = int(km.counts[k])
        y.index_add_(0, pout[k, :m].long(), x[pin[k, :m].long()].double() @ w[k].double().T)
    return y


@pytest.mark.parametrize("n,bits,cin,cout", [(8193, 5, 64, 128), (16257, 5, 64, 128), (1100, 4, 128, 128), (1217, 4, 100, 128),
                                             (16449, 5, 64, 64), (32769, 6, 32, 64), (16513, 5, 64, 128),
                                             (20000, 5, 100, 128),                                                                 # slices past the last channel
                                             (65536, 5, 96, 96), (65537, 5, 24, 40), (70000, 5, 48, 48), (70001, 5, 36, 100), (66000, 6, 128, 32)])
def test_rows_slices_and_channel_tiles(sp, n, bits, cin, cout):  # noqa: F811
    c, km, g = cloud(sp, n, bits, n + cin)
    assert sp.sp_conv_kernel_name(km, cin, cout, torch.float32) == "gather_split_kernel"
    x, w = torch.randn((n, cin), device="cuda", generator=g), torch.randn((27, cout, cin), device="cuda", generator=g)
    for got, want in ((sp.sp_conv_fwd(km, x, w), fwd64(km, x, w)),
                      (sp.sp_conv_bwd_data(km, x, w.transpose(1, 2).contiguous()), fwd64(km, x, w.flip(0)))):   # the input side: offsets reversed
        err, rms = got.double() - want, want.square().mean().sqrt()
        assert float(err.square().mean().sqrt() / rms) <= 3e-7
        assert float(err.abs().max() / rms) <= 1e-5


@pytest.mark.parametrize("n,bits,K,cin,cout,kernel", [
    (40000, 5, 1, 64, 128, "wave"), (40000, 5, 2, 64, 128, "split"), (40000, 6, 2, 32, 128, "wave"), (30000, 6, 2, 32, 128, "split"),      # in place of wave
    (16385, 8, 3, 128, 128, "tile"), (16385, 6, 3, 128, 128, "split"), (12000, 6, 3, 36, 100, "tile"), (20000, 6, 3, 36, 100, "split"),    # of tile, under 64 k rows
    (66000, 6, 3, 64, 40, "tile"), (66000, 5, 3, 64, 40, "split"), (66000, 6, 3, 128, 64, "split"), (66000, 6, 3, 72, 56, "tile"),         # .. from there on
    (66000, 6, 5, 96, 96, "tile"), (66000, 5, 3, 24, 40, "split"), (66000, 6, 3, 128, 32, "split"),
    (66000, 5, 3, 80, 24, "tile"), (66000, 5, 3, 96, 96, "split")])
def test_links_of_a_tile_and_offset(sp, n, bits, K, cin, cout, kernel):  # noqa: F811
    """Both sides of the lines that the links of an offset in a tile of rows draw; the results on each against fp64 (1e-6 of the rms
    for the other kernels' sums of up to 125 * 128 products)."""
    c, _, g = cloud(sp, n, bits, n + cin)
    km, _ = sp.sp_kmap_build(c, K, 1, 1)
    assert sp.sp_conv_kernel_name(km, cin, cout, torch.float32) == "gather_%s_kernel" % kernel
    x, w = torch.randn((n, cin), device="cuda", generator=g), torch.randn((K ** 3, cout, cin), device="cuda", generator=g)
    want = fwd64(km, x, w)
    err, rms = sp.sp_conv_fwd(km, x, w).double() - want, want.square().mean().sqrt()
    assert float(err.square().mean().sqrt() / rms) <= (3e-7 if kernel == "split" else 1e-6)


@pytest.mark.parametrize("cin,cout", [(64, 64), (32, 64), (128, 128)])
def test_values_beyond_bf16(sp, cin, cout):  # noqa: F811
    """Infinities, NaN and values that round to a bf16 infinity give what fp32 multiply-adds give, and only where they reach;
    subnormal pieces keep their places."""
    c, km, g = cloud(sp, 40000, 5, 5)
    x, w = torch.randn((km.n_in, cin), device="cuda", generator=g), torch.randn((27, cout, cin), device="cuda", generator=g)
    x[5, 3], x[100, 7], x[200, 1], x[300, 2], w[3, 5, 6] = float("inf"), float("nan"), 3.4e38, -float("inf"), 1e38
    want = fwd64(km, x, w)
    ok = want.abs() < 3.4e38
    got = sp.sp_conv_fwd(km, x, w)
    assert torch.equal(torch.isnan(got), torch.isnan(want)) and torch.equal(torch.isinf(got), ~ok & ~torch.isnan(want))
    assert torch.allclose(got[ok].double(), want[ok], rtol=1e-4, atol=1e-3)
    x = torch.randn((km.n_in, cin), device="cuda", generator=g) * 1e-33
    w = torch.randn((27, cout, cin), device="cuda", generator=g)
    want, got = fwd64(km, x, w), sp.sp_conv_fwd(km, x, w).double()
    assert float((got - want).norm() / want.norm()) <= 3e-7


@pytest.mark.parametrize("size_x,size_w", [(1e-33, 1.0), (1e-35, 1.0), (1e-37, 1e4), (1e-40, 1e30), (1.0, 1e-36), (1e10, 1e-38), (1e30, 1e-37),
                                           (1e-18, 1e-18), (1e-22, 1e18), (1e30, 1.0), (1e10, 1e14), (1e25, 1e10), (1.0, 1e33)])
def test_magnitudes(sp, size_x, size_w):  # noqa: F811
    """Any finite size of either operand: fp32 products and sums carry 24 bits, down to values that are themselves subnormal, as long
    as the results are normal numbers (fp32 matrix cores, to which the largest results fall back: 2.5e-7 of the rms)."""
    c, km, g = cloud(sp, 40000, 5, 5)
    x, w = torch.randn((km.n_in, 64), device="cuda", generator=g) * size_x, torch.randn((27, 64, 64), device="cuda", generator=g) * size_w
    assert sp.sp_conv_kernel_name(km, 64, 64, torch.float32) == "gather_split_kernel"
    for got, want in ((sp.sp_conv_fwd(km, x, w), fwd64(km, x, w)), (sp.sp_conv_bwd_data(km, x, w), fwd64(km, x, w.flip(0).transpose(1, 2)))):
        err, rms = got.double() - want, want.square().mean().sqrt()
        print("rms error", float(err.square().mean().sqrt() / rms), "largest", float(err.abs().max() / rms))
        assert float(err.square().mean().sqrt() / rms) <= 3e-7
        assert float(err.abs().max() / rms) <= 1e-5


def test_without_allocations(sp):  # noqa: F811
    """Weights' pieces that fit the static scratch: the bits of sp_conv_fwd; pieces that do not, though the weights would: within
    the parity bound."""
    c, km, g = cloud(sp, 20000, 5, 9)
    x, w = torch.randn((km.n_in, 100), device="cuda", generator=g), torch.randn((27, 384, 100), device="cuda", generator=g)
    y = torch.full((km.n_out, 384), float("nan"), device="cuda")
    assert sp.sp_conv_kernel_name(km, 100, 384, torch.float32) == "gather_split_kernel"     # 4.0 MB of weights, 8 MB of padded pieces
    sp.sp_conv_fwd_noalloc(km, x, w, y)
    want = fwd64(km, x, w)
    assert not torch.equal(y, sp.sp_conv_fwd(km, x, w)) and float((y.double() - want).norm() / want.norm()) <= 1e-6
    for cin, cout, same in ((64, 128, True), (128, 256, True), (64, 640, False)):
        x, w = torch.randn((km.n_in, cin), device="cuda", generator=g), torch.randn((27, cout, cin), device="cuda", generator=g)
        y = torch.full((km.n_out, cout), float("nan"), device="cuda")
        if not same:
            with pytest.raises(sp.SpError):       # a narrow layer whose copy does not fit either is refused, as ever
                sp.sp_conv_fwd_noalloc(km, x, w, y)
            continue
        sp.sp_conv_fwd_noalloc(km, x, w, y)
        assert torch.equal(y, sp.sp_conv_fwd(km, x, w))
