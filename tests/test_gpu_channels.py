"""Channel counts that no 16-, 32- or 64-channel tile divides, and the row counts where tiles of 64 and 128 rows begin and
end: forward and both gradients against the fp64 oracle.  Tolerances are the parity bounds (fp32 1e-5, bf16 2e-2 of one
rounding to 8 bits, see util.py): channel counts change nothing about how a term is rounded."""
import numpy as np
import pytest
import torch

from test_gpu_parity import conv_case, full_cubes, random_coords, sp  # noqa: F401  (sp: the binding fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cin,cout", [(1, 1), (3, 16), (5, 64), (6, 32), (7, 13), (17, 33), (20, 24), (24, 48), (48, 20),
                                      (48, 48), (65, 40), (80, 40), (100, 130), (300, 31)])
@pytest.mark.parametrize("bf16", [False, True])
def test_any_channel_count(sp, cin, cout, bf16):  # noqa: F811
    conv_case(sp, random_coords(31 + cin, 1500, 12, batches=2, lo=-5), 1, 3, 1, 1, cin, cout, bf16, seed=7 * cin + cout)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 127, 128, 129, 257])
def test_ragged_tiles(sp, n):  # noqa: F811
    raw = np.unique(random_coords(5 + n, 4 * n, max(2, int(round(n ** (1 / 3))) + 1), batches=2), axis=0)[:n]
    conv_case(sp, raw, 1, 3, 1, 1, 20, 128, False, seed=n)


@pytest.mark.parametrize("K,stride,cin,cout,transposed", [(5, 1, 40, 24, False), (2, 2, 24, 48, False), (2, 2, 48, 24, True),
                                                          (3, 2, 5, 48, False), (1, 1, 33, 17, False)])
def test_other_kernels_and_strides(sp, K, stride, cin, cout, transposed):  # noqa: F811
    for bf16 in (False, True):
        conv_case(sp, full_cubes(8, 2), 1, K, stride, 1, cin, cout, bf16, seed=K + cin, transposed=transposed)


@pytest.mark.parametrize("cin,cout", [(128, 128), (256, 48), (64, 80)])
def test_128_row_tiles_fp32(sp, cin, cout):  # noqa: F811
    # enough rows that the 128-row tiles are chosen; rows not a multiple of 64
    raw = np.unique(random_coords(77, 90000, 60, batches=3), axis=0)[:65601]
    conv_case(sp, raw[np.random.default_rng(2).permutation(len(raw))], 1, 3, 1, 1, cin, cout, False, seed=cin + cout)


@pytest.mark.parametrize("n", [(1 << 17) - 1, 1 << 17, (1 << 17) + 64 * 73 + 1])
@pytest.mark.parametrize("cin,cout,dt", [(16, 16, torch.float32), (32, 96, torch.bfloat16), (64, 64, torch.bfloat16)])
def test_sub_tiles_dealt_in_runs(sp, n, cin, cout, dt):  # noqa: F811
    """From 2^17 rows on the XCDs take runs of eight sub-tiles, the last group of runs may be short: every row is written."""
    g = torch.Generator(device="cuda").manual_seed(n)
    i = torch.randperm(1 << 20, device="cuda", generator=g)[:n].to(torch.int32)
    c = sp.sp_coords_build(torch.stack([i >> 18, i >> 12 & 63, i >> 6 & 63, i & 63], dim=1).contiguous(), 1)
    km, _ = sp.sp_kmap_build(c, 3, 1, 1)
    assert sp.sp_conv_kernel_name(km, cin, cout, dt) == "gather_wave_kernel"
    x = torch.randn((n, cin), device="cuda", generator=g).to(dt)
    w = torch.randn((27, cout, cin), device="cuda", generator=g).to(dt)
    pin, pout = km.pairs_strided()
    want = torch.zeros((n, cout), device="cuda")
    for k in range(27):
        m = int(km.counts[k])
        want.index_add_(0, pout[k, :m], x[pin[k, :m].long()].float() @ w[k].float().T)
    got = sp.sp_conv_fwd(km, x, w).float()
    tol = 1e-5 if dt == torch.float32 else 1e-2
    assert float((got - want).norm() / want.norm()) <= tol
    assert float((got - want).abs().max() / want.square().mean().sqrt()) <= 10 * tol


@pytest.mark.parametrize("n", [1, 65535, 65536])
@pytest.mark.parametrize("cin,cout,dt", [(96, 96, torch.bfloat16), (96, 48, torch.bfloat16), (48, 288, torch.bfloat16), (96, 96, torch.float32)])
def test_weight_gradient_tiles_of_few_links(sp, n, cin, cout, dt):  # noqa: F811
    """96 channels are tiles of 32 below 2^16 links (bf16), of 48 from there on.  Sums of up to 65536 exact products in fp32
    against fp64: the parity bound."""
    i = torch.arange(n, device="cuda", dtype=torch.int32)
    c = sp.sp_coords_build(torch.stack([i * 0, i >> 8, i & 255, i * 0], dim=1).contiguous(), 1)
    km, _ = sp.sp_kmap_build(c, 1, 1, 1)
    g = torch.Generator(device="cuda").manual_seed(n + cin)
    x, dy = (torch.randn((n, ch), device="cuda", generator=g).to(dt) for ch in (cin, cout))
    got = sp.sp_conv_bwd_weight(km, x, dy)[0].double()
    want = dy.double().T @ x.double()
    assert float((got - want).norm() / want.norm()) <= 1e-5


@pytest.mark.parametrize("K", [2, 3, 4, 5])
@pytest.mark.parametrize("cin,cout,dt", [(16, 16, torch.float32), (16, 64, torch.float32), (32, 32, torch.float32), (32, 32, torch.bfloat16),
                                         (32, 64, torch.bfloat16), (64, 32, torch.bfloat16)])
def test_sub_tiles_with_the_most_blocks(sp, K, cin, cout, dt):  # noqa: F811
    """A full box of voxels: sub-tiles with four blocks of nearly every offset, the most there is room for, in a launch large
    enough that none is split; 27 offsets and fewer keep a block's first link, more do not."""
    n = 80 * 64 * 64
    g = torch.Generator(device="cuda").manual_seed(K)
    i = torch.randperm(n, device="cuda", generator=g).to(torch.int32)
    c = sp.sp_coords_build(torch.stack([i * 0, i >> 12, i >> 6 & 63, i & 63], dim=1).contiguous(), 1)
    km, _ = sp.sp_kmap_build(c, K, 1, 1)
    assert sp.sp_conv_kernel_name(km, cin, cout, dt) == "gather_wave_kernel"
    x = torch.randn((n, cin), device="cuda", generator=g).to(dt)
    w = torch.randn((K ** 3, cout, cin), device="cuda", generator=g).to(dt)
    pin, pout = km.pairs_strided()
    want = torch.zeros((n, cout), device="cuda")
    for k in range(K ** 3):
        m = int(km.counts[k])
        want.index_add_(0, pout[k, :m], x[pin[k, :m].long()].float() @ w[k].float().T)
    got = sp.sp_conv_fwd(km, x, w).float()
    assert float((got - want).norm() / want.norm()) <= (1e-5 if dt == torch.float32 else 1e-2)
