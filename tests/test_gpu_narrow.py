"""Layers with few channels on one side (plain multiply-adds, csrc/sp_conv_narrow.hip): where threads per row, rows per workgroup,
chunks of 27 offsets and turns over the rows begin and end.  Tolerances are the parity bounds (fp32 1e-5, bf16 2e-2): sums of
at most 125 * 256 products, each link's first."""
import numpy as np
import pytest
import torch

from test_gpu_parity import conv_case, full_cubes, random_coords, sp  # noqa: F401  (sp: the binding fixture)
from test_gpu_split import cloud

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cin,cout", [(1, 1), (2, 7), (3, 33), (4, 32), (5, 20), (7, 16), (8, 16), (3, 128), (6, 256), (8, 8), (1, 64)])
@pytest.mark.parametrize("bf16", [False, True])
def test_narrow_layers(sp, cin, cout, bf16):  # noqa: F811
    conv_case(sp, random_coords(3 + cin, 1500, 12, batches=2, lo=-5), 1, 3, 1, 1, cin, cout, bf16, seed=11 * cin + cout)


F, B = torch.float32, torch.bfloat16


@pytest.mark.parametrize("rows,bits,K,cin,cout,dt,fwd,bwd", [
    # forward cin -> cout and data gradient cout -> cin: 1 where the kernel has it; by rows, channels and offsets
    (1000, 4, 3, 8, 8, F, 0, 0), (100000, 6, 3, 8, 8, F, 1, 1), (1000, 4, 3, 8, 8, B, 0, 0), (100000, 6, 3, 8, 8, B, 1, 1),
    (1000, 4, 3, 6, 16, F, 1, 0), (100000, 6, 3, 6, 16, B, 1, 1), (4096, 4, 3, 7, 18, B, 1, 0), (4096, 4, 3, 2, 64, F, 1, 1),
    (100000, 6, 3, 2, 64, F, 0, 1), (100000, 6, 3, 2, 64, B, 0, 1), (100000, 6, 3, 4, 32, F, 0, 1), (16384, 5, 3, 4, 128, F, 0, 1),
    (40000, 5, 3, 4, 128, B, 0, 0), (16384, 5, 3, 2, 256, F, 0, 1), (40000, 5, 3, 6, 64, F, 0, 1), (40000, 5, 3, 6, 64, B, 0, 0),
    (16384, 5, 4, 1, 64, F, 1, 1), (16384, 5, 4, 8, 8, F, 0, 0), (16384, 5, 4, 3, 8, B, 1, 0), (1000, 4, 5, 3, 8, F, 1, 0),
    (100000, 6, 5, 3, 8, F, 1, 1), (100000, 6, 5, 8, 8, F, 1, 1), (16384, 5, 5, 1, 64, B, 1, 1), (1000, 4, 5, 8, 8, B, 0, 0),
    (4096, 4, 2, 3, 32, F, 1, 1), (100000, 6, 2, 2, 64, F, 0, 1), (40000, 5, 2, 8, 8, B, 1, 1)])
def test_where_the_kernel_begins(sp, rows, bits, K, cin, cout, dt, fwd, bwd):  # noqa: F811
    """Both sides of each line of the choice, and what runs there, against fp64: fp32 sums of up to 125 * 128 products; bf16 results
    rounded once (2^-9 of the value, and the sums' error)."""
    c, _, g = cloud(sp, rows, bits, rows + cin)
    km, _ = sp.sp_kmap_build(c, K, 1, 1)
    assert [sp.sp_conv_kernel_name(km, cin, cout, dt, d) == "gather_narrow_kernel" for d in (0, 1)] == [bool(fwd), bool(bwd)]
    x, dy = (torch.randn((c.n, ch), device="cuda", generator=g).to(dt) for ch in (cin, cout))
    w = torch.randn((K ** 3, cout, cin), device="cuda", generator=g).to(dt)
    y, dx = (torch.zeros((c.n, ch), device="cuda", dtype=torch.float64) for ch in (cout, cin))
    pin, pout = km.pairs_strided()
    for k in range(K ** 3):
        m = int(km.counts[k])
        a, b = pin[k, :m].long(), pout[k, :m].long()
        y.index_add_(0, b, x[a].double() @ w[k].double().T)
        dx.index_add_(0, a, dy[b].double() @ w[k].double())
    for got, want in ((sp.sp_conv_fwd(km, x, w), y), (sp.sp_conv_bwd_data(km, dy, w), dx)):
        err, rms = (got.double() - want).abs(), want.square().mean().sqrt()
        if dt == B:
            assert bool((err <= want.abs() * 2.0 ** -8 + rms * 1e-5).all())
        else:
            assert float(err.square().mean().sqrt() / rms) <= 1e-6


@pytest.mark.parametrize("K,stride,transposed", [(1, 1, False), (2, 2, False), (2, 2, True), (3, 2, False), (3, 2, True), (5, 1, False)])
def test_narrow_layers_of_other_maps(sp, K, stride, transposed):  # noqa: F811
    for bf16 in (False, True):
        conv_case(sp, full_cubes(8, 2), 1, K, stride, 1, 3, 32, bf16, seed=K, transposed=transposed)


@pytest.mark.parametrize("n", [1, 63, 64, 85, 86, 128 * 2048 + 1])
def test_narrow_rows(sp, n):  # noqa: F811
    """Few rows, and more than the resident workgroups take in one turn; forward and data gradient against fp64."""
    g = torch.Generator(device="cuda").manual_seed(n)
    i = torch.randperm(1 << 20, device="cuda", generator=g)[:n].to(torch.int32)
    c = sp.sp_coords_build(torch.stack([i >> 18, i >> 12 & 63, i >> 6 & 63, i & 63], dim=1).contiguous(), 1)
    km, _ = sp.sp_kmap_build(c, 3, 1, 1)
    pin, pout = km.pairs_strided()
    for cin, cout in ((3, 12), (3, 32)):
        assert sp.sp_conv_kernel_name(km, cin, cout, torch.float32, 0) == sp.sp_conv_kernel_name(km, 3, 32, torch.float32, 1) == "gather_narrow_kernel"
        x, dy = (torch.randn((n, ch), device="cuda", generator=g) for ch in (cin, cout))
        w = torch.randn((27, cout, cin), device="cuda", generator=g)
        y, dx = (torch.zeros((n, ch), device="cuda", dtype=torch.float64) for ch in (cout, cin))
        for k in range(27):
            m = int(km.counts[k])
            a, b = pin[k, :m].long(), pout[k, :m].long()
            y.index_add_(0, b, x[a].double() @ w[k].double().T)
            dx.index_add_(0, a, dy[b].double() @ w[k].double())
        for got, want in ((sp.sp_conv_fwd(km, x, w), y), (sp.sp_conv_bwd_data(km, dy, w), dx)):
            assert float((got.double() - want).norm() / want.norm()) <= 1e-6


def test_values_that_are_not_finite_stay_in_their_rows(sp):  # noqa: F811
    c = sp.sp_coords_build(torch.from_numpy(random_coords(9, 4000, 20, batches=2)).cuda(), 1)
    km, _ = sp.sp_kmap_build(c, 3, 1, 1)
    x, w = torch.randn((km.n_in, 3), device="cuda"), torch.randn((27, 32, 3), device="cuda")
    x[5, 1], x[77, 0], w[4, 3, 2] = float("inf"), float("nan"), float("inf")
    pin, pout = km.pairs()
    koff = np.concatenate([[0], np.cumsum(km.counts)])
    for got, f, mats in ((sp.sp_conv_fwd(km, x, w), x, w.transpose(1, 2)), (sp.sp_conv_bwd_data(km, torch.ones_like(w[0, :, 0]).repeat(km.n_out, 1), w), None, w)):
        want = torch.zeros_like(got)
        for k in range(27):
            a, b = pin[koff[k]:koff[k + 1]].long(), pout[koff[k]:koff[k + 1]].long()
            src = f[a] if f is not None else torch.ones((len(a), 32), device="cuda")
            want.index_add_(0, b if f is not None else a, (src[:, :, None] * mats[k][None]).sum(1))
        assert torch.equal(torch.isfinite(got), torch.isfinite(want))
        ok = torch.isfinite(want)
        assert torch.allclose(got[ok], want[ok], rtol=1e-4, atol=1e-4)
