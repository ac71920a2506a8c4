"""Calls at the limits of the convolution kernels: weights beyond the scratch of the allocation-free entry point, features
beyond 32-bit byte offsets."""
import pytest
import torch

from test_gpu_parity import dev, random_coords, sp  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,cin,cout,bf16,in_place", [(3, 256, 256, False, True), (3, 300, 200, False, False), (5, 48, 512, False, True),
                                                      (5, 96, 400, True, True), (5, 65, 300, False, False)])
def test_noalloc_takes_weights_beyond_its_scratch(sp, K, cin, cout, bf16, in_place):  # noqa: F811
    """More than 4 MiB of weights: whole fragments are read in place (same bits as sp_conv_fwd), other widths run on the
    plain kernel (fp32 sums of up to 8125 terms in another order: the parity bounds)."""
    c = sp.sp_coords_build(dev(random_coords(3, 300, 7)), 1)
    km, _ = sp.sp_kmap_build(c, K, 1, 1)
    dt = torch.bfloat16 if bf16 else torch.float32
    g = torch.Generator(device="cuda").manual_seed(1)
    x = torch.randn((c.n, cin), device="cuda", generator=g).to(dt)
    w = torch.randn((K ** 3, cout, cin), device="cuda", generator=g).to(dt)
    assert w.numel() * w.element_size() > 4 << 20
    y = torch.full((c.n, cout), float("nan"), device="cuda", dtype=dt)
    sp.sp_conv_fwd_noalloc(km, x, w, y)
    want = sp.sp_conv_fwd(km, x, w)
    if in_place:
        assert torch.equal(y, want)
    assert float((y.float() - want.float()).norm() / want.float().norm()) <= (1e-2 if bf16 else 1e-5)


def test_features_beyond_32_bit_offsets(sp):  # noqa: F811
    """4.3 GB of features: the tile kernel with 64-bit addresses, against fp64 products of some of the rows."""
    side, cin, cout = 257, 64, 64
    n = side ** 3
    i = torch.arange(n, device="cuda", dtype=torch.int32)
    raw = torch.stack([torch.zeros_like(i), i // (side * side), i // side % side, i % side], dim=1).contiguous()
    c = sp.sp_coords_build(raw, 1)
    km, _ = sp.sp_kmap_build(c, 1, 1, 1)
    x = torch.randn((n, cin), device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))
    w = torch.randn((1, cout, cin), device="cuda", generator=torch.Generator(device="cuda").manual_seed(2))
    assert x.numel() * 4 > 1 << 32
    assert sp.sp_conv_kernel_name(km, cin, cout, torch.float32) == "gather_tile_kernel"
    y = sp.sp_conv_fwd(km, x, w)
    at = torch.cat([torch.arange(0, n, 1009, device="cuda"), torch.arange(n - 200, n, device="cuda")])
    want = x[at].double() @ w[0].double().T
    assert float((y[at].double() - want).norm() / want.norm()) <= 1e-6


@pytest.mark.parametrize("K,n,wide,narrow,bf16", [(3, 1_050_000, 1040, 24, False),   # 4.4 GB of features, 17 slices of 64
                                                  (3, 1_050_000, 2056, 40, True),    # the same of bf16, 33 slices
                                                  (5, 8_650_000, 32, 16, False),     # 4.3 GB per list, slices of 32
                                                  (5, 8_650_000, 32, 16, True)])
def test_several_offsets_and_slices_beyond_32_bit_offsets(sp, K, n, wide, narrow, bf16):  # noqa: F811
    """The 64-bit tile kernels with many offsets and slices, forward and data gradient (the reversed side of the same
    lists), against fp64 sums for some of the rows.  fp32: the parity bound; bf16: one rounding, at most 2^-8 of a value."""
    dt, elt = (torch.bfloat16, 2) if bf16 else (torch.float32, 4)
    g = torch.Generator(device="cuda").manual_seed(n + wide)
    side = 256 if K == 5 else 128                      # 4 clouds, an eighth of the sites taken
    i = torch.randperm(4 * side ** 3, device="cuda", generator=g)[:n].to(torch.int32)
    c = sp.sp_coords_build(torch.stack([i // side ** 3, i // side ** 2 % side, i // side % side, i % side], dim=1).contiguous(), 1)
    km, _ = sp.sp_kmap_build(c, K, 1, 1)
    kvol = K ** 3
    assert max(n * wide * elt, n * kvol * 4) > 1 << 32
    at = torch.cat([torch.arange(0, n, n // 500, device="cuda"), torch.arange(n - 100, n, device="cuda")])
    nbr = km.table()[0][:, at].long()
    f = torch.randn((n, wide), device="cuda", generator=g).to(dt)
    for backward in (False, True):
        assert sp.sp_conv_kernel_name(km, *((narrow, wide) if backward else (wide, narrow)), dt, int(backward)) == "gather_tile_kernel"
        w = torch.randn((kvol, wide, narrow) if backward else (kvol, narrow, wide), device="cuda", generator=g).to(dt)
        got = sp.sp_conv_bwd_data(km, f, w) if backward else sp.sp_conv_fwd(km, f, w)
        want = torch.zeros((len(at), narrow), device="cuda", dtype=torch.float64)
        for k in range(kvol):
            rows = torch.where(nbr[k, :, None] >= 0, f[nbr[k].clamp_min(0)], torch.zeros((), device="cuda", dtype=dt)).double()
            want += rows @ (w[kvol - 1 - k].double() if backward else w[k].double().T)
        assert float((got[at].double() - want).norm() / want.norm()) <= (2.0 ** -8 if bf16 else 1e-5)


@pytest.mark.parametrize("cin,cout,bf16", [(20, 24, False), (65, 40, True), (3, 128, False), (128, 100, False), (128, 128, False)])
def test_without_memory_for_scratch(sp, cin, cout, bf16):  # noqa: F811
    """An allocator that has nothing to give: convolutions need weight copies, padded rows and partial blocks only to be
    fast.  (Layers of the other kernels report SP_ERR_ALLOC.)"""
    c = sp.sp_coords_build(dev(random_coords(3, 300, 7)), 1)
    km, _ = sp.sp_kmap_build(c, 3, 1, 1)
    dt = torch.bfloat16 if bf16 else torch.float32
    g = torch.Generator(device="cuda").manual_seed(1)
    x, dy = (torch.randn((c.n, ch), device="cuda", generator=g).to(dt) for ch in (cin, cout))
    w = torch.randn((27, cout, cin), device="cuda", generator=g).to(dt)
    calls = [lambda: sp.sp_conv_fwd(km, x, w), lambda: sp.sp_conv_bwd_data(km, dy, w)]
    if cin % 16 or cout % 16:
        calls.append(lambda: sp.sp_conv_bwd_weight(km, x, dy))
    want = [f().float() for f in calls]
    asked = []
    sp.sp_set_allocator(lambda nbytes, stream: asked.append(nbytes) or 0, lambda ptr: None)
    try:
        got = [f().float() for f in calls]
    finally:
        sp.sp_set_allocator()
    assert asked
    for a, b in zip(got, want):   # sums of up to 3500 terms in another order; one rounding to bf16
        assert float((a - b).norm() / b.norm()) <= (1e-2 if bf16 else 1e-5)


@pytest.mark.parametrize("cin,cout,K", [(64, 64, 3), (64, 128, 3), (128, 64, 3), (128, 256, 3), (64, 192, 5)])
def test_forward_of_row_stationary_layers_without_memory(sp, cin, cout, K):  # noqa: F811
    """bf16 layers that the row-stationary kernel, which needs no weight copy, has on larger maps: the forward pass needs no memory
    on small ones either, and gives the same bits."""
    c = sp.sp_coords_build(dev(random_coords(3, 900, 7)), 1)
    km, _ = sp.sp_kmap_build(c, K, 1, 1)
    assert km.total >= 0.25 * K ** 3 * c.n
    g = torch.Generator(device="cuda").manual_seed(1)
    x = torch.randn((c.n, cin), device="cuda", generator=g).to(torch.bfloat16)
    w = torch.randn((K ** 3, cout, cin), device="cuda", generator=g).to(torch.bfloat16)
    want = sp.sp_conv_fwd(km, x, w)
    sp.sp_set_allocator(lambda nbytes, stream: 0, lambda ptr: None)
    try:
        got = sp.sp_conv_fwd(km, x, w)
    finally:
        sp.sp_set_allocator()
    assert torch.equal(got, want)
