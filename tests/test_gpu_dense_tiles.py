"""Row-stationary kernel (csrc/sp_conv_dense.hip): tiles of 256 destination rows taken in position-class order and as they are, with
one row, full and nearly empty last tiles, every channel tile and slice width.  bf16 results rounded once (2^-8 of the value, and
1e-5 of the rms for fp32 sums of up to 27 * 256 products)."""
import pytest
import torch

from test_gpu_parity import sp  # noqa: F401  (the binding fixture)
from test_gpu_split import cloud, fwd64

pytestmark = pytest.mark.gpu
B = torch.bfloat16


def close(got, want):
    err, rms = (got.double() - want).abs(), want.square().mean().sqrt()
    return bool((err <= want.abs() * 2.0 ** -8 + rms * 1e-5).all())


@pytest.mark.parametrize("n", [1, 63, 255, 256, 257, 1000])
@pytest.mark.parametrize("K,cin,cout", [(2, 64, 128), (3, 64, 64), (3, 128, 64), (3, 128, 128), (3, 256, 256), (3, 64, 256)])
def test_class_order(sp, n, K, cin, cout):  # noqa: F811
    """Data gradient of a strided layer: destinations are the fine rows in the order of their position classes."""
    c, _, g = cloud(sp, n, 4, n + K)
    km, _ = sp.sp_kmap_build(c, K, 2, 1)
    assert sp.sp_conv_kernel_name(km, cin, cout, B, 1) == "gather_dense_kernel"
    dy, w = torch.randn((km.n_out, cout), device="cuda", generator=g).to(B), torch.randn((K ** 3, cout, cin), device="cuda", generator=g).to(B)
    pin, pout = km.pairs_strided()
    want = torch.zeros((km.n_in, cin), device="cuda", dtype=torch.float64)
    for k in range(K ** 3):
        m = int(km.counts[k])
        want.index_add_(0, pin[k, :m].long(), dy[pout[k, :m].long()].double() @ w[k].double())
    assert close(sp.sp_conv_bwd_data(km, dy, w), want)


@pytest.mark.parametrize("n,cin,cout", [(64001, 128, 128), (64255, 128, 64), (64257, 64, 128), (64000, 64, 64), (20001, 256, 256), (30000, 256, 128)])
def test_rows_as_they_are(sp, n, cin, cout):  # noqa: F811
    c, km, g = cloud(sp, n, 5, n)
    assert sp.sp_conv_kernel_name(km, cin, cout, B) == "gather_dense_kernel"
    x, w = torch.randn((n, cin), device="cuda", generator=g).to(B), torch.randn((27, cout, cin), device="cuda", generator=g).to(B)
    assert close(sp.sp_conv_fwd(km, x, w), fwd64(km, x, w))
    assert close(sp.sp_conv_bwd_data(km, x, w.transpose(1, 2).contiguous()), fwd64(km, x, w.flip(0)))
