"""Small launches of the wavefront-private kernel (csrc/sp_conv.hip): four wavefronts a sub-tile with weights read as they are
stored and from the copy, one wavefront a sub-tile, and where the row-stationary and the split kernel begin.  Against fp64: fp32
sums of up to 27 * 128 products (bound 1e-6 of the rms, measured up to 4e-7), bf16 results rounded once (2^-9 of the value, and
the sums' error)."""
import pytest
import torch

from test_gpu_parity import sp  # noqa: F401  (the binding fixture)
from test_gpu_split import cloud, fwd64

pytestmark = pytest.mark.gpu
F, B = torch.float32, torch.bfloat16


@pytest.mark.parametrize("n,bits,cin,cout,dt,kernel", [
    (1, 2, 16, 16, F, "wave"), (63, 2, 32, 32, B, "wave"), (65, 3, 64, 64, B, "wave"), (100, 2, 64, 64, F, "wave"),     # full and nearly empty sub-tiles
    (1500, 4, 16, 48, F, "wave"), (1500, 6, 32, 64, F, "wave"), (4096, 4, 64, 128, B, "wave"), (3000, 4, 128, 256, B, "wave"),
    (16384, 4, 64, 128, B, "wave"), (16385, 5, 128, 64, B, "wave"),                                                        # as many as fit at once, one more
    (16384, 5, 64, 64, F, "wave"), (16385, 5, 64, 64, F, "split"), (32768, 6, 32, 64, F, "wave"), (32769, 6, 32, 64, F, "split"),
    (49152, 5, 32, 32, F, "wave"), (49153, 5, 32, 32, F, "wave"), (81984, 6, 16, 16, F, "wave"),
    (24000, 5, 128, 256, B, "wave"), (16384, 4, 128, 256, B, "dense"), (64000, 5, 64, 64, B, "dense")])
def test_launch_sizes(sp, n, bits, cin, cout, dt, kernel):  # noqa: F811
    c, km, g = cloud(sp, n, bits, n + cin)
    assert sp.sp_conv_kernel_name(km, cin, cout, dt) == "gather_%s_kernel" % kernel
    x, w = torch.randn((n, cin), device="cuda", generator=g).to(dt), torch.randn((27, cout, cin), device="cuda", generator=g).to(dt)
    y = torch.full((n, cout), float("nan"), device="cuda", dtype=dt)
    got = sp.sp_conv_fwd(km, x, w)
    sp.sp_conv_fwd_noalloc(km, x, w, y)
    assert torch.equal(y, got)
    for got, want in ((got, fwd64(km, x, w)), (sp.sp_conv_bwd_data(km, x, w.transpose(1, 2).contiguous()), fwd64(km, x, w.flip(0)))):
        err, rms = (got.double() - want).abs(), want.square().mean().sqrt()
        if dt == B:
            assert bool((err <= want.abs() * 2.0 ** -8 + rms * 1e-5).all())
        else:
            assert float(err.square().mean().sqrt() / rms) <= 1e-6


@pytest.mark.parametrize("n,bits,K,cin,cout,kernel", [
    (8000, 5, 1, 64, 64, "dense"), (3000, 5, 1, 128, 128, "wave"), (30000, 5, 1, 128, 128, "dense"), (8000, 5, 2, 64, 64, "wave"),
    (60000, 5, 2, 64, 64, "dense"), (12000, 4, 2, 64, 192, "dense"), (12000, 4, 2, 128, 128, "wave"), (12000, 4, 3, 64, 64, "wave"),
    (60000, 5, 3, 128, 64, "dense"), (30000, 5, 4, 128, 64, "wave"), (12000, 4, 3, 64, 192, "dense")])
def test_launch_sizes_by_offsets(sp, n, bits, K, cin, cout, kernel):  # noqa: F811
    """Where the row-stationary kernel begins for few offsets and for channels that are no multiples of 128; bf16 results rounded once."""
    c, _, g = cloud(sp, n, bits, n + cin)
    km, _ = sp.sp_kmap_build(c, K, 1, 1)
    assert sp.sp_conv_kernel_name(km, cin, cout, B) == "gather_%s_kernel" % kernel
    x, w = torch.randn((n, cin), device="cuda", generator=g).to(B), torch.randn((K ** 3, cout, cin), device="cuda", generator=g).to(B)
    want = fwd64(km, x, w)
    err, rms = (sp.sp_conv_fwd(km, x, w).double() - want).abs(), want.square().mean().sqrt()
    assert bool((err <= want.abs() * 2.0 ** -8 + rms * 1e-5).all())


@pytest.mark.parametrize("n,bits", [(1, 1), (100, 2), (600, 5), (1500, 4), (3000, 4), (20000, 5)])
@pytest.mark.parametrize("cin,cout,dt", [(16, 16, F), (64, 64, F), (20, 24, F), (64, 64, B), (256, 256, B)])
def test_weight_gradient_of_short_lists(sp, n, bits, cin, cout, dt):  # noqa: F811
    """Lists cut into 1, 2, 4 and 8 strips, partial blocks added in 4 and in 16 slices; fp32 sums (double totals in fp32) of up to n
    products against fp64."""
    c, km, g = cloud(sp, n, bits, n)
    x, dy = torch.randn((n, cin), device="cuda", generator=g).to(dt), torch.randn((n, cout), device="cuda", generator=g).to(dt)
    dw, (pin, pout) = sp.sp_conv_bwd_weight(km, x, dy), km.pairs_strided()
    for k in range(27):
        m = int(km.counts[k])
        want = dy[pout[k, :m].long()].double().T @ x[pin[k, :m].long()].double()
        assert float((dw[k].double() - want).norm()) <= 1e-6 * float(want.norm()) + 1e-6 * m ** 0.5


def test_weights_beyond_the_static_scratch(sp):  # noqa: F811
    """K = 5, 64 -> 512 and 128 -> 320 in bf16: 8 and 10 MB of weights, read where they are stored by the allocation-free call."""
    for n, cin, cout in ((500, 64, 512), (500, 128, 320), (20000, 128, 256)):
        c, _, g = cloud(sp, n, 5, n)
        km, _ = sp.sp_kmap_build(c, 5, 1, 1)
        x, w = torch.randn((n, cin), device="cuda", generator=g).to(B), torch.randn((125, cout, cin), device="cuda", generator=g).to(B)
        y = torch.full((n, cout), float("nan"), device="cuda", dtype=B)
        if sp.sp_conv_kernel_name(km, cin, cout, B) == "gather_wave_kernel" and km.total < n * 125 * (0.06 if cin == 128 else 0.25):
            with pytest.raises(sp.SpError):                   # a map whose layer the row-stationary kernel would not have had
                sp.sp_conv_fwd_noalloc(km, x, w, y)
            continue
        sp.sp_conv_fwd_noalloc(km, x, w, y)
        assert torch.equal(y, sp.sp_conv_fwd(km, x, w))


def test_allocation_free_calls_of_two_streams(sp):  # noqa: F811
    """bf16 layers that the row-stationary kernel has on larger maps leave the static array alone at every size: calls with different
    weights that overlap on two streams give the bits of sp_conv_fwd."""
    shapes = [(1500, 64, 64, 3), (3000, 128, 128, 4), (16384, 64, 128, 4), (64000, 64, 64, 5)]
    for n, cin, cout, bits in shapes:
        c, km, g = cloud(sp, n, bits, n)
        assert km.total >= (0.06 if cin == 128 else 0.25) * 27 * n       # the row-stationary kernel's maps
        x = torch.randn((n, cin), device="cuda", generator=g).to(B)
        ws = [torch.randn((27, cout, cin), device="cuda", generator=g).to(B) for _ in range(2)]
        want = [sp.sp_conv_fwd(km, x, w) for w in ws]
        ys = [[torch.full((n, cout), float("nan"), device="cuda", dtype=B) for _ in range(20)] for _ in ws]
        streams = [torch.cuda.Stream(), torch.cuda.Stream()]
        torch.cuda.synchronize()
        for i in range(20):
            for s, w, y in zip(streams, ws, ys):
                with torch.cuda.stream(s):
                    sp.sp_conv_fwd_noalloc(km, x, w, y[i])
        torch.cuda.synchronize()
        for outs, ref in zip(ys, want):
            assert all(torch.equal(y, ref) for y in outs)


def test_a_captured_forward_pass_of_a_row_stationary_layer_holds_no_pool_memory(sp):  # noqa: F811
    """sp_conv_fwd itself, whose weight copy would be another call's memory by the time of a replay: one node, right on every replay."""
    from test_gpu_streams import node_count
    c, km, g = cloud(sp, 1500, 3, 5)
    x = torch.randn((1500, 64), device="cuda", generator=g).to(B)
    ws = [torch.randn((27, 64, 64), device="cuda", generator=g).to(B) for _ in range(2)]
    want = sp.sp_conv_fwd(km, x, ws[0])
    y = torch.empty_like(want)
    torch.cuda.synchronize()
    graph, side = torch.cuda.CUDAGraph(keep_graph=True), torch.cuda.Stream()
    with torch.cuda.stream(side):
        graph.capture_begin()
        sp.sp_conv_fwd(km, x, ws[0], y)
        graph.capture_end()
    assert node_count(graph) == 1
    graph.instantiate()
    for _ in range(3):
        y.fill_(float("nan"))
        sp.sp_conv_fwd(km, x, ws[1])
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want)
