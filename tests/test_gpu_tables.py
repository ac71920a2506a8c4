"""The forms of the coordinate table (one workgroup's table in LDS, hash table, cell grid) where one ends and the next
begins, and what decides between them: row counts, extent, lattice.  Coordinates, maps and their transposes are whole
numbers: equal to the oracle's, bit for bit."""
import numpy as np
import pytest
import torch

from test_gpu_parity import check_map, dev, random_coords, sp, test_coords_build_matches_oracle, test_kmap_matches_oracle  # noqa: F401
from util import oracle_steps

pytestmark = pytest.mark.gpu
check_set, check_maps = test_coords_build_matches_oracle, test_kmap_matches_oracle
del test_coords_build_matches_oracle, test_kmap_matches_oracle


def scaled(raw, ts, shift=0):
    return raw * np.array([1, ts, ts, ts], np.int32) + np.array([0, shift, shift, shift], np.int32)


@pytest.mark.parametrize("n", [1, 1023, 1024, 1025, 8191, 8192, 8193, 32768, 32769, 65535, 65536, 65537])
def test_row_counts_at_which_the_table_changes(sp, n):  # noqa: F811
    raw = random_coords(n, n, 28, batches=2, lo=-14)
    check_set(sp, "", raw)
    check_maps(sp, "", raw, 1, 3, 1, 1)
    check_maps(sp, "", raw, 1, 3, 2, 1)


N = 70000                                                             # more than the hash form takes for certain
DENSE = random_coords(11, N, 37, batches=3, lo=-19) + np.array([5, 0, 0, 0], np.int32)
CORNER = random_coords(12, N, 40, batches=2, lo=32728) + np.array([65534, 0, 0, 0], np.int32)
LOW = random_coords(13, N, 40, batches=2, lo=-32768)
FAR = random_coords(14, N, 20000, batches=9, lo=-10000)               # a box too large for a grid
PLANE = DENSE * np.array([1, 9, 1, 0], np.int32)
WIDE = random_coords(15, 300000, 4000, batches=2, lo=-2000) // np.array([1, 1, 20, 100], np.int32)   # the same, all columns a thread
CASES = [("grid", DENSE, 1, 3, 1, 1), ("grid_k5", DENSE, 1, 5, 1, 1), ("grid_k4", DENSE, 1, 4, 1, 1), ("grid_k2", DENSE, 1, 2, 1, 1),
         ("grid_d2", DENSE, 1, 3, 1, 2), ("grid_d5", DENSE, 1, 3, 1, 5), ("grid_k5_d7", DENSE, 1, 5, 1, 7),
         ("grid_s2", DENSE, 1, 3, 2, 1), ("grid_s3", DENSE, 1, 3, 3, 1), ("grid_k2s2", DENSE, 1, 2, 2, 1), ("grid_k4s2", DENSE, 1, 4, 2, 1),
         ("plane", PLANE, 1, 3, 1, 1), ("corner_d2", CORNER, 1, 3, 1, 2), ("corner_s2", CORNER, 1, 3, 2, 1), ("low_k5", LOW, 1, 5, 1, 1),
         ("low_s2", LOW, 1, 3, 2, 1), ("hash", FAR, 1, 3, 1, 1), ("hash_s2", FAR, 1, 3, 2, 1), ("hash_k2s2", FAR, 1, 2, 2, 1),
         ("hash_wide", WIDE, 1, 3, 1, 1), ("hash_wide_d2", WIDE, 1, 3, 1, 2), ("hash_wide_s2", WIDE, 1, 3, 2, 1),
         ("ts4", scaled(DENSE, 4), 4, 3, 1, 1), ("ts4_s2", scaled(DENSE, 4), 4, 3, 2, 1), ("ts3_shifted", scaled(DENSE, 3, 1), 3, 3, 1, 1),
         ("ts2_shifted_s2", scaled(DENSE, 2, 1), 2, 3, 2, 1), ("off_lattice", DENSE, 2, 3, 1, 1), ("off_lattice_s2", DENSE, 2, 3, 2, 1)]


# the same sets with fewer rows, in the hash form of middle-sized sets
CASES += [(c[0] + "_40000", c[1][:40000], *c[2:]) for c in CASES if len(c[1]) == N]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_forms_match_oracle(sp, case):  # noqa: F811
    if case[3:5] == (3, 1):
        check_set(sp, case[0], case[1])
    check_maps(sp, *case)


def test_hash_of_more_than_a_million_rows_with_duplicates(sp):  # noqa: F811
    """From 2^20 rows on the insertion looks at the slot before it spends an atomic."""
    check_set(sp, "", WIDE[np.random.default_rng(16).integers(0, 200000, 1_100_000)])


@pytest.mark.parametrize("n", [N, (1 << 21) - 1, 1 << 21, (1 << 21) + 1])
def test_numbering_of_tiles_and_of_one_launch(sp, n):  # noqa: F811
    """Up to 2^21 rows numbered by tiles, beyond in one launch: both forms of table, tiles without a first row (all rows of the
    second half are repeats), the next set's likewise."""
    for some in (random_coords(17, n // 2 + 1, 180, batches=2, lo=-90), random_coords(17, n // 2 + 1, 30000, batches=2, lo=-9000)):
        raw = np.concatenate([some, some[::-1]])[:n]
        check_set(sp, "", raw)
        km, c = sp.sp_kmap_build(sp.sp_coords_build(dev(raw), 1), 2, 2, 1)
        want = oracle_steps(np.unique(raw, axis=0), 2, 2, 1, 1)
        assert c.n == len(want["c_out"]) and np.array_equal(np.sort(km.counts), np.sort(want["counts"]))


def test_out_of_range_row_among_many(sp):  # noqa: F811
    for bad in ([0, 32768, 0, 0], [0, 0, -32769, 0], [65536, 0, 0, 0], [-1, 0, 0, 0]):
        raw = DENSE.copy()
        raw[20000] = bad
        c = sp.sp_coords_build(dev(raw), 1)
        with pytest.raises(sp.SpError) as e:
            _ = c.n
        assert e.value.code == -2 or "outside" in str(e.value)


def test_two_levels_built_without_waiting(sp):  # noqa: F811
    """A stack of strided maps whose counts the host never asked for: every level's grid comes from its parent's box."""
    c0 = sp.sp_coords_build(dev(DENSE), 1)
    k1, c1 = sp.sp_kmap_build(c0, 3, 2, 1)
    k2, c2 = sp.sp_kmap_build(c1, 3, 2, 1)
    k3, _ = sp.sp_kmap_build(c2, 3, 1, 1)
    u, v = np.unique(DENSE, axis=0), lambda a, s: np.unique(a * np.array([1, 0, 0, 0]) + a // s * s * np.array([0, 1, 1, 1]), axis=0)
    assert (c0.n, c1.n, c2.n) == (len(u), len(v(u, 2)), len(v(u, 4)))
    top = {tuple(r) for r in v(u, 4)}
    links = sum((b, x + 4 * i, y + 4 * j, z + 4 * k) in top for b, x, y, z in top for i in (-1, 0, 1) for j in (-1, 0, 1) for k in (-1, 0, 1))
    assert k3.total == links and k1.n_out == c1.n and k2.n_in == c1.n


FULL = np.unique(random_coords(21, 260000, 52, batches=3, lo=-27), axis=0)    # enough rows that the coarse sets are grids too


@pytest.mark.parametrize("resolved", [True, False])
@pytest.mark.parametrize("K,ts,shift", [(2, 1, 0), (3, 1, 0), (2, 2, 1), (2, 3, 2), (3, 4, 0)])
def test_sets_of_half_the_resolution(sp, K, ts, shift, resolved):  # noqa: F811
    """Coarse sets out of the blocks of their parent's grid, level by level: rows, parents, pairs and tables against the oracle's,
    with lowest coordinates odd and even, lattices off zero, row counts known to the host and not."""
    raw = scaled(FULL[np.random.default_rng(ts).permutation(len(FULL))], ts, shift) + np.array([0, 0, ts, 0], np.int32)
    c = sp.sp_coords_build(dev(np.concatenate([raw, raw[:5000]])), ts)
    rows, step = raw, ts
    for _ in range(3):
        if resolved:
            assert c.n == len(rows)
        km, co = sp.sp_kmap_build(c, K, 2, 1)
        want = oracle_steps(rows, K, 2, 1, step)
        assert co.n == len(want["c_out"])
        assert np.array_equal(co.coords().cpu().numpy(), want["c_out"])
        assert np.array_equal(co.inverse().cpu().numpy(), want["parent"])
        if K == 2 and shift:                                           # off the lattice of zero: each row at one place of its cell
            nbr_out, nbr_in = (t.cpu().numpy() for t in km.table()[:2])
            k, o = np.nonzero(nbr_out >= 0)
            assert len(k) == len(rows) and np.array_equal(nbr_in[k, nbr_out[k, o]], o) and np.array_equal(want["parent"][nbr_out[k, o]], o)
            assert np.count_nonzero(nbr_in >= 0) == len(rows) == km.total
            c, rows, step = co, want["c_out"], 2 * step
            shift = 0
            continue
        check_map(sp, km, want, len(rows), len(want["c_out"]))
        for side, i, o, n in ((0, want["pair_in"], want["pair_out"], km.n_out), (1, want["pair_out"], want["pair_in"], km.n_in)):
            table, base = np.full((K ** 3, n), -1, np.int32), 0
            for k, cnt in enumerate(want["counts"]):
                table[k, o[base:base + cnt]] = i[base:base + cnt]
                base += cnt
            assert np.array_equal(km.table()[side].cpu().numpy(), table)
        if K == 3:                                                     # the coarse set's own table is searched
            k1, _ = sp.sp_kmap_build(co, 3, 1, 1)
            assert np.array_equal(k1.counts, oracle_steps(want["c_out"], 3, 1, 1, 2 * step)["counts"])
        c, rows, step = co, want["c_out"], 2 * step


@pytest.mark.parametrize("ts,shift", [(1, 0), (2, 0), (2, 1), (3, -1), (3, 2)])
@pytest.mark.parametrize("box", ["wide", "grid, then wide", "grid"])
def test_both_sides_of_a_cell_map_agree_off_the_lattice(sp, ts, shift, box):  # noqa: F811
    """2 x 2 x 2, stride 2 on sets whose coordinates are no multiples of the tensor stride: a row's place in its cell decides on both
    sides, whatever the form of the two tables (boxes too wide for a grid; a parent with a grid under a coarse set without)."""
    rng = np.random.default_rng(5)
    some = FULL[:90000] if box == "grid" else FAR[:40000]
    if box == "grid, then wide":
        some = np.stack([rng.integers(0, hi, 70000) for hi in (4, 320, 320, 656)], 1).astype(np.int32)
    near = some + rng.integers(0, 2, (len(some), 4)).astype(np.int32) * np.array([0, 1, 1, 1], np.int32)
    rows = scaled(np.concatenate([some, near]), ts, shift)
    rows = rows[np.sort(np.unique(rows, axis=0, return_index=True)[1])]
    assert len(rows) > 65536
    # many repeats: room for a grid in the parent's table, none in that of a set made from its distinct rows
    c = sp.sp_coords_build(dev(np.tile(rows, (24, 1)) if box == "grid, then wide" else rows), ts)
    assert c.n == len(rows)
    km, co = sp.sp_kmap_build(c, 2, 2, 1)
    want = oracle_steps(rows, 2, 2, 1, ts)
    assert np.array_equal(co.coords().cpu().numpy(), want["c_out"]) and np.array_equal(co.inverse().cpu().numpy(), want["parent"])
    nbr_out, nbr_in = (t.cpu().numpy() for t in km.table()[:2])
    k, o = np.nonzero(nbr_out >= 0)
    assert len(k) == len(rows) == km.total == np.count_nonzero(nbr_in >= 0)
    assert np.array_equal(nbr_in[k, nbr_out[k, o]], o) and np.array_equal(want["parent"][nbr_out[k, o]], o)
    if shift == 0:
        check_map(sp, km, want, len(rows), len(want["c_out"]))


def test_memory_of_coarse_sets(sp):  # noqa: F811
    """A set of half the resolution holds what other coarse sets of the same parent hold, once its map is built."""
    c = sp.sp_coords_build(dev(FULL), 1)
    live, held = {}, []

    def alloc(nbytes, stream):
        p = torch.cuda.caching_allocator_alloc(max(nbytes, 512), stream=stream)
        live[p] = nbytes
        return p

    def free(p):
        del live[p]
        torch.cuda.caching_allocator_delete(p)

    sp.sp_set_allocator(alloc, free)
    try:
        for K, stride in ((3, 3), (3, 2), (2, 2)):
            before = sum(live.values())
            km, co = sp.sp_kmap_build(c, K, stride, 1)
            km.close()
            held.append((sum(live.values()) - before, co))
    finally:
        sp.sp_set_allocator()
    assert held[0][0] == held[1][0] == held[2][0] > 0
    for _, co in held:
        co.close()


@pytest.mark.parametrize("cin,cout,bf16", [(32, 32, False), (128, 128, True), (20, 24, False)])
@pytest.mark.parametrize("warm", [True, False])
def test_lists_of_the_input_side_under_capture(sp, cin, cout, bf16, warm):  # noqa: F811
    """The lists and the class order of a strided map's input side are made by the first call that walks them: here on
    another stream than the captured one, or by the captured call itself."""
    c = sp.sp_coords_build(dev(DENSE), 1)
    km, _ = sp.sp_kmap_build(c, 3, 2, 1)
    kt = sp.sp_kmap_transpose(km)
    dt = torch.bfloat16 if bf16 else torch.float32
    g = torch.Generator(device="cuda").manual_seed(1)
    xs = [torch.randn((km.n_out, cin), device="cuda", generator=g).to(dt) for _ in range(3)]
    w = torch.randn((27, cout, cin), device="cuda", generator=g).to(dt)
    kt2 = sp.sp_kmap_transpose(sp.sp_kmap_build(c, 3, 2, 1)[0])
    want = [sp.sp_conv_fwd(kt2, x, w) for x in xs]                       # also the one-time set-up of the kernels
    if warm:
        sp.sp_conv_fwd(kt, xs[0], w)
    x, y = torch.empty_like(xs[0]), torch.empty_like(want[0])
    sp.sp_conv_fwd_noalloc(kt2, xs[0], w, y)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        sp.sp_conv_fwd_noalloc(kt, x, w, y)
    for i in (0, 1, 2):
        x.copy_(xs[i])
        y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want[i])
        assert torch.equal(sp.sp_conv_fwd(kt, xs[i], w), want[i])


@pytest.mark.parametrize("n", [1 << 20, (1 << 20) + 1, 2500000])
def test_lists_and_classes_of_many_tiles(sp, n):  # noqa: F811
    """Beyond 1024 tiles of 1024 rows the sums of earlier tiles come from a prefix launch: pair lists against the neighbour
    table they compact (whole numbers), the lists and the class order of an input side through the convolutions that walk them."""
    g = torch.Generator(device="cuda").manual_seed(n)
    i = torch.randperm(3 << 20, device="cuda", generator=g)[:n].to(torch.int32)       # 5 of 6 sites, or a third of a lattice
    raw = torch.stack([i >> 20, i >> 13 & 127, i >> 6 & 127, i & 63], dim=1).contiguous()
    c = sp.sp_coords_build(raw, 1)
    for K, stride in ((2, 1), (3, 2)):
        km, _ = sp.sp_kmap_build(c, K, stride, 1)
        nbr = km.table()[0]
        pin, pout = km.pairs_strided()
        for k in range(K ** 3):
            dst = torch.nonzero(nbr[k] >= 0)[:, 0]
            m = len(dst)
            assert m == km.counts[k]
            assert torch.equal(pout[k, :m].long(), dst) and torch.equal(pin[k, :m], nbr[k][dst])
    kt = sp.sp_kmap_transpose(km)
    tin, tout = kt.pairs_strided()
    for ch, dt, tol in ((16, torch.float32, 1e-5), (128, torch.bfloat16, 1e-2)):       # link lists; class order
        assert sp.sp_conv_kernel_name(kt, ch, ch, dt) == ("gather_wave_kernel" if ch == 16 else "gather_dense_kernel")
        x = torch.randn((kt.n_in, ch), device="cuda", generator=g).to(dt)
        w = torch.randn((27, ch, ch), device="cuda", generator=g).to(dt)
        want = torch.zeros((kt.n_out, ch), device="cuda")
        for k in range(27):
            m = int(kt.counts[k])
            want.index_add_(0, tout[k, :m], x[tin[k, :m].long()].float() @ w[k].float().T)
        got = sp.sp_conv_fwd(kt, x, w).float()
        assert float((got - want).norm() / want.norm()) <= tol
        assert float((got - want).abs().max() / want.square().mean().sqrt()) <= 50 * tol
