"""Kernels whose launch shape depends on the size of the call, at row counts just below, at and above the
tile edges and in every range of the dispatch rules, against float64 on the same device."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def spv():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2007_16100_amd import spv as s
    s.lib()
    return s


def rand(gen, *shape, dtype=torch.float32, std=1.0):
    return (torch.randn(*shape, generator=gen, device="cuda") * std).to(dtype)


def close16(got, ref, dtype):
    """One rounding to the storage type (half an ulp: 2^-9 of a bf16, 2^-12 of an f16 value, taken
    twice for values next to a rounding boundary) plus float32 sums of at most 27 * 256 terms of
    order max|ref| / sqrt(terms), whose rounding is below 2^-14 of the largest output."""
    ulp = 2.0 ** -8 if dtype == torch.bfloat16 else 2.0 ** -11
    d = (got.double() - ref).abs()
    assert torch.isfinite(got.float()).all()
    assert bool((d <= ulp * ref.abs() + 2.0 ** -14 * ref.abs().max()).all()), float((d / ref.abs().max()).max())


# rows around the tile edges (64, 128, 192, 256, 384 and 512 rows of a workgroup); a table with and without
# 16-byte alignment; a device row count; the same bits again
@pytest.mark.parametrize("cin,cout,dtype", [(32, 32, "bf16"), (96, 96, "f16"), (64, 128, "bf16"), (256, 96, "bf16"),
                                            (128, 256, "f16"), (256, 256, "bf16")])
@pytest.mark.parametrize("m", [1, 65, 511, 9001, 31_100, 70_001, 110_003])
def test_conv_nbr_tiles(spv, cin, cout, dtype, m):
    dt = {"bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    gen = torch.Generator(device="cuda").manual_seed(cin * 1000 + cout + m)
    x, W = rand(gen, m, cin, dtype=dt), rand(gen, 27, cin, cout, dtype=dt, std=(27 * cin) ** -0.5)
    sc, sh = torch.rand(cout, generator=gen, device="cuda") + 0.5, rand(gen, cout)
    res = rand(gen, m, cout, dtype=dt)
    # a fifth of the entries present, runs of rows without any at an offset (blocks that are skipped)
    nbr = torch.randint(1, m + 1, (m, 27), generator=gen, device="cuda", dtype=torch.int32)
    nbr[torch.rand(m, 27, generator=gen, device="cuda") < 0.8] = 0
    nbr[m // 3: m // 2, 5:20] = 0
    buf = torch.zeros(m * 27 + 1, dtype=torch.int32, device="cuda")
    table = buf[1:].view(m, 27) if m % 2 else buf[:-1].view(m, 27)  # odd m: 4-byte aligned only
    table.copy_(nbr)
    live = m - m // 7
    xd, ref = x.double(), torch.zeros(live, cout, dtype=torch.float64, device="cuda")
    for k in range(27):
        j = torch.nonzero(nbr[:live, k])[:, 0]
        ref[j] += xd[(nbr[j, k] - 1).long()] @ W[k].double()
    ref = (ref * sc + sh + res[:live].double()).relu()
    ws = spv.Workspace.for_ops(max(m, 64), 256)
    out = torch.full((m, cout), 7.0, dtype=dt, device="cuda")
    P = spv.spv_pack_weights(W)
    m_dev = torch.tensor([live], dtype=torch.int64, device="cuda")
    spv.spv_sparse_conv_nbr_packed(ws, x, table, P, cout, m, m_out_dev=m_dev, scale=sc, shift=sh, relu=True, res=res,
                                   out=out)
    close16(out[:live], ref, dt)
    assert bool((out[live:] == 7.0).all())  # rows past the count stay
    again = torch.empty_like(out)
    spv.spv_sparse_conv_nbr_packed(ws, x, table, P, cout, m, m_out_dev=m_dev, scale=sc, shift=sh, relu=True, res=res,
                                   out=again)
    assert torch.equal(again[:live].view(torch.int16), out[:live].view(torch.int16))


# Row counts among which the rule takes each tile that it ever takes, at every pair of widths (64-row tiles up to
# 8,232 rows, or 5,530 or 4,100 at 96 or 256 output channels, 128-row tiles of a slice of the channels up to twice
# that, 128-row tiles of all up to twice that again, 192, 256 and up to 512 rows above): the same bits from all.
@pytest.mark.parametrize("cin", [32, 64, 96, 128, 256])
@pytest.mark.parametrize("cout,dtype", [(32, "bf16"), (64, "f16"), (96, "bf16"), (128, "f16"), (256, "bf16")])
def test_conv_nbr_every_tile(spv, cin, cout, dtype):
    dt = {"bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    gen = torch.Generator(device="cuda").manual_seed(cin * 1000 + cout)
    m = 70_001
    x, W = rand(gen, m, cin, dtype=dt), rand(gen, 27, cin, cout, dtype=dt, std=(27 * cin) ** -0.5)
    nbr = torch.randint(1, m + 1, (m, 27), generator=gen, device="cuda", dtype=torch.int32)
    nbr[torch.rand(m, 27, generator=gen, device="cuda") < 0.7] = 0
    nbr[m // 3: m // 2, 5:20] = 0
    xd, ref = x.double(), torch.zeros(m, cout, dtype=torch.float64, device="cuda")
    for k in range(27):
        j = torch.nonzero(nbr[:, k])[:, 0]
        ref[j] += xd[(nbr[j, k] - 1).long()] @ W[k].double()
    ws, P = spv.Workspace.for_ops(m, 256), spv.spv_pack_weights(W)
    whole = spv.spv_sparse_conv_nbr_packed(ws, x, nbr, P, cout, m)
    close16(whole, ref, dt)
    for rows in (3000, 6001, 9003, 12_005, 20_000, 28_009, 40_003, 58_111):
        part = spv.spv_sparse_conv_nbr_packed(ws, x, nbr, P, cout, rows)
        assert torch.equal(part.view(torch.int16), whole[:rows].view(torch.int16)), rows


# A device row count far below the capacity that the tile was picked for: the live rows are spread over the chip
# up to 49,152 of them (12 waves of 16 rows; 32,768 of 8 waves, half of that in two slices of 256 channels)
@pytest.mark.parametrize("cin,cout,dtype", [(32, 32, "f16"), (96, 64, "bf16"), (128, 128, "bf16"), (256, 96, "f16"),
                                            (64, 256, "f16"), (256, 256, "bf16")])
def test_conv_nbr_few_live_rows(spv, cin, cout, dtype):
    dt = {"bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    gen = torch.Generator(device="cuda").manual_seed(cin * 1000 + cout)
    cap = 120_000
    x, W = rand(gen, cap, cin, dtype=dt), rand(gen, 27, cin, cout, dtype=dt, std=(27 * cin) ** -0.5)
    nbr = torch.randint(1, cap + 1, (cap, 27), generator=gen, device="cuda", dtype=torch.int32)
    nbr[torch.rand(cap, 27, generator=gen, device="cuda") < 0.7] = 0
    ws, P, res = spv.Workspace.for_ops(cap, 256), spv.spv_pack_weights(W), rand(gen, cap, cout, dtype=dt)
    whole = spv.spv_sparse_conv_nbr_packed(ws, x, nbr, P, cout, cap, res=res)
    for live in (0, 1, 17, 4096, 4097, 12_289, 16_384, 16_385, 32_769, 49_152, 49_153, 120_000):
        out = torch.full((cap, cout), 7.0, dtype=dt, device="cuda")
        spv.spv_sparse_conv_nbr_packed(ws, x, nbr, P, cout, cap, res=res, out=out,
                                       m_out_dev=torch.tensor([live], dtype=torch.int64, device="cuda"))
        assert torch.equal(out[:live].view(torch.int16), whole[:live].view(torch.int16)), live
        assert bool((out[live:] == 7.0).all()), live


# 16, 32 and 64 rows of a workgroup and the capacities at which the rule changes between them; widths
# that are no multiple of 4 (element loads), of 16, and over one workgroup's 64 output channels
@pytest.mark.parametrize("cin,cout,dtype", [(16, 16, "f32"), (5, 19, "f32"), (48, 70, "f32"), (6, 9, "bf16"),
                                            (20, 33, "f16")])
@pytest.mark.parametrize("m", [1, 17, 1500, 16_385, 32_769])
def test_conv_rows_tiles(spv, cin, cout, dtype, m):
    dt = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    gen = torch.Generator(device="cuda").manual_seed(cin * 1000 + cout + m)
    side = int((4 * m) ** (1 / 3)) + 1
    cell = torch.randperm(side ** 3, generator=gen, device="cuda")[:m].sort().values
    m = len(cell)
    coords = torch.stack([torch.zeros_like(cell), cell // side ** 2, cell // side % side, cell % side], 1).int()
    ws = spv.Workspace.for_ops(max(m, 64), 256)
    km = spv.spv_kernel_map(ws, coords.contiguous())
    assert spv.spv_conv_kernel(27, cin, cout, dt, m, m, km.total) == 2
    x, W = rand(gen, m, cin, dtype=dt), rand(gen, 27, cin, cout, dtype=dt, std=(27 * cin) ** -0.5)
    W[4, 0, 0] = float("inf")  # reaches the rows that have offset 4 and no other
    res = rand(gen, m, cout, dtype=dt)
    out = spv.spv_sparse_conv_sliced(ws, x, km.off, km.pairs, W, cin, cout, m, res=res)
    assert spv.spv_status_check(ws) == 0
    off, pairs = km.off.tolist(), km.pairs.long()
    ref, xd = res.double(), x.double()
    for k in range(27):
        i, j = pairs[off[k]: off[k + 1]].T
        ref[j] += xd[i] @ W[k].double()
    fine = torch.isfinite(ref)
    assert bool((fine == torch.isfinite(out.double())).all())
    d, scale = (out.double() - ref)[fine].abs(), ref[fine].abs()
    # half an ulp of the storage type (twice) and float32 sums of 27 * 48 terms at most
    ulp = {"f32": 2.0 ** -23, "bf16": 2.0 ** -8, "f16": 2.0 ** -11}[dtype]
    assert bool((d <= ulp * scale + 2.0 ** -18 * scale.max()).all()), float((d / scale.max()).max())


# Each offset's products are summed by themselves.  With u = 2^-24, a float32 sum of n terms of equal variance is
# off by u sqrt(n / 6) of its size in the root mean square (the rounding of a step is at most u of a partial sum,
# a third of its square on average, and the partial sums' squares grow as 1 .. n); so a row of P offsets of cin
# products is off by u sqrt(cin / 6 + P / 6), and once more by its own rounding.  One chain over a wave's seven
# offsets would be off by u sqrt(7 cin / 6).
@pytest.mark.parametrize("cin,cout", [(64, 16), (96, 33), (256, 64)])
@pytest.mark.parametrize("side", [12, 30])  # 16 and 32 rows of a workgroup
def test_conv_rows_f32_precision(spv, cin, cout, side):
    gen = torch.Generator(device="cuda").manual_seed(cin + side)
    cell = torch.arange(side ** 3, device="cuda")
    coords = torch.stack([torch.zeros_like(cell), cell // side ** 2, cell // side % side, cell % side], 1).int()
    m = len(cell)
    ws = spv.Workspace.for_ops(m, 256)
    km = spv.spv_kernel_map(ws, coords.contiguous())
    x, W = rand(gen, m, cin), rand(gen, 27, cin, cout)
    out = spv.spv_sparse_conv(ws, x, km.off, km.pairs, W, m)
    off, pairs = km.off.tolist(), km.pairs.long()
    ref, xd = torch.zeros(m, cout, dtype=torch.float64, device="cuda"), x.double()
    for k in range(27):
        i, j = pairs[off[k]: off[k + 1]].T
        ref[j] += xd[i] @ W[k].double()
    err = float((out.double() - ref).norm() / ref.norm())
    assert err <= 2.0 ** -24 * (cin / 6 + 27 / 6 + 1) ** 0.5, err


def stride2(spv, gen, m):
    """A random set of m fine voxels, its stride-2 map, the parents and offsets of the voxels."""
    side = int((3 * m) ** (1 / 3)) + 2
    cell = torch.randperm(side ** 3, generator=gen, device="cuda")[:m].sort().values
    coords = torch.stack([torch.zeros_like(cell), cell // side ** 2, cell // side % side, cell % side], 1).int()
    ws = spv.Workspace.for_ops(max(len(cell), 64), 256)
    km = spv.spv_kernel_map(ws, coords.contiguous(), K=2, stride=2)
    mc = int(km.m_out_dev.item())
    off, pairs = km.off.tolist(), km.pairs[: km.total].long()
    parent, kof = torch.empty(2, len(cell), dtype=torch.long, device="cuda")
    for k in range(8):
        i, j = pairs[off[k]: off[k + 1]].T
        parent[i], kof[i] = j, k
    return ws, km, mc, parent, kof


# the 2x2x2 conv by output and the upsampling (64 or 128 coarse rows of a workgroup, the output channels in one
# to eight passes), around the edges of their tiles
@pytest.mark.parametrize("fine,coarse,dtype", [(32, 64, "bf16"), (96, 96, "f16"), (96, 128, "bf16"), (64, 256, "bf16"),
                                               (256, 32, "f16"), (256, 256, "bf16")])
@pytest.mark.parametrize("m", [1, 130, 2049, 30_011, 90_001])
def test_stride2_tiles(spv, fine, coarse, dtype, m):
    dt = {"bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    gen = torch.Generator(device="cuda").manual_seed(fine * 1000 + coarse + m)
    ws, km, mc, parent, kof = stride2(spv, gen, m)
    m = len(parent)
    x, W = rand(gen, m, fine, dtype=dt), rand(gen, 8, fine, coarse, dtype=dt, std=(2 * fine) ** -0.5)
    sc, sh = torch.rand(coarse, generator=gen, device="cuda") + 0.5, rand(gen, coarse)
    ref = torch.zeros(mc, coarse, dtype=torch.float64, device="cuda")
    for k in range(8):
        i = torch.nonzero(kof == k)[:, 0]
        ref[parent[i]] += x[i].double() @ W[k].double()
    y = spv.spv_sparse_conv(ws, x, km.off, km.pairs, W, mc, scale=sc, shift=sh)
    assert spv.spv_status_check(ws) == 0
    close16(y, ref * sc + sh, dt)
    # an infinite weight reaches the rows that have its offset and no other
    Wi = W.clone()
    Wi[3, 0, 1] = float("inf")
    yi = spv.spv_sparse_conv(ws, x, km.off, km.pairs, Wi, mc, scale=sc, shift=sh)
    has = torch.zeros(mc, dtype=torch.bool, device="cuda")
    has[parent[kof == 3]] = True
    assert bool((torch.isfinite(yi[:, 1].float()) == ~has).all())
    close16(yi[~has], (ref * sc + sh)[~has], dt)
    # a workspace without room for the table of 8: the pairs themselves
    small = pairs_workspace(mc, fine, coarse)
    close16(spv.spv_sparse_conv(small, x, km.off, km.pairs, W, mc, scale=sc, shift=sh), ref * sc + sh, dt)

    z, Wt = rand(gen, mc, coarse, dtype=dt), rand(gen, 8, coarse, fine, dtype=dt, std=coarse ** -0.5)
    su, hu, res = torch.rand(fine, generator=gen, device="cuda") + 0.5, rand(gen, fine), rand(gen, m, fine, dtype=dt)
    children = spv.spv_map_children(ws, km.off, km.pairs, m, mc)
    refu = torch.empty(m, fine, dtype=torch.float64, device="cuda")
    for k in range(8):
        i = torch.nonzero(kof == k)[:, 0]
        refu[i] = z[parent[i]].double() @ Wt[k].double()
    up = spv.spv_sparse_conv_up(ws, z, children, Wt, fine, m, scale=su, shift=hu, relu=True, res=res)
    close16(up, (refu * su + hu + res.double()).relu(), dt)
    packed = spv.spv_sparse_conv_up_packed(ws, z, children, spv.spv_pack_weights(Wt), fine, m, scale=su, shift=hu,
                                           relu=True, res=res)
    assert torch.equal(packed.view(torch.int16), up.view(torch.int16))


def pairs_workspace(mc, cin, cout):
    """A workspace with room for the pairs' kernel of a 2x2x2 map and none for its table of 8: the status
    header, the tile bounds of each offset and the packed weights, each at a multiple of 256 bytes."""
    from paper_2007_16100_amd import spv
    return spv.Workspace(256 + (8 * (-(-mc // 16) + 1) * 4 + 255) // 256 * 256 + 8 * cin * cout * 2)


# the 2x2x2 conv by output sums each offset's products by themselves, on the table of 8 and on the pairs: the
# same bits whichever of the two a workspace has room for, infinite weights and sums among them
@pytest.mark.parametrize("cin,cout,dtype", [(32, 32, "bf16"), (64, 96, "f16"), (96, 128, "bf16"), (128, 256, "f16"),
                                            (256, 96, "bf16"), (256, 256, "f16")])
@pytest.mark.parametrize("m", [1, 130, 5003, 30_011, 120_001])
def test_down_same_bits_on_table_and_pairs(spv, cin, cout, dtype, m):
    dt = {"bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    gen = torch.Generator(device="cuda").manual_seed(cin * 1000 + cout + m)
    ws, km, mc, parent, kof = stride2(spv, gen, m)
    x, W = rand(gen, len(parent), cin, dtype=dt), rand(gen, 8, cin, cout, dtype=dt, std=(2 * cin) ** -0.5)
    W[5, 0, 3] = float("inf")
    sc, sh = torch.rand(cout, generator=gen, device="cuda") + 0.5, rand(gen, cout)
    small = pairs_workspace(mc, cin, cout)
    table, pairs = (spv.spv_sparse_conv(w, x, km.off, km.pairs, W, mc, scale=sc, shift=sh) for w in (ws, small))
    assert spv.spv_status_check(ws) == 0 and spv.spv_status_check(small) == 0
    assert torch.equal(table.view(torch.int16), pairs.view(torch.int16))


# the same for the table of 8, whose rule takes its largest tile above 16,486 to 100,078 coarse rows
@pytest.mark.parametrize("cin", [32, 64, 96, 128, 256])
@pytest.mark.parametrize("cout,dtype", [(32, "f16"), (64, "bf16"), (96, "f16"), (128, "bf16"), (256, "f16")])
def test_down_every_tile(spv, cin, cout, dtype):
    dt = {"bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    gen = torch.Generator(device="cuda").manual_seed(cin * 1000 + cout)
    ws, km, mc, parent, kof = stride2(spv, gen, 290_000)
    assert mc > 100_100
    x, W = rand(gen, len(parent), cin, dtype=dt), rand(gen, 8, cin, cout, dtype=dt, std=(2 * cin) ** -0.5)
    pairs = spv.spv_sparse_conv(pairs_workspace(mc, cin, cout), x, km.off, km.pairs, W, mc)
    ref = torch.zeros(mc, cout, dtype=torch.float64, device="cuda")
    for k in range(8):
        i = torch.nonzero(kof == k)[:, 0]
        ref[parent[i]] += x[i].double() @ W[k].double()
    close16(pairs, ref, dt)
    for rows in (3000, 6001, 9003, 12_005, 23_000, 29_009, 40_003, 58_111, 70_001, mc):
        part = spv.spv_sparse_conv(ws, x, km.off, km.pairs, W, rows)
        assert torch.equal(part.view(torch.int16), pairs[:rows].view(torch.int16)), rows
    for live in (0, 1, 5003, 33_001):  # of a buffer for all
        out = torch.full((mc, cout), 7.0, dtype=dt, device="cuda")
        spv.spv_sparse_conv(ws, x, km.off, km.pairs, W, mc, out=out,
                            m_out_dev=torch.tensor([live], dtype=torch.int64, device="cuda"))
        assert torch.equal(out[:live].view(torch.int16), pairs[:live].view(torch.int16)), live
        assert bool((out[live:] == 7.0).all()), live


# a 2x2x2 map read backwards has one offset per output row, also where the coarse side's buffer has the fine
# side's capacity: it runs on the pairs (the table of 8 would do eight times the products), which shows in the
# workspace past what the pairs need staying as it was
@pytest.mark.parametrize("m", [1, 3001])
@pytest.mark.parametrize("fine,coarse", [(64, 128), (96, 96)])
def test_transposed_2x2x2_at_equal_capacities(spv, fine, coarse, m):
    gen = torch.Generator(device="cuda").manual_seed(m + fine)
    _, km, mc, parent, kof = stride2(spv, gen, m)
    m = len(parent)
    z = torch.full((m, coarse), float("nan"), dtype=torch.bfloat16, device="cuda")  # rows past mc: never read
    z[:mc] = rand(gen, mc, coarse, dtype=torch.bfloat16)
    Wup = rand(gen, 8, coarse, fine, dtype=torch.bfloat16, std=coarse ** -0.5)
    Wdown = Wup.transpose(1, 2).contiguous()  # whose input gradient is the same product
    ref = torch.empty(m, fine, dtype=torch.float64, device="cuda")
    for k in range(8):
        i = torch.nonzero(kof == k)[:, 0]
        ref[i] = z[parent[i]].double() @ Wup[k].double()
    used = pairs_workspace(m, coarse, fine).nbytes
    ws = spv.Workspace(used + 64 * m + 4096)
    start = ws.ptr.value - ws.buf.data_ptr()
    for call in (lambda: spv.spv_sparse_conv(ws, z, km.off, km.pairs, Wup, m, transposed=True),
                 lambda: spv.spv_sparse_conv_dgrad(ws, z, km.off, km.pairs, Wdown, m)):
        ws.buf.fill_(0x5A)
        close16(call(), ref, torch.bfloat16)
        assert spv.spv_status_check(ws) == 0
        assert bool((ws.buf[start + used:] == 0x5A).all())


# 16-bit widths of the tile kernel whose pair list has no 32-bit byte offsets (its capacity counts, not its
# pairs) run on the rows kernel, over the tile kernel's plan of up to 128 rows
@pytest.mark.parametrize("cin,cout", [(32, 32), (96, 64)])
@pytest.mark.parametrize("m", [100, 5003])
def test_rows_kernel_on_the_tile_kernels_plan(spv, cin, cout, m):
    gen = torch.Generator(device="cuda").manual_seed(m + cin)
    ws, km, mc, parent, kof = stride2(spv, gen, m)
    m = len(parent)
    pairs = torch.empty((0xFFFFE000 // 8 + 1, 2), dtype=torch.int32, device="cuda")
    pairs[: km.total] = km.pairs[: km.total]
    assert spv.spv_conv_kernel(8, cin, cout, torch.bfloat16, mc, m, len(pairs), True) == 2
    z, W = rand(gen, mc, cin, dtype=torch.bfloat16), rand(gen, 8, cin, cout, dtype=torch.bfloat16, std=cin ** -0.5)
    ref = torch.empty(m, cout, dtype=torch.float64, device="cuda")
    for k in range(8):
        i = torch.nonzero(kof == k)[:, 0]
        ref[i] = z[parent[i]].double() @ W[k].double()
    out = spv.spv_sparse_conv(ws, z, km.off, pairs, W, m, transposed=True)
    assert spv.spv_status_check(ws) == 0
    close16(out, ref, torch.bfloat16)


# A wave of the linear kernels takes blocks of 16 rows at a stride of 65,536 rows, two per turn of its loop: row
# counts with one block per wave, with a second for a few waves, a third, a ragged last one
@pytest.mark.parametrize("cin,cout,dtype", [(32, 32, "bf16"), (96, 256, "f16"), (128, 128, "bf16"), (256, 96, "bf16"),
                                            (256, 256, "f16"), (160, 64, "bf16")])
@pytest.mark.parametrize("m", [65_536, 65_537, 131_090, 200_003])
@pytest.mark.parametrize("residual", ["none", "before", "after"])
def test_linear_blocks_per_wave(spv, cin, cout, dtype, m, residual):
    dt = {"bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    gen = torch.Generator(device="cuda").manual_seed(cin * 1000 + cout + m)
    live = m - 3 if m % 2 else m
    x, W = rand(gen, m, cin, dtype=dt), rand(gen, cin, cout, dtype=dt, std=cin ** -0.5)
    sc, sh = torch.rand(cout, generator=gen, device="cuda") + 0.5, rand(gen, cout)
    res = None if residual == "none" else rand(gen, m, cout, dtype=dt)
    out = torch.full((m, cout), 7.0, dtype=dt, device="cuda")
    spv.spv_linear(spv.Workspace.for_ops(64, 256), x, W, m_dev=torch.tensor([live], device="cuda"), scale=sc, shift=sh,
                   relu=True, res=res, res_after_act=residual == "after", out=out)
    ref = (x[:live].double() @ W.double()) * sc + sh
    r = 0 if res is None else res[:live].double()
    close16(out[:live], (ref + r).relu() if residual == "before" else ref.relu() + r, dt)
    assert bool((out[live:] == 7.0).all())  # rows past the count stay


# key widths on both sides of where the sort's geometry changes (24, 28 and 32 bits below a bucket's first
# fine bin) and of where the buckets end and the passes take over (40 bits)
@pytest.mark.parametrize("bits", [31, 32, 33, 36, 37, 40, 41])
@pytest.mark.parametrize("n", [300, 70_001, 262_144])
def test_sort_key_widths(spv, bits, n):
    gen = torch.Generator(device="cuda").manual_seed(bits * 10 + n)
    # z in 7 bits, y in 12, the rest shared by x and the batch; clusters make buckets of many sizes
    bx = min(bits - 19, 14)
    fields = (bits - 19 - bx, bx, 12, 7)
    q = torch.stack([torch.randint(0, 2 ** b, (n,), generator=gen, device="cuda") for b in fields], 1)
    q[n // 2:, 1] = q[n // 2:, 1] % 97 + 5
    q[0], q[1] = 0, torch.tensor([2 ** (bits - 19 - bx) - 1, 2 ** bx - 1, 4095, 127])
    xyz = (q[:, 1:] + 0.5).float().contiguous()
    ws = spv.Workspace.for_ops(n, 16)
    vox = spv.spv_voxelize(ws, xyz, 1.0, batch=q[:, 0].int().contiguous())
    keys = ((q[:, 0] << 40) | (q[:, 1] << 20) | (q[:, 2] << 8) | q[:, 3])
    ref, of, counts = torch.unique(keys, return_inverse=True, return_counts=True)
    assert vox.m == len(ref) and spv.spv_status_check(ws) == 0
    c = vox.coords[: vox.m].long()
    assert torch.equal((c[:, 0] << 40) | (c[:, 1] << 20) | (c[:, 2] << 8) | c[:, 3], ref)
    assert torch.equal(vox.pt2vox.long(), of) and torch.equal(vox.counts[: vox.m].long(), counts)
