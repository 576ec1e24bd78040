"""The sort by buckets (most significant digits first, children cut by sampled splitters, finished in LDS) against the
oracle: the edges of its tiles, children and key widths, rows and clusters that a digit cannot part, lists that are
not 16-byte aligned, and the inputs that it hands on to the digit passes."""
import numpy as np
import pytest

from oracle import unisparse_oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2403_05802_amd import binding as B
    return B.Context("cuda:0")


def entries(rng, nr, nc, n, kind):
    """n distinct coordinates (fewer where `kind` repeats itself), in random order."""
    if kind == "sorted" or kind == "uniform":
        lin = rng.choice(nr * nc, n, replace=False) if nr * nc < 1 << 25 else np.unique(rng.integers(0, nr * nc, n))
    elif kind == "heavy":        # half of the entries in two rows, the rest spread
        lin = np.concatenate([rng.integers(0, nr * nc, n // 2), nr // 2 * nc + rng.integers(0, nc, n // 3),
                              (nr - 1) * nc + rng.integers(0, nc, n // 6)])
    elif kind == "clusters":     # rows of very different lengths, most columns within a few hundred of the row
        row = (nr * rng.random(n) ** 3).astype(np.int64)
        col = np.where(rng.random(n) < 0.7, np.clip(row * nc // nr + rng.integers(-200, 201, n), 0, nc - 1), rng.integers(0, nc, n))
        lin = row * nc + col
    else:                        # "powers": keys that crowd towards zero, more in every octave than a cut can part
        lin = (2.0 ** (rng.random(n) * np.log2(nr * nc - 1))).astype(np.int64)
    lin = np.unique(lin)
    if kind != "sorted":
        lin = rng.permutation(lin)
    r, c = (lin // nc).astype(np.int32), (lin % nc).astype(np.int32)
    return r, c, rng.uniform(0.1, 1, r.size).astype(np.float32)


def unaligned(a):
    """The array on the GPU, four bytes past a 16-byte boundary."""
    import torch
    t = torch.empty(a.size + 1, dtype=torch.from_numpy(a[:0]).dtype, device="cuda")
    t[1:] = torch.from_numpy(a).cuda()
    return t[1:]


def run(ctx, nr, nc, r, c, v, d, put):
    """The layout and the kernels of the conversion."""
    from paper_2403_05802_amd import binding as B
    from helpers import us_desc_of
    ctx.enable_profile(); ctx.profile_reset()
    try:
        g = B.us_convert(ctx, nr, nc, put(r), put(c), put(v), us_desc_of(d))
        return g, {e["kernel"]: e["launches"] for e in ctx.profile_report()}
    finally:
        ctx.disable_profile()


# one parent (32 bits at most, up to 65,536 entries): one child and the second, the tile of 4096, the last size; beyond it
# parents of one and of several children, up to 32, 33 and 42 bits; two sizes that stay with the digit passes
SIZES = [(1, 1, 1), (64, 64, 1000), (4096, 4096, 1024), (4096, 4096, 1025), (4096, 4096, 4096), (4096, 4096, 4097), (3, 4097, 9001),
         (4096, 4096, 65536), (4096, 4096, 65537), (4096, 4095, 300_001), (4096, 4097, 65536), (4096, 4097, 65537),
         (1 << 21, 1 << 21, 5000), (1 << 22, 1 << 20, 262_144), (65536, 65536, 270_000), (65537, 65536, 270_001),
         (1 << 21, 1 << 21, 300_000), (5, 1 << 24, 400_000), (1 << 22, 9, 700_003)]


@pytest.mark.parametrize("kind", ["uniform", "sorted", "heavy", "clusters"])
@pytest.mark.parametrize("nr,nc,n", SIZES)
def test_matches_the_oracle(ctx, nr, nc, n, kind):
    from helpers import assert_same_layout, dev
    r, c, v = entries(np.random.default_rng(nr + nc + n), nr, nc, n, kind)
    put = unaligned if kind == "clusters" else dev
    descs = [O.CSR(), O.CSC(), O.COO()] + ([O.DCSR()] if kind == "heavy" else [])
    for d in descs:
        g, launches = run(ctx, nr, nc, r, c, v, d, put)
        if nr * nc > 1:
            passes = 65536 < r.size <= 262144 and nr * nc <= 1 << 24      # three digit passes are as quick there
            assert ("bucket_split" in launches) != passes and ("radix_scatter" in launches) == passes, (d, launches)
        assert_same_layout(g, O.convert(nr, nc, r, c, v, d), f"{kind} {nr}x{nc}, {r.size} entries -> {d}")
        g.free()


def sampled(n, k):
    """Where the sort looks for ns = 64 keys per child among n entries: evenly spaced pieces, a scattered place in each."""
    ns = min(4096, 64 * k, n)
    i = np.arange(ns, dtype=np.uint64)
    return (i * n // ns + ((i * 0x9E3779B1 & 0xFFFFFFFF) >> 8) % (n // ns)).astype(np.int64)


def fullest_bin(keys, width, bins):
    """Most keys of a bin when 64 of them, every len / 64th, cut [0, width) into intervals and each of these is cut evenly."""
    cuts = np.sort(keys[np.arange(64) * len(keys) // 64]).astype(np.float64)
    cuts[0] = 0
    ends = np.append(cuts[1:], width)
    at = np.searchsorted(cuts, keys, side="right") - 1
    each = bins // 64
    inside = np.minimum(((keys - cuts[at]) * each / (ends[at] - cuts[at] + 1)).astype(np.int64), each - 1)
    return np.bincount(at * each + inside).max()


@pytest.mark.parametrize("nr,nc,n", [(4096, 4096, 60_000), (1 << 20, 1 << 20, 400_000)])
def test_keys_that_crowd_in_every_octave(ctx, nr, nc, n):
    from helpers import assert_same_layout, dev
    r, c, v = entries(np.random.default_rng(n), nr, nc, n, "powers")
    for d in (O.CSR(), O.COO()):
        g, launches = run(ctx, nr, nc, r, c, v, d, dev)
        assert "bucket_finish" in launches and "radix_scatter" not in launches, launches
        assert_same_layout(g, O.convert(nr, nc, r, c, v, d), f"{r.size} entries -> {d}")
        g.free()


@pytest.mark.parametrize("clusters,gap", [(70, 1), (16, 1), (30, 3)])
def test_splitters_of_clusters(ctx, clusters, gap):
    """One parent of 32 bits whose keys lie in clusters: more of the sampled keys share a bin than are put in order by
    comparison (33), so the bins of the sample are cut again."""
    from helpers import assert_same_layout, dev
    rng = np.random.default_rng(clusters)
    nr = nc = 65536
    at = rng.integers(0, nr * nc - (1 << 20), clusters)
    lin = np.unique((at[:, None] + gap * np.arange(60_000 // clusters)[None]).ravel())
    lin = rng.permutation(lin)
    keys = lin[sampled(lin.size, -(-lin.size // 1024))]
    assert lin.size <= 65536 and fullest_bin(keys, nr * nc, 4096) > 33
    r, c = (lin // nc).astype(np.int32), (lin % nc).astype(np.int32)
    v = rng.uniform(0.1, 1, r.size).astype(np.float32)
    for d in (O.CSR(), O.COO()):
        g, launches = run(ctx, nr, nc, r, c, v, d, dev)
        assert "bucket_finish" in launches and "radix_scatter" not in launches, launches
        assert_same_layout(g, O.convert(nr, nc, r, c, v, d), str(d))
        g.free()


def test_a_child_that_no_bins_part(ctx):
    """1024 parents of 2048 rows and 2^32 keys each.  Every one holds its largest key, which leaves the 64 keys that cut a
    child without a mark for "none" when it is among them, so the child's range is one interval of 2048 bins; its other keys,
    130 to 2000 of them, lie in the first bin, too many for comparisons.  Which 64 keys are looked at depends on the order
    in which atomics arrive: 64 / m of the children of m keys come here on average, some hundred of the 1024."""
    import torch
    rng = np.random.default_rng(7)
    nr = nc = 1 << 21
    size = rng.integers(130, 1024, 1024)
    size[::16] = rng.integers(1024, 2000, 64)
    assert (64 / size).sum() > 100
    base = np.arange(1024, dtype=np.int64) << 32
    lin = np.concatenate([np.append(b + rng.choice(1 << 21, m, replace=False), b + (1 << 32) - 1) for b, m in zip(base, size)])
    assert np.bincount((lin & 0xFFFFFFFF) * 2048 >> 32).max() == size.sum()     # (in bin 0 of the 2048)
    for d in (O.CSR(), O.COO()):
        launches = on_the_gpu(ctx, nr, nc, torch.from_numpy(lin).cuda(), d)
        assert "bucket_finish" in launches and "radix_scatter" not in launches, launches


def on_the_gpu(ctx, nr, nc, lin, d):
    """Converts a list made on the GPU (distinct row * nc + column in random order) to CSR or COO and compares with torch's
    sort of the same numbers; the kernels of the conversion."""
    import torch
    lin = lin[torch.randperm(lin.numel(), device="cuda")]
    row = torch.div(lin, nc, rounding_mode="floor")
    col, val = (lin - row * nc).int(), torch.arange(lin.numel(), device="cuda", dtype=torch.int32).view(torch.float32)
    g, launches = run(ctx, nr, nc, row.int(), col, val, d, lambda x: x)
    order = torch.sort(lin)
    assert torch.equal(g.val().view(torch.int32), order.indices.int())
    want = torch.div(order.values, nc, rounding_mode="floor")
    assert torch.equal(g.idx(1).long(), order.values - want * nc)
    if d == O.COO():
        assert torch.equal(g.idx(0).long(), want)
    else:
        assert torch.equal(g.ptr(1).long(), torch.searchsorted(want, torch.arange(nr + 1, device="cuda")))
    g.free()
    return launches


# rows that crowd: in the first rows (as in order of length, or an R-MAT graph), in the last ones, in a few that are used at
# all (one share holds every entry), in few rows and the first columns (shares are pieces of rows); small and large tiles
SKEWED = [(1 << 20, 1 << 20, 300_000, 4), (1 << 20, 1 << 20, 1_000_000, 5), (100_003, 100_003, 1_000_000, -5), (5, 1 << 24, 1_500_000, 5),
          (1 << 21, 1 << 21, 2_000_000, 3), ((1 << 21) - 3, 1 << 18, 9_000_000, 8), (1 << 20, 1 << 20, 17_000_000, 6),
          (300_007, 1 << 22, 36_000_000, -8)]


@pytest.mark.parametrize("swap", [False, True])
@pytest.mark.parametrize("nr,nc,n,power", SKEWED)
def test_shares_of_too_many_entries_are_cut(ctx, nr, nc, n, power, swap):
    """A share of the rows with more entries than a parent may have used to send the whole call to the digit passes."""
    import torch
    gen = torch.Generator("cuda").manual_seed(n)
    x = torch.rand(n, device="cuda", dtype=torch.float64, generator=gen) ** abs(power)
    if nr == 5:
        lin = (nr * nc * x).long()
    else:
        row = (x * nr).long() if abs(power) > 4 else torch.randint(0, power, (n,), device="cuda", generator=gen)
        lin = (row if power > 0 else nr - 1 - row) * nc + torch.randint(0, nc, (n,), device="cuda", generator=gen)
    lin = torch.unique(lin)
    if swap:   # the same along the columns, to CSC's order by way of the transposed matrix
        row = torch.div(lin, nc, rounding_mode="floor")
        c, r = row.int(), (lin - row * nc).int()
        order = torch.randperm(lin.numel(), device="cuda", generator=gen)
        val = torch.rand(lin.numel(), device="cuda", generator=gen)
        g, launches = run(ctx, nc, nr, r[order], c[order], val[order], O.CSC(), lambda t: t)
        assert torch.equal(g.val(), val) and torch.equal(g.idx(1), r)
        assert torch.equal(g.ptr(1).long(), torch.searchsorted(row, torch.arange(nr + 1, device="cuda")))
        g.free()
    else:
        launches = on_the_gpu(ctx, nr, nc, lin, O.CSR() if nr < 1 << 21 else O.COO())
    assert "bucket_finish" in launches and "radix_scatter" not in launches, launches


def test_a_parent_of_too_many_entries_goes_to_the_digit_passes(ctx):
    """300,000 entries, every second one in 4 of 2^20 rows, but none of these where the sample looks."""
    from helpers import assert_same_layout, dev
    rng = np.random.default_rng(3)
    nr = nc = 1 << 20
    lin = np.unique(np.concatenate([rng.integers(0, 4 * nc, 150_000), rng.integers(4 * nc, nr * nc, 150_000)]))
    lin = rng.permutation(lin)
    n = lin.size
    ns = n // 2048
    i = np.arange(ns, dtype=np.uint64)
    seen = (i * n // ns + ((i * 0x9E3779B1 & 0xFFFFFFFF) >> 8) % (n // ns)).astype(np.int64)
    light = np.setdiff1d(np.flatnonzero(lin >= 4 * nc), seen)
    for a, b in zip(seen[lin[seen] < 4 * nc], light):
        lin[a], lin[b] = lin[b], lin[a]
    assert (lin < 4 * nc).sum() > 131_072
    r, c = (lin // nc).astype(np.int32), (lin % nc).astype(np.int32)
    v = rng.uniform(0.1, 1, r.size).astype(np.float32)
    for d in (O.CSR(), O.COO()):
        g, launches = run(ctx, nr, nc, r, c, v, d, dev)
        assert launches["radix_scatter"] == 5, launches
        assert_same_layout(g, O.convert(nr, nc, r, c, v, d), str(d))
        g.free()


def test_parents_share_the_rows_that_there_are(ctx):
    """36 M entries, rows up to 2.5 times the average: with parents by the top bits of a row number just above 2^20 half of
    them were empty and the fullest of the others had more entries (175,000) than a parent may have."""
    import torch
    nr, nc = (1 << 20) + 2, 1 << 21
    u = torch.rand(36_000_000, device="cuda", dtype=torch.float64, generator=torch.Generator("cuda").manual_seed(nr))
    row = (nr * (u + 0.6 * torch.sin(2 * np.pi * u) / (2 * np.pi))).long().clamp_(0, nr - 1)
    lin = torch.unique(row * nc + torch.randint(0, nc, row.shape, device="cuda", generator=torch.Generator("cuda").manual_seed(nc)))
    launches = on_the_gpu(ctx, nr, nc, lin, O.CSR())
    assert "bucket_finish" in launches and "radix_scatter" not in launches, launches


# the division of a row number by the rows of a share: rows below, at and above the number of shares, up to 2^31 - 1
@pytest.mark.parametrize("nr,nc,n", [(1023, 4097, 270_000), (1024, 1 << 20, 300_000), (1025, 1 << 20, 300_000), (44, 1 << 22, 270_000),
                                     (45, 1 << 22, 270_000), (1536, 1 << 30, 300_000), (2047, (1 << 31) - 1, 300_000),
                                     ((1 << 31) - 1, 2000, 70_000), ((1 << 21) - 1, 1 << 21, 2_000_000), (1 << 21, 1 << 21, 2_000_000)])
def test_shares_of_rows(ctx, nr, nc, n):
    import torch
    gen = torch.Generator("cuda").manual_seed(n)
    lin = torch.randint(0, nr * nc, (n,), device="cuda", generator=gen)
    ends = torch.tensor([0, nc - 1, (nr - 1) * nc, nr * nc - 1], device="cuda")   # the corners of the matrix among them
    edges = torch.arange(min(nr, 4096), device="cuda") * (nr // min(nr, 4096)) * nc   # first and last entries of rows
    lin = torch.unique(torch.cat([lin, ends, edges, edges + nc - 1]))
    launches = on_the_gpu(ctx, nr, nc, lin, O.COO() if nr > 1 << 24 else O.CSR())
    assert "bucket_finish" in launches and "radix_scatter" not in launches, launches


@pytest.mark.parametrize("n", [1, 1000, 65_536, 1_000_000])
def test_scratch_of_wide_keys_goes_with_the_entries(ctx, n):
    """42 key bits make 1024 parents however few entries there are.  Per entry: the list by parent 8 bytes, a region of 2048
    records of 8 bytes for every child that shares its parent, at most two children per 1024 entries: 40 bytes; the layout
    itself 12; tables of the parents and, per workgroup of the first pass (4096 entries), of their counts 1 byte each."""
    import torch
    from paper_2403_05802_amd import binding as B
    from helpers import dev, us_desc_of
    nr = nc = 1 << 21
    r, c, v = entries(np.random.default_rng(n), nr, nc, n, "uniform")
    r, c, v = dev(r), dev(c), dev(v)
    torch.cuda.synchronize()
    torch.cuda.reset_peak_memory_stats()
    before = torch.cuda.memory_allocated()
    B.us_convert(ctx, nr, nc, r, c, v, us_desc_of(O.COO())).free()
    assert torch.cuda.max_memory_allocated() - before <= 56 * n + 200_000


@pytest.mark.parametrize("nr,nc,n", [(4096, 4096, 30_000), (70_000, 70_000, 300_000)])
def test_errors_are_reported(ctx, nr, nc, n):
    from paper_2403_05802_amd import binding as B
    from helpers import dev, us_desc_of
    rng = np.random.default_rng(n)
    r, c, v = entries(rng, nr, nc, n, "heavy")
    for at in (0, r.size // 2, int(np.flatnonzero(r == nr // 2)[5])):
        r2, c2, v2 = np.append(r, r[at]), np.append(c, c[at]), np.append(v, np.float32(1))
        for d in (O.CSR(), O.CSC(), O.COO()):
            with pytest.raises(B.UnisparseError) as ei:
                B.us_convert(ctx, nr, nc, dev(r2), dev(c2), dev(v2), us_desc_of(d))
            assert ei.value.code == "US_ERR_DUPLICATE"
    for bad in ((nr, 0), (0, nc), (-1, 3), (3, -1), (2**31 - 1, 2**31 - 1)):
        r2, c2, v2 = np.append(r, np.int32(bad[0])), np.append(c, np.int32(bad[1])), np.append(v, np.float32(1))
        for d in (O.CSR(), O.CSC(), O.DCSR(), O.ELL()):
            with pytest.raises(B.UnisparseError) as ei:
                B.us_convert(ctx, nr, nc, dev(r2), dev(c2), dev(v2), us_desc_of(d))
            assert ei.value.code == "US_ERR_INDEX_RANGE"


def test_more_entries_than_the_matrix_has_places(ctx):
    """Four keys in all: shares that no splitter can cut."""
    from paper_2403_05802_amd import binding as B
    from helpers import dev, us_desc_of
    rng = np.random.default_rng(2)
    r, c = rng.integers(0, 2, (2, 600_000)).astype(np.int32)
    for d in (O.CSR(), O.COO()):
        with pytest.raises(B.UnisparseError) as ei:
            B.us_convert(ctx, 2, 2, dev(r), dev(c), dev(np.ones(r.size, np.float32)), us_desc_of(d))
        assert ei.value.code == "US_ERR_DUPLICATE"


@pytest.mark.parametrize("kind", ["uniform", "clusters"])
def test_large_tiles_and_transposing(ctx, kind):
    """8.4 M entries and more (tiles of 12,288 in the first pass), there and back."""
    from paper_2403_05802_amd import binding as B
    from helpers import assert_same_layout, dev, us_desc_of
    nr, nc = 300_007, 1_000_003
    r, c, v = entries(np.random.default_rng(8), nr, nc, 8_500_000 if kind == "uniform" else 11_000_000, kind)
    assert r.size >= 1 << 23
    want = {d: O.convert(nr, nc, r, c, v, d) for d in (O.CSR(), O.CSC())}
    g, launches = run(ctx, nr, nc, r, c, v, O.CSR(), dev)
    if kind == "uniform":
        assert "bucket_finish" in launches and "radix_scatter" not in launches, launches
    assert_same_layout(g, want[O.CSR()], "CSR")
    t = B.us_convert_formatted(ctx, g, us_desc_of(O.CSC()))
    assert_same_layout(t, want[O.CSC()], "CSR -> CSC")
    back = B.us_convert_formatted(ctx, t, us_desc_of(O.CSR()))
    assert_same_layout(back, want[O.CSR()], "CSC -> CSR")
    for x in (g, t, back):
        x.free()
