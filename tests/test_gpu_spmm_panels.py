"""SpMM over entries grouped by row, a panel of columns of X at a time: column counts around every panel shape, rows and lists
around the sixteen entries of a lane group, the 64 of a wavefront and the 512 of a tile, few entries in very many rows, rows of X
and Y that begin at any float, and operands of more than 4 GB."""
import numpy as np
import pytest
import scipy.sparse as sp
import torch

import helpers as H

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2403_05802_amd import binding as B
    return B.Context("cuda:0")


# row lengths in their order; columns are drawn from 1 .. ncols - 1 (column 0 has no entry, its row of X is infinite: nothing of
# it may reach a result, also where the last tile is not full)
PATTERNS = {
    "one entry": [0, 0, 1],
    "groups": [16, 16, 0, 15, 17, 1, 31, 32, 33, 0, 0, 0, 48, 7],
    "wavefronts": [64, 63, 65, 0, 1, 127, 128, 129, 1, 1, 1, 61],
    "a full tile": [500, 12],
    "a full tile and one": [512, 1],
    "one less": [3, 508],
    "rows of whole tiles": [512, 512, 0, 1024, 512],
    "one long row": [5000],
    "long rows cut anywhere": [5, 1500, 0, 2, 700, 1, 1, 1200, 3],
    "single entries, many empty rows": [0, 1] * 1500 + [0] * 900 + [1],
}


def matrix(pattern, rng, ncols=6000):
    length = np.array(PATTERNS[pattern])
    row = np.repeat(np.arange(length.size), length).astype(np.int32)
    col = np.concatenate([1 + rng.choice(ncols - 1, k, replace=False) for k in length]).astype(np.int32)
    return length, row, col, rng.uniform(-1, 1, row.size).astype(np.float32), ncols


def descs():
    from paper_2403_05802_amd import binding as B
    return [B.us_desc_preset(B.US_F_CSR), B.us_desc_preset(B.US_F_COO), B.us_desc_preset(B.US_F_DCSR), B.us_desc_preset(B.US_F_CISR_PLUS, 3)]


def check(ctx, m, N, ldx, ldy, offset, rng, what):
    from paper_2403_05802_amd import binding as B
    length, row, col, val, ncols = m
    nrows = length.size
    X = rng.uniform(-1, 1, (ncols, N)).astype(np.float32)
    X[0] = np.inf
    xmem = torch.full((offset + ncols * ldx,), float("nan"), device="cuda")
    Xd = xmem[offset:].view(ncols, ldx)[:, :N]
    Xd.copy_(H.dev(X))
    A = sp.csr_matrix((val.astype(np.float64), (row, col)), shape=(nrows, ncols))
    X64 = np.where(np.isinf(X), 0.0, X).astype(np.float64)
    ref, scale = A @ X64, abs(A) @ np.abs(X64)
    Y0 = rng.uniform(-1, 1, (nrows, ldy)).astype(np.float32)
    for desc in descs():
        g = B.us_convert(ctx, nrows, ncols, H.dev(row), H.dev(col), H.dev(val), desc)
        for add in (False, True):
            ymem = torch.full((offset + nrows * ldy + 64,), 7.0, device="cuda")
            whole = ymem[offset:offset + nrows * ldy].view(nrows, ldy)
            whole.copy_(H.dev(Y0))
            B.us_spmm(ctx, g, Xd, whole[:, :N], accumulate=add)
            got = H.host(whole)
            r, s = (ref + Y0[:, :N], scale + np.abs(Y0[:, :N])) if add else (ref, scale)
            H.assert_product(got[:, :N], r, s, H.row_terms(nrows, row, int(add))[:, None], f"{what} trim {desc.trim_s} add {add}")
            assert np.array_equal(got[:, N:], Y0[:, N:])                              # the caller's columns
            assert (H.host(ymem[offset + nrows * ldy:]) == 7.0).all()
            whole.copy_(H.dev(Y0))
            B.us_spmm(ctx, g, Xd, whole[:, :N], accumulate=add)                       # bit for bit the same again
            assert np.array_equal(H.host(whole).view(np.int32), got.view(np.int32))
        g.free()


@pytest.mark.parametrize("pattern", list(PATTERNS))
@pytest.mark.parametrize("N,ldx,ldy,offset", [(1, 1, 1, 0), (33, 33, 36, 0), (64, 64, 64, 0), (130, 131, 130, 1)])
def test_rows_around_groups_wavefronts_and_tiles(ctx, pattern, N, ldx, ldy, offset):
    rng = np.random.default_rng(len(pattern) * 1000 + N)
    check(ctx, matrix(pattern, rng), N, ldx, ldy, offset, rng, f"{pattern} N={N}")


# (a list this short: panels of 64 columns, the last one with what is left)
@pytest.mark.parametrize("N,ldx", [(15, 15), (16, 16), (17, 17), (18, 20), (31, 31), (32, 32), (33, 64), (63, 63), (65, 65), (66, 96),
                                   (127, 127), (128, 128), (129, 129), (131, 160), (191, 192), (193, 193), (255, 255), (256, 256),
                                   (257, 257), (258, 260), (321, 321), (384, 385), (515, 515)])
def test_columns_around_every_panel_shape(ctx, N, ldx):
    rng = np.random.default_rng(N)
    check(ctx, matrix("long rows cut anywhere", rng), N, ldx, N + (N & 1), 0, rng, f"N={N}")


def spread(rows, rng, ncols=6000):
    """an entry in every row of the (ascending) list, columns distinct within a row"""
    row = np.asarray(rows)
    first = np.searchsorted(row, row)
    start = rng.integers(0, ncols - 1, row.size)[first]
    col = (1 + (start + np.arange(row.size) - first) % (ncols - 1)).astype(np.int32)
    return np.zeros(int(row.max()) + 1, dtype=np.int32), row.astype(np.int32), col, rng.uniform(-1, 1, row.size).astype(np.float32), ncols


def blocks_of_rows(rows, per_row, gap):
    """a third of the rows, `gap` empty ones, another third, ..."""
    r = np.arange(rows)
    return (r + r // (rows // 3 + 1) * gap).repeat(per_row)


# the parents between the first and the last entry of a tile are walked up to 4096 of them, beyond that every entry looks for its own
@pytest.mark.parametrize("last", [4094, 4095, 4096, 4097, 4098, 513 * 512, 100_000])
def test_few_entries_around_the_longest_walk(ctx, last):
    rng = np.random.default_rng(last)
    check(ctx, spread([0, last], rng), 1, 1, 1, 0, rng, f"rows 0 and {last}")
    inner = np.sort(rng.integers(0, last + 1, 700))
    check(ctx, spread(np.concatenate([[0, 0], inner, [last]]), rng), 17, 17, 17, 0, rng, f"700 entries of {last + 1} rows")


@pytest.mark.parametrize("rows,per_row,gap,N", [(25_000, 6, 30_000, 3), (25_000, 6, 30_000, 100), (25_000, 6, 30_000, 130), (30_000, 18, 5_000, 1), (60_000, 18, 5_000, 1),
                                                (6_000, 90, 4_500, 300)])
def test_gaps_inside_tiles_of_long_lists(ctx, rows, per_row, gap, N):
    rng = np.random.default_rng(rows + N)
    check(ctx, spread(blocks_of_rows(rows, per_row, gap), rng), N, N, N, 0, rng, f"{rows} rows of {per_row}, gaps of {gap}, N={N}")


# long lists, 1055 tiles: whole lines (rows of X begin at multiples of 32 floats) in panels of 64 columns, others in one of 128 or
# of 256 and more of these; a rest in the panel that fits it
@pytest.mark.parametrize("N,ldx", [(64, 64), (70, 96), (95, 96), (130, 160), (65, 65), (200, 200), (256, 257), (272, 272), (288, 290), (301, 301),
                                   (350, 350), (450, 450)])
def test_columns_of_long_lists(ctx, N, ldx):
    rng = np.random.default_rng(N)
    check(ctx, spread(np.arange(6000).repeat(90), rng), N, ldx, N, 0, rng, f"long list N={N}")


# tiles * panels on both sides of what is resident at once (512), half, twice and four times as much
@pytest.mark.parametrize("entries,N", [(512 * 256, 100), (512 * 256 + 1, 100), (512 * 51, 300), (512 * 51 + 1, 300), (512 * 204, 300), (512 * 205, 300),
                                       (512 * 512, 300), (512 * 512 + 1, 300), (512 * 1024, 30), (512 * 1024 + 1, 30), (512 * 2048, 5), (512 * 2048 + 1, 5)])
def test_lists_around_the_short_ones(ctx, entries, N):
    rng = np.random.default_rng(entries)
    check(ctx, spread(np.sort(rng.integers(0, 20_000, entries)), rng), N, N, N, 0, rng, f"{entries} entries N={N}")


@pytest.mark.parametrize("entries,N", [(500, 1), (500, 300), (20_000, 64), (50_000, 200), (50_000, 300), (150_000, 1), (150_000, 300)])
def test_short_lists_take_one_launch_and_the_fixup(entries, N):
    from paper_2403_05802_amd import binding as B
    rng = np.random.default_rng(entries)
    profiled = B.Context("cuda:0", profile=True)
    _, row, col, val, ncols = spread(np.concatenate([np.sort(rng.integers(0, 8000, entries - 1)), [7999]]), rng)
    X, Y = torch.ones((ncols, N), device="cuda"), torch.zeros((8000, N), device="cuda")
    for desc, name in zip(descs()[:2], ("spmm_csr", "spmm_coo")):
        g = B.us_convert(profiled, 8000, ncols, H.dev(row), H.dev(col), H.dev(val), desc)
        torch.cuda.synchronize()
        profiled.profile_reset()
        B.us_spmm(profiled, g, X, Y, accumulate=True)
        assert {k["kernel"]: k["launches"] for k in profiled.profile_report()} == {name: 1, "spmm_rows_fixup": 1}
        g.free()


@pytest.mark.parametrize("where", ["strays", "at both ends"])
def test_few_entries_in_ten_million_rows(ctx, where):
    from paper_2403_05802_amd import binding as B
    rng = np.random.default_rng(3)
    nrows = 10_000_000
    rows = np.sort(rng.integers(0, nrows, 1000)) if where == "strays" else np.concatenate([np.arange(300), np.arange(nrows - 300, nrows)]).repeat(3)
    _, row, col, val, ncols = spread(rows, rng)
    X = rng.uniform(-1, 1, (ncols, 2)).astype(np.float32)
    g = B.us_convert(ctx, nrows, ncols, H.dev(row), H.dev(col), H.dev(val), B.us_desc_preset(B.US_F_CSR))
    Xd, Y = H.dev(X), torch.full((nrows, 2), 3.0, device="cuda")
    B.us_spmm(ctx, g, Xd, Y, accumulate=True)
    used = np.unique(row)
    A = sp.csr_matrix((val.astype(np.float64), (np.searchsorted(used, row), col)), shape=(used.size, ncols))
    X64 = X.astype(np.float64)
    H.assert_product(H.host(Y[H.dev(used).long()]), A @ X64 + 3.0, abs(A) @ np.abs(X64) + 3.0, H.row_terms(used.size, np.searchsorted(used, row), 1)[:, None], where)
    assert int((Y != 3.0).any(1).sum()) <= used.size
    # the time does not depend on the rows without entries: some 20 us (8,500 where a workgroup walked them)
    best, a, b = float("inf"), torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    for _ in range(5):
        a.record()
        B.us_spmm(ctx, g, Xd, Y, accumulate=True)
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b))
    assert best < 1.0, f"{best} ms"
    g.free()


def test_operands_of_more_than_4_gb(ctx):
    rng = np.random.default_rng(9)
    length = np.full(700, 3)
    length[::5] = 0
    row = np.repeat(np.arange(700), length).astype(np.int32)
    col = np.concatenate([1 + rng.choice(699, k, replace=False) for k in length]).astype(np.int32)
    m = length, row, col, rng.uniform(-1, 1, row.size).astype(np.float32), 700
    from paper_2403_05802_amd import binding as B
    N, ld = 150, 1 << 21                                 # 700 rows, 8 MB apart
    X = rng.uniform(-1, 1, (700, N)).astype(np.float32)
    A = sp.csr_matrix((m[3].astype(np.float64), (row, col)), shape=(700, 700))
    Xd, Yd = torch.empty((700, ld), device="cuda")[:, :N], torch.empty((700, ld), device="cuda")[:, :N]
    Xd.copy_(H.dev(X))
    for desc in descs()[:2]:
        g = B.us_convert(ctx, 700, 700, H.dev(row), H.dev(col), H.dev(m[3]), desc)
        Yd.fill_(3.0)
        B.us_spmm(ctx, g, Xd, Yd)
        H.assert_product(H.host(Yd.contiguous()), A @ X.astype(np.float64), abs(A) @ np.abs(X).astype(np.float64),
                         H.row_terms(700, row)[:, None], f"4 GB trim {desc.trim_s}")
        g.free()
