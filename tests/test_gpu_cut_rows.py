"""SpMV over compressed rows where the workgroup that ends a row goes over the part of it that earlier workgroups hold: rows of
up to several tiles, column counts and tile counts on both sides of where that ends, empty rows, rows that end on a tile's edge,
accumulation."""
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


def check(ctx, length, ncols, seed):
    from paper_2403_05802_amd import binding as B
    rng = np.random.default_rng(seed)
    nrows = length.size
    row = np.repeat(np.arange(nrows), length).astype(np.int32)
    col = np.concatenate([np.sort(rng.choice(ncols, k, replace=False)) for k in length] or [[]]).astype(np.int32)
    val = rng.uniform(-1, 1, row.size).astype(np.float32)
    x, y0 = rng.uniform(-1, 1, ncols).astype(np.float32), rng.uniform(-1, 1, nrows).astype(np.float32)
    A = sp.csr_matrix((val.astype(np.float64), (row, col)), shape=(nrows, ncols))
    ref, scale = A @ x.astype(np.float64), abs(A) @ np.abs(x).astype(np.float64)
    for layout in (B.US_F_CSR, B.US_F_DCSR):
        g = B.us_convert(ctx, nrows, ncols, H.dev(row), H.dev(col), H.dev(val), B.us_desc_preset(layout))
        for add in (False, True):
            memory = torch.full((nrows + 64,), 7.0, device="cuda")
            memory[:nrows] = H.dev(y0)
            B.us_spmv(ctx, g, H.dev(x), memory[:nrows], accumulate=add)
            got = H.host(memory)
            r, s = (ref + y0, scale + np.abs(y0)) if add else (ref, scale)
            H.assert_product(got[:nrows], r, s, H.row_terms(nrows, row, int(add)), f"{nrows} x {ncols}, {row.size} entries, add {add}")
            assert (got[nrows:] == 7.0).all()
        g.free()


@pytest.mark.parametrize("ncols", [4096, 8191, 8192, 8193])
def test_rows_of_several_tiles(ctx, ncols):
    rng = np.random.default_rng(ncols)
    n = rng.integers(0, 9, 700)
    n[::50] = ncols                     # as long as a row can be
    n[7::90] = rng.integers(1500, 4096, n[7::90].size)
    check(ctx, n, ncols, 1)
    check(ctx, np.full(3, ncols), ncols, 2)


@pytest.mark.parametrize("first", [2045, 2046, 2047, 2048, 2049, 4094, 4095, 4096])
def test_rows_that_end_at_a_tile(ctx, first):
    check(ctx, np.array([first, 0, 0, 1, 2047, 5, 0, 2048, 1, 0]), 5000, first)


def test_short_rows(ctx):
    for nrows in (1, 2, 2047, 2048, 2049, 30_000):
        check(ctx, np.random.default_rng(nrows).integers(0, 3, nrows), 300, nrows)


# rows of `length` entries are length + 1 steps each: 128 rows of 4095 are 256 tiles of 2048 steps
@pytest.mark.parametrize("ncols,length,nrows,launches", [
    (8192, 4095, 128, 1), (8192, 4095, 129, 2),       # tiles * columns on both sides of 2 M
    (4096, 4095, 256, 1), (4096, 4095, 257, 2),
    (2048, 2047, 1024, 1), (2048, 2047, 1025, 2),     # 1024 tiles, and one more
    (100, 63, 32768, 1), (100, 63, 32800, 2)])
def test_one_launch_only_where_little_is_read_again(ctx, ncols, length, nrows, launches):
    from paper_2403_05802_amd import binding as B
    rng = np.random.default_rng(length)
    start, step = rng.integers(0, ncols, nrows), 1 + 2 * rng.integers(0, ncols // 2, nrows) if ncols & (ncols - 1) == 0 else np.ones(nrows, int)
    col = ((start[:, None] + np.arange(length) * step[:, None]) % ncols).ravel().astype(np.int32)   # distinct within a row
    row = np.repeat(np.arange(nrows), length).astype(np.int32)
    val, x = rng.uniform(-1, 1, row.size).astype(np.float32), rng.uniform(-1, 1, ncols).astype(np.float32)
    A = sp.csr_matrix((val.astype(np.float64), (row, col)), shape=(nrows, ncols))
    profiled = B.Context("cuda:0", profile=True)
    g = B.us_convert(profiled, nrows, ncols, H.dev(row), H.dev(col), H.dev(val), B.us_desc_preset(B.US_F_CSR))
    y = torch.full((nrows,), 7.0, device="cuda")
    torch.cuda.synchronize()
    profiled.profile_reset()
    B.us_spmv(profiled, g, H.dev(x), y)
    H.assert_product(H.host(y), A @ x.astype(np.float64), abs(A) @ np.abs(x).astype(np.float64), H.row_terms(nrows, row), f"{nrows} x {ncols}")
    assert sum(k["launches"] for k in profiled.profile_report()) == launches
    g.free()
