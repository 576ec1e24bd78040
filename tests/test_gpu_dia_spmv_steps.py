"""SpMV over DIA with numbers of diagonals around what the kernels load together, row counts that are multiples of four and not,
diagonals that leave the matrix at either end, and a remainder of a few entries added on top."""
import numpy as np
import pytest
import scipy.sparse as sp

import helpers as H

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2403_05802_amd import binding as B
    return B.Context("cuda:0")


@pytest.mark.parametrize("ndiag", [1, 2, 3, 4, 5, 6, 7, 8, 9, 13, 14, 16, 17, 18])
@pytest.mark.parametrize("nrows,ncols", [(1, 1), (3, 9), (8, 8), (256, 250), (1021, 1030), (1024, 1024), (4096, 300)])
def test_diagonals(ctx, nrows, ncols, ndiag):
    from paper_2403_05802_amd import binding as B
    rng = np.random.default_rng(ndiag * 31 + nrows)
    every = np.arange(-(nrows - 1), ncols)
    offsets = np.unique(np.concatenate([every[:1], every[-1:], rng.choice(every, min(ndiag, every.size), replace=False)]))[-ndiag:]
    row = np.concatenate([np.arange(max(0, -o), min(nrows, ncols - o)) for o in offsets])
    col = np.concatenate([np.arange(max(0, -o), min(nrows, ncols - o)) + o for o in offsets])
    val = rng.uniform(0.1, 1, row.size).astype(np.float32)
    extra = np.setdiff1d(rng.integers(0, nrows * ncols, 5), row.astype(np.int64) * ncols + col)   # a remainder of a few rows
    x, y0 = rng.uniform(-1, 1, ncols).astype(np.float32), rng.uniform(-1, 1, nrows).astype(np.float32)
    lists = lambda r, c, v: [H.dev(r.astype(np.int32)), H.dev(c.astype(np.int32)), H.dev(v)]
    main = sp.csr_matrix((val.astype(np.float64), (row, col)), shape=(nrows, ncols))
    for layout in (B.US_F_DIA, B.US_F_DIA_VARIANT):
        g = B.us_convert(ctx, nrows, ncols, *lists(row, col, val), B.us_desc_preset(layout))
        for add in (False, True):
            y = H.dev(y0.copy())
            B.us_spmv(ctx, g, H.dev(x), y, accumulate=add)
            ref, scale = main @ x.astype(np.float64), abs(main) @ np.abs(x).astype(np.float64)
            if add:
                ref, scale = ref + y0, scale + np.abs(y0)
            H.assert_product(H.host(y), ref, scale, H.row_terms(nrows, row, int(add)), f"{nrows} x {ncols}, {ndiag} diagonals, add {add}")
        g.free()
    v = rng.uniform(0.1, 1, extra.size).astype(np.float32)
    for layout in (B.US_F_CSR, B.US_F_DCSR):
        g = B.us_convert(ctx, nrows, ncols, *lists(extra // ncols, extra % ncols, v), B.us_desc_preset(layout))
        y = H.dev(y0.copy())
        B.us_spmv(ctx, g, H.dev(x), y, accumulate=True)
        rest = sp.csr_matrix((v.astype(np.float64), (extra // ncols, extra % ncols)), shape=(nrows, ncols))
        H.assert_product(H.host(y), y0 + rest @ x.astype(np.float64), np.abs(y0) + abs(rest) @ np.abs(x).astype(np.float64),
                         H.row_terms(nrows, extra // ncols, 1), f"{nrows} x {ncols}, {extra.size} entries added")
        g.free()
