"""The rank split of a decomposition: row counts around the tiles of its kernels, lists whose second part is one long row, one
entry in each of a few of very many rows, or empty, lengths of more than one digit of the percentile, and parts that are
lists as well as an ELL slab."""
import numpy as np
import pytest

import helpers as H

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2403_05802_amd import binding as B
    return B.Context("cuda:0")


def lengths(kind, nrows, ncols, rng):
    if kind == "mixed":
        n = np.where(rng.random(nrows) < 0.3, 0, rng.integers(0, min(ncols, 12) + 1, nrows))
    elif kind == "one row":       # holds all there is
        n = np.zeros(nrows, np.int64)
        n[rng.integers(0, nrows)] = min(ncols, 70_000)
    elif kind == "few beyond":    # one entry more than the others in a few rows
        n = np.full(nrows, 2)
        n[rng.choice(nrows, min(nrows, 5), replace=False)] = 3
    else:                         # "long": lengths that share their upper digits and others that do not
        n = rng.integers(0, 3, nrows)
        n[rng.choice(nrows, min(nrows, 40), replace=False)] = rng.integers(2040, 4200, min(nrows, 40))
    return np.minimum(n, ncols)


def check(ctx, kind, nrows, ncols, cut, first, seed):
    from paper_2403_05802_amd import binding as B
    rng = np.random.default_rng(seed)
    n = lengths(kind, nrows, ncols, rng)
    row = np.repeat(np.arange(nrows, dtype=np.int64), n)
    rank = np.arange(row.size) - np.repeat(np.cumsum(n) - n, n)
    # ascending distinct columns of a row: its entries evenly spaced, moved by a random number smaller than the space
    space = np.maximum(ncols // np.maximum(n, 1), 1)[row]
    col = rank * space + (rng.random(row.size) * space).astype(np.int64)
    val = rng.uniform(-1, 1, row.size).astype(np.float32)
    if isinstance(cut, tuple):
        pred = B.make_predicate([B.expr(B.US_E_AFFINE, 1, 0)], B.US_P_RANK_LT_PERCENTILE, *cut)
        K = int(np.sort(n)[max(0, -(-cut[0] * nrows // cut[1]) - 1)])
    else:
        pred = B.make_predicate([B.expr(B.US_E_AFFINE, 1, 0)], B.US_P_RANK_LT_ABS, abs_=cut)
        K = cut
    if min(K, int(n.max())) * nrows >= 1 << 26:   # too wide a slab
        first = B.US_F_CSR
    order = rng.permutation(row.size)
    what = f"{kind}, {nrows} x {ncols}, {row.size} entries, cut {cut}, first {first}"
    print(what, flush=True)
    a, b = B.us_decompose(ctx, nrows, ncols, H.dev(row[order].astype(np.int32)), H.dev(col[order].astype(np.int32)),
                          H.dev(val[order]), B.us_desc_preset(first), B.us_desc_preset(B.US_F_COO), pred)
    below = rank < K
    for k, expected in ((0, row), (1, col)):
        assert np.array_equal(H.host(b.idx(k)), expected[~below]), what
    assert np.array_equal(H.host(b.val()), val[~below]), what
    assert (a.nnz, b.nnz) == (below.sum(), (~below).sum()), what
    if first == B.US_F_ELL:
        width = int(min(K, n.max()))
        c, v = np.full((width, nrows), -1, np.int32), np.zeros((width, nrows), np.float32)
        c[rank[below], row[below]], v[rank[below], row[below]] = col[below], val[below]
        assert np.array_equal(H.host(a.idx(2)).reshape(width, nrows), c) and np.array_equal(H.host(a.val()).reshape(width, nrows), v), what
    else:
        assert np.array_equal(H.host(a.ptr(1)), np.concatenate([[0], np.cumsum(np.minimum(n, K))])), what
        assert np.array_equal(H.host(a.idx(1)), col[below]) and np.array_equal(H.host(a.val()), val[below]), what
    a.free(); b.free()


@pytest.mark.parametrize("kind", ["mixed", "one row", "few beyond", "long"])
@pytest.mark.parametrize("nrows", [1, 7, 255, 257, 2047, 2048, 2049, 4095, 4096, 4097, 65_537, 1_050_001])
def test_rows_and_lengths(ctx, kind, nrows):
    from paper_2403_05802_amd import binding as B
    ncols = 8_000 if kind != "one row" else 100_000
    for cut in (0, 2, (9, 10), (1, 1)):
        check(ctx, kind, nrows, ncols, cut, B.US_F_ELL, nrows)


@pytest.mark.parametrize("cut", [0, 1, 5, 1 << 40, (0, 1), (1, 2), (999, 1000)])
def test_cuts(ctx, cut):
    from paper_2403_05802_amd import binding as B
    for kind in ("mixed", "long", "few beyond"):
        for first in (B.US_F_ELL, B.US_F_CSR):
            check(ctx, kind, 5_000, 5_000_000, cut, first, 11)   # lengths of three digits


def test_one_column(ctx):
    from paper_2403_05802_amd import binding as B
    for kind in ("mixed", "few beyond"):
        check(ctx, kind, 3, 1, (1, 2), B.US_F_ELL, 0)
