"""Numbers of the groups a query keeps, and pointers over more groups than there are entries: group counts around the tiles of
their kernels, few and all groups kept, entries in one group or spread."""
import numpy as np
import pytest
import torch

import helpers as H

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2403_05802_amd import binding as B
    return B.Context("cuda:0")


@pytest.mark.parametrize("nrows,ncols", [(1, 1), (1024, 1024), (1024, 1025), (1025, 1025), (1, 2049), (2049, 1), (3000, 1096), (3000, 1097),
                                         (3000, 1098), (5, 70_000)])
@pytest.mark.parametrize("kept", ["some", "all"])
def test_diagonals(ctx, nrows, ncols, kept):
    from paper_2403_05802_amd import binding as B
    rng = np.random.default_rng(nrows * 7 + ncols)
    offsets = np.arange(-(nrows - 1), ncols)
    size = np.minimum(nrows, ncols - offsets) - np.maximum(0, -offsets)
    if kept == "some":                                   # a few full ones, and one entry in each of many others
        full = np.unique(np.concatenate([offsets[:1], offsets[-1:], rng.choice(offsets, min(offsets.size, 6))]))
        rest = np.setdiff1d(offsets[::3], full)
        cut = (9, 10)
    else:                                                # an entry in every diagonal, and all that have one are kept
        full, rest, cut = offsets[:0], offsets, None
    i = [np.arange(max(0, -o), min(nrows, ncols - o)) for o in full] + [[max(0, -o)] for o in rest]
    d = [np.full(len(k), o) for k, o in zip(i, np.concatenate([full, rest]))]
    row, d = np.concatenate(i).astype(np.int64), np.concatenate(d).astype(np.int64)
    order = rng.permutation(row.size)
    row, d = row[order], d[order]
    val = rng.uniform(0.5, 1, row.size).astype(np.float32)
    lists = [H.dev(a.astype(np.int32)) for a in (row, row + d)] + [H.dev(val)]
    if cut:
        pred = B.make_predicate([B.expr(B.US_E_AFFINE, -1, 1)], B.US_P_SUM_GE_FRAC_OF_CAPACITY, *cut)
        a, b = B.us_decompose(ctx, nrows, ncols, *lists, B.us_desc_preset(B.US_F_DIA), B.us_desc_preset(B.US_F_COO), pred)
        keep = np.sort(np.concatenate([full, rest[size[rest + nrows - 1] == 1]]))
    else:
        a, b, keep = B.us_convert(ctx, nrows, ncols, *lists, B.us_desc_preset(B.US_F_DIA)), None, offsets
    assert np.array_equal(H.host(a.idx(0)), keep)
    slab = np.zeros((keep.size, nrows), np.float32)
    at = np.searchsorted(keep, d)
    inside = (at < keep.size) & (keep[np.minimum(at, keep.size - 1)] == d)
    slab[at[inside], row[inside]] = val[inside]
    assert np.array_equal(H.host(a.val()).reshape(slab.shape), slab)
    if b is not None:
        left = np.lexsort((row + d, row))
        left = left[~inside[left]]
        assert np.array_equal(H.host(b.idx(0)), row[left]) and np.array_equal(H.host(b.val()), val[left])


@pytest.mark.parametrize("nrows,n", [(1, 0), (2046, 5), (2047, 2046), (2048, 300), (2049, 1), (70_001, 5_000), (70_001, 70_000),
                                     (524_287, 5_000), (524_288, 5_000), (526_335, 80_000), (526_336, 300), (526_337, 1), (1_000_003, 40_000)])
@pytest.mark.parametrize("where", ["spread", "first row", "last row", "crowded"])
def test_pointers_over_more_rows_than_entries(ctx, nrows, n, where):
    from paper_2403_05802_amd import binding as B
    rng = np.random.default_rng(n)
    ncols = 80_000
    row = {"spread": rng.integers(0, nrows, n), "first row": np.zeros(n, np.int64), "last row": np.full(n, nrows - 1),
           "crowded": nrows // 2 + rng.integers(0, min(nrows, 3), n) * (nrows > 6)}[where]
    key = np.unique(row * ncols + rng.permutation(ncols)[:n])
    row, col = key // ncols, key % ncols
    order = rng.permutation(row.size)
    val = rng.uniform(0.5, 1, row.size).astype(np.float32)
    g = B.us_convert(ctx, nrows, ncols, H.dev(row[order].astype(np.int32)), H.dev(col[order].astype(np.int32)), H.dev(val[order]),
                     B.us_desc_preset(B.US_F_CSR))
    assert np.array_equal(H.host(g.ptr(1)), np.searchsorted(row, np.arange(nrows + 1)))
    assert np.array_equal(H.host(g.idx(1)), col) and np.array_equal(H.host(g.val()), val)


@pytest.mark.parametrize("nrows,n,name", [(3_000, 300, "ptr_lower_bound"), (100_000, 70_000, "ptr_lower_bound"), (400_000, 40_000, "ptr_lower_bound"),
                                          (700_000, 70_000, "ptr_sparse")])
def test_rows_are_searched_a_tile_at_a_time_only_where_there_are_many(nrows, n, name):
    from paper_2403_05802_amd import binding as B
    rng = np.random.default_rng(n)
    profiled = B.Context("cuda:0", profile=True)
    row = rng.permutation(nrows)[:n].astype(np.int32)
    g = B.us_convert(profiled, nrows, 1000, H.dev(row), H.dev(row % 1000), torch.ones(n, device="cuda"), B.us_desc_preset(B.US_F_CSR))
    assert [k["kernel"] for k in profiled.profile_report() if k["kernel"].startswith("ptr_")] == [name]
    assert np.array_equal(H.host(g.ptr(1)), np.searchsorted(np.sort(row), np.arange(nrows + 1)))
    g.free()
