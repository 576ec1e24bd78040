"""SpMV over ELL with few rows, several wavefronts for the same rows, against the fp64 reference: the edges of the row
groups, of the slot groups of each wavefront and of the rule; rows of very different lengths, empty ones; accumulation."""
import numpy as np
import pytest

import helpers as H
from oracle import unisparse_oracle as O

pytestmark = pytest.mark.gpu


# (rows, longest row): plain up to 8 slots and beyond 131,072 rows, 16 wavefronts up to 16,384 rows of 64 slots, else 4
@pytest.mark.parametrize("nr,longest", [(1, 9), (63, 8), (64, 9), (65, 16), (127, 17), (1000, 63), (1000, 64), (129, 65), (777, 200),
                                        (16384, 64), (16385, 64), (131072, 9), (131073, 9)])
def test_every_row(nr, longest):
    from paper_2403_05802_amd import binding as B
    ctx = B.Context("cuda:0")
    rng = np.random.default_rng(nr + longest)
    nc = 5003
    length = np.minimum(rng.geometric(0.2, nr) - 1, longest)
    length[rng.integers(0, nr)] = longest
    row = np.repeat(np.arange(nr), length)
    lin = np.unique(row * nc + rng.integers(0, nc, row.size))
    lin = rng.permutation(np.union1d(lin, int(np.argmax(length)) * nc + np.arange(longest)))   # one row of `longest` for certain
    r, c = (lin // nc).astype(np.int32), (lin % nc).astype(np.int32)
    keep = np.zeros(r.size, bool)                     # at most `longest` a row
    order = np.argsort(r, kind="stable")
    rank = np.arange(r.size) - np.searchsorted(r[order], r[order])
    keep[order] = rank < longest
    r, c = r[keep], c[keep]
    v = rng.uniform(-1, 1, r.size).astype(np.float32)
    x, y0 = rng.uniform(-1, 1, nc).astype(np.float32), rng.uniform(-1, 1, nr).astype(np.float32)
    g = B.us_convert(ctx, nr, nc, H.dev(r), H.dev(c), H.dev(v), H.us_desc_of(O.ELL()))
    assert g.size(0) == longest
    terms = v.astype(np.float64) * x[c]
    for acc in (False, True):
        ref = np.bincount(r, terms, nr) + (y0 if acc else 0.0)
        scale = np.bincount(r, np.abs(terms), nr) + (np.abs(y0) if acc else 0.0)
        y = H.dev(y0.copy())
        B.us_spmv(ctx, g, H.dev(x), y, accumulate=acc)
        # n terms in any order: at most n roundings of the sum and one of each product, 2^-24 of the terms' total each
        bound = (np.bincount(r, minlength=nr) + 2) * 2.0 ** -24 * scale
        assert (np.abs(H.host(y).astype(np.float64) - ref) <= bound).all(), (acc, np.abs(H.host(y) - ref).max())
    g.free()
