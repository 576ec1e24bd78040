"""SpMM over ELL: row counts around what a lane group, a wavefront and a workgroup take, slot counts around what a group takes at a
time, column counts around every panel shape and where the wide kernel takes over, strides and accumulation."""
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


def check(ctx, nrows, longest, N, ldx, ldy, seed):
    from paper_2403_05802_amd import binding as B
    rng = np.random.default_rng(seed)
    ncols = 300
    length = np.where(rng.random(nrows) < 0.3, 0, rng.integers(0, longest + 1, nrows))
    length[rng.integers(0, nrows)] = longest                                 # as many slots as asked for
    row = np.repeat(np.arange(nrows), length).astype(np.int32)
    col = np.concatenate([1 + rng.choice(ncols - 1, k, replace=False) for k in length]).astype(np.int32)
    val = rng.uniform(-1, 1, row.size).astype(np.float32)
    X = rng.uniform(-1, 1, (ncols, N)).astype(np.float32)
    X[0] = np.inf                                                            # no entry in column 0: pads must not read it
    Xd = torch.full((ncols, ldx), float("nan"), device="cuda")[:, :N]
    Xd.copy_(H.dev(X))
    A = sp.csr_matrix((val.astype(np.float64), (row, col)), shape=(nrows, ncols))
    X64 = np.where(np.isinf(X), 0.0, X).astype(np.float64)
    ref, scale = A @ X64, abs(A) @ np.abs(X64)
    Y0 = rng.uniform(-1, 1, (nrows, ldy)).astype(np.float32)
    g = B.us_convert(ctx, nrows, ncols, H.dev(row), H.dev(col), H.dev(val), B.us_desc_preset(B.US_F_ELL))
    for add in (False, True):
        memory = torch.full((nrows * ldy + 64,), 7.0, device="cuda")
        whole = memory[:nrows * ldy].view(nrows, ldy)
        whole.copy_(H.dev(Y0))
        B.us_spmm(ctx, g, Xd, whole[:, :N], accumulate=add)
        got = H.host(whole)
        r, s = (ref + Y0[:, :N], scale + np.abs(Y0[:, :N])) if add else (ref, scale)
        H.assert_product(got[:, :N], r, s, H.row_terms(nrows, row, int(add))[:, None], f"rows {nrows} slots {longest} N={N} add {add}")
        assert np.array_equal(got[:, N:], Y0[:, N:]) and (H.host(memory[nrows * ldy:]) == 7.0).all()
    g.free()


@pytest.mark.parametrize("nrows", [1, 3, 4, 5, 15, 16, 17, 63, 65, 511, 513])
@pytest.mark.parametrize("longest", [1, 3, 4, 5, 8, 33])
def test_rows_and_slots(ctx, nrows, longest):
    for N, ldx, ldy in ((5, 5, 7), (64, 64, 64), (130, 131, 130)):
        check(ctx, nrows, longest, N, ldx, ldy, nrows * 100 + longest)


@pytest.mark.parametrize("N,ldx", [(1, 1), (2, 3), (15, 15), (16, 16), (17, 17), (31, 31), (32, 32), (33, 40), (63, 63), (65, 65), (127, 127),
                                   (128, 128), (129, 129), (131, 131), (193, 193), (255, 255), (256, 256), (257, 257), (333, 333),
                                   (384, 384), (514, 516)])
@pytest.mark.parametrize("nrows", [70, 16_400])   # fewer and more than where the panels take over from 256 columns on
def test_columns_around_every_panel_shape(ctx, nrows, N, ldx):
    check(ctx, nrows, 9, N, ldx, N + (N & 1), N)


def test_operands_of_more_than_4_gb(ctx):
    check(ctx, 300, 5, 150, 1 << 22, 150, 3)                                 # 300 rows of X, 16 MB apart
