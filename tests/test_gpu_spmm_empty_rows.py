"""A plain SpMM over CSR stores the rows that hold entries and clears the others by a kernel of its own: which rows and
columns that kernel covers, how many rows it takes, and what it costs."""
import numpy as np
import pytest
import torch

from oracle import unisparse_oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2403_05802_amd import binding as B
    return B.Context("cuda:0")


def csr(ctx, n, nc, keys):
    """CSR of the entries at the sorted, distinct linear positions `keys`, on the GPU."""
    from paper_2403_05802_amd import binding as B
    r = torch.div(keys, nc, rounding_mode="floor")
    v = torch.rand(keys.numel(), device="cuda") + 0.5
    return B.us_convert(ctx, n, nc, r.int(), (keys - r * nc).int(), v, B.us_desc_preset(B.US_F_CSR))


# 64, 16 or 8 rows a wavefront (up to 32, 128 or more columns, words or loads of four), fewer where there are few wavefronts;
# pieces of 512 columns
@pytest.mark.parametrize("n", [1, 31, 65, 257, 700])
@pytest.mark.parametrize("N,ld_extra,offset", [(1, 0, 0), (3, 2, 0), (32, 0, 1), (33, 0, 0), (128, 4, 0), (129, 0, 0), (255, 1, 0),
                                               (511, 0, 0), (513, 0, 0), (132, 0, 0), (516, 0, 0), (2048, 0, 0), (2052, 8, 0)])
def test_rows_without_entries_are_cleared_and_nothing_else(ctx, n, N, ld_extra, offset):
    check_product(ctx, n, N, ld_extra, offset)


@pytest.mark.parametrize("n,N,ld_extra,offset", [
    (65_471, 1, 0, 0), (65_473, 1, 3, 0), (65_537, 3, 0, 0), (65_600, 31, 1, 1), (65_599, 32, 0, 0), (70_001, 128, 0, 0),
    (16_383, 33, 0, 0), (16_385, 127, 0, 0), (17_003, 132, 0, 0), (8_199, 129, 0, 0), (8_191, 515, 0, 0), (4_099, 520, 0, 0)])
def test_as_many_rows_as_fill_the_wavefronts(ctx, n, N, ld_extra, offset):
    check_product(ctx, n, N, ld_extra, offset)


def check_product(ctx, n, N, ld_extra, offset):
    from paper_2403_05802_amd import binding as B
    from helpers import assert_product, dev, host, row_terms
    rng = np.random.default_rng(n * 4096 + N)
    nc = 90
    length = np.where(rng.random(n) < 0.6, 0, rng.integers(1, 4, n))
    length[n // 4:n // 2] = 0
    length[n - 1] = 1                                       # at least one entry: an empty matrix takes another path
    r = np.repeat(np.arange(n), length).astype(np.int32)
    c = np.concatenate([rng.choice(nc, k, replace=False) for k in length]).astype(np.int32)
    v = rng.uniform(-1, 1, r.size).astype(np.float32)
    g = B.us_convert(ctx, n, nc, dev(r), dev(c), dev(v), B.us_desc_preset(B.US_F_CSR))
    X = rng.uniform(-1, 1, (nc, N)).astype(np.float32)
    ld = N + ld_extra
    memory = torch.full((offset + n * ld + 64,), float("nan"), device="cuda")
    whole = memory[offset:offset + n * ld].view(n, ld)
    B.us_spmm(ctx, g, dev(X), whole[:, :N])
    got = host(whole[:, :N].contiguous())
    assert_product(got, O.spmm_coo(n, nc, r, c, v, X), O.spmm_coo(n, nc, r, c, np.abs(v), np.abs(X)),
                   row_terms(n, r)[:, None], f"n={n} N={N} ld+{ld_extra}")
    assert (got[length == 0] == 0).all()
    assert torch.isnan(whole[:, N:]).all() and torch.isnan(memory[:offset]).all() and torch.isnan(memory[offset + n * ld:]).all()
    g.free()


def test_more_rows_than_threads_of_one_grid(ctx):
    """600 M rows, one column: a grid of a fixed number of threads per row would pass 2^32 threads."""
    from paper_2403_05802_amd import binding as B
    n, nc = 600_000_000, 64
    rows = torch.unique(torch.randint(0, n, (1000,), device="cuda"))
    rows[0], rows[-1] = 0, n - 1
    g = csr(ctx, n, nc, rows * nc + rows % nc)
    x = torch.rand(nc, 1, device="cuda") + 0.5
    y = torch.full((n, 1), float("nan"), device="cuda")
    B.us_spmm(ctx, g, x, y)
    want = g.val() * x[rows % nc, 0]                        # one entry a row: one product, no sum
    assert torch.equal(y[rows, 0], want)
    y[rows] = 0.0
    assert int(torch.count_nonzero(y)) == 0                 # NaN counts as nonzero
    g.free()


# results of more than 512 MB are written past the caches: words and loads of four, one piece of columns and several
@pytest.mark.parametrize("n,N", [(2_100_001, 61), (1_300_003, 100), (300_007, 513), (130_001, 1000), (1001, 131_076)])
def test_large_results(ctx, n, N):
    from paper_2403_05802_amd import binding as B
    nc = 100
    rows = torch.unique(torch.randint(0, n, (n // 3,), device="cuda"))
    rows[-1] = n - 1
    g = csr(ctx, n, nc, rows * nc + rows % nc)
    X = torch.rand(nc, N, device="cuda") + 0.5
    Y = torch.full((n, N), float("nan"), device="cuda")
    B.us_spmm(ctx, g, X, Y)
    for part in torch.arange(rows.numel(), device="cuda").split(100_000):   # one entry a row: one product, no sum
        assert torch.equal(Y[rows[part]], g.val()[part, None] * X[rows[part] % nc])
    Y[rows] = 0.0
    assert int(torch.count_nonzero(Y)) == 0
    g.free()


def best_us(f, calls=20, rounds=6):
    """Least time of a call among others, microseconds."""
    for _ in range(3):
        f()
    best = float("inf")
    for _ in range(rounds):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(calls):
            f()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / calls)
    return best


@pytest.mark.parametrize("n,nc,nnz,N", [(2_000_000, 2_000_000, 147_000, 1), (2_000_000, 2_000_000, 147_000, 4),
                                        (8, 1000, 3, 1_000_000), (200, 1000, 20, 100_000),
                                        (2_000_000, 2_000_000, 147_000, 100)])
def test_clearing_the_rows_costs_no_more_than_clearing_all(ctx, n, nc, nnz, N):
    """Mostly empty matrices: a plain product against clearing all of Y and adding to it, which writes as much and reads
    the stored rows besides.  (A quarter is left for what the two runs differ by; clearing row by row took 1.6 times as
    long at one column and 10 to 40 times with few rows.)"""
    from paper_2403_05802_amd import binding as B
    g = csr(ctx, n, nc, torch.unique(torch.randint(0, n * nc, (nnz,), device="cuda")))
    X, Y = torch.rand(nc, N, device="cuda"), torch.empty(n, N, device="cuda")

    def clear_and_add():
        Y.zero_()
        B.us_spmm(ctx, g, X, Y, accumulate=True)

    plain, both = best_us(lambda: B.us_spmm(ctx, g, X, Y)), best_us(clear_and_add)
    print(f"\n[n={n} N={N}: plain {plain:.1f} us, clear and add {both:.1f} us]")
    assert plain <= 1.25 * both
    g.free()
