"""The DIA slab put together bin by bin (lists in random order, slabs beyond the caches) against plain indexing: both
slab orders, the edges of the bins and of the rule, an empty-slot pattern among the values, duplicates, a remainder."""
import numpy as np
import pytest

from oracle import unisparse_oracle as O

pytestmark = pytest.mark.gpu
OFFSETS = (-700, -1, 0, 1, 64, 2048, 30_000)


@pytest.fixture(scope="module")
def ctx():
    from paper_2403_05802_amd import binding as B
    return B.Context("cuda:0")


def banded(nr, nc, seed, extra=0):
    """Every slot of the diagonals inside the matrix and `extra` entries elsewhere, in random order, on the GPU."""
    import torch
    g = torch.Generator(device="cuda"); g.manual_seed(seed)
    i = torch.arange(nr, device="cuda")
    lin = torch.cat([(i * nc + i + o)[(i + o >= 0) & (i + o < nc)] for o in OFFSETS])
    if extra:
        e = torch.randint(0, nr * nc, (extra,), generator=g, device="cuda")
        off = torch.remainder(e, nc) - torch.div(e, nc, rounding_mode="floor")
        lin = torch.cat([lin, e[~torch.isin(off, torch.tensor(OFFSETS, device="cuda"))].unique()])
    lin = lin[torch.randperm(lin.numel(), generator=g, device="cuda")]
    r = torch.div(lin, nc, rounding_mode="floor")
    v = torch.rand(lin.numel(), generator=g, device="cuda") + 0.5
    return r.int(), (lin - r * nc).int(), v


def slab(nr, nc, r, c, v, by_col):
    import torch
    L = nc if by_col else nr
    out = torch.zeros(len(OFFSETS), L, device="cuda")
    for k, o in enumerate(OFFSETS):
        on = c - r == o
        out[k, (c if by_col else r)[on].long()] = v[on]
    return out.flatten()


def launches(ctx, call):
    ctx.enable_profile(); ctx.profile_reset()
    try:
        out = call()
        return out, {e["kernel"] for e in ctx.profile_report()}
    finally:
        ctx.disable_profile()


# rows so that 7 slabs end just below the rule, just on it, inside a bin, on the edge of one; rectangular; bins of 32,768
@pytest.mark.parametrize("nr,nc", [(224_694, 224_694), (224_695, 224_695), (300_007, 250_001), (16384 * 16, 16384 * 17), (4_793_491, 4_793_491)])
def test_slab_equals_plain_indexing(ctx, nr, nc):
    import torch
    from paper_2403_05802_amd import binding as B
    from helpers import us_desc_of
    r, c, v = banded(nr, nc, nr)
    v[v.numel() // 2] = torch.tensor(0x7FC5A5A5, dtype=torch.int32).view(torch.float32).item()   # the pattern of an empty slot
    bits = v.view(torch.int32)
    bits[v.numel() // 2] = 0x7FC5A5A5
    for desc, by_col in ((O.DIA(), False), (O.DIA_VARIANT(), True)):
        g, names = launches(ctx, lambda: B.us_convert(ctx, nr, nc, r, c, v, us_desc_of(desc)))
        slots = len(OFFSETS) * (nc if by_col else nr)
        assert ("dia_image" in names) == (slots >= 3 << 19), (names, slots)
        assert g.idx(0).tolist() == list(OFFSETS)
        assert torch.equal(g.val().view(torch.int32), slab(nr, nc, r, c, v, by_col).view(torch.int32))
        g.free()


def test_remainder_duplicates_and_sorted_lists(ctx):
    import torch
    from paper_2403_05802_amd import binding as B
    from helpers import us_desc_of
    nr = nc = 400_003
    r, c, v = banded(nr, nc, 5, extra=30_000)
    pred = B.make_predicate([B.expr(B.US_E_AFFINE, -1, 1)], B.US_P_SUM_GE_FRAC_OF_CAPACITY, 9, 10)
    call = lambda r, c, v: B.us_decompose(ctx, nr, nc, r, c, v, us_desc_of(O.DIA()), us_desc_of(O.COO()), pred)
    (a, b), names = launches(ctx, lambda: call(r, c, v))
    assert "dia_image" in names and "dia_split_scatter" not in names
    assert torch.equal(a.val(), slab(nr, nc, r, c, v, False))
    rest = ~torch.isin(c - r, torch.tensor(OFFSETS, device="cuda", dtype=torch.int32))
    order = torch.argsort(r[rest].long() * nc + c[rest])
    for got, want in ((b.idx(0), r), (b.idx(1), c), (b.val(), v)):
        assert torch.equal(got, want[rest][order])
    a.free(); b.free()
    # the same entries sorted by rows go straight into the slab
    order = torch.argsort(r.long() * nc + c)
    (a, b), names = launches(ctx, lambda: call(r[order].contiguous(), c[order].contiguous(), v[order].contiguous()))
    assert "dia_image" not in names and torch.equal(a.val(), slab(nr, nc, r, c, v, False))
    a.free(); b.free()
    # a second copy of an entry on a diagonal
    at = int(torch.nonzero(c - r == 64)[1000])
    r2, c2, v2 = (torch.cat([x, x[at:at + 1]]) for x in (r, c, v))
    p = torch.randperm(r2.numel(), device="cuda")
    with pytest.raises(B.UnisparseError) as ei:
        call(r2[p].contiguous(), c2[p].contiguous(), v2[p].contiguous())
    assert ei.value.code == "US_ERR_DUPLICATE"
