"""The work that users of this library have it do, as timed cases.

A case is one pass through the public entry points of `paper_2403_05802_amd.binding`: a conversion of an unsorted COO
list, a decomposition into a hybrid, a conversion from one layout to another, or a product over a resident matrix.
The matrices have the structure of the configurations in `workloads.py` (uniform, power-law rows, power-law rows with
local columns, few diagonals, dense 4x4 blocks in a band) but are drawn on the GPU, so that new inputs cost little.

`listed()` names the cases, `draw(rng)` gives another one from the same ranges.  `prepare` makes what a program has in
hand (the COO list, or the resident layout and its dense operand), `run` is the pass, `work` the bytes and operations
it cannot do without, `tolerance` how far another correct implementation may be off.
"""
import functools
import math

import numpy as np
import torch

from paper_2403_05802_amd import binding as B

DEVICE = "cuda:0"
MAX_ROW = 20000                                    # longest row of the power-law matrices
OFFSETS = (-2048, -1024, -1, 0, 1, 1024, 2048)     # diagonals of the banded matrices
EXTRA = 0.01                                       # scattered entries beside them
BLOCKS_PER_ROW, BAND_BLOCKS = 24, 1024             # blocked band matrices: 4x4 blocks per block row, half width of the band
WINDOW, LOCAL = 512, 0.7                           # local columns: half width and share


def listed():
    return [
        # the smallest calls, where latency counts: one product / one conversion of a 41 k entry matrix (configuration 1)
        dict(name="spmv csr small", op="spmv", matrix="uniform", n=4096, nnz=40960, layout="csr"),
        dict(name="convert csr small", op="convert", matrix="uniform", n=4096, nnz=40960, layout="csr"),
        # the ordinary conversion and product: a power-law graph to CSR, SpMV over it (configuration 2)
        dict(name="convert csr power-law", op="convert", matrix="powerlaw", n=1 << 20, nnz=1 << 24, layout="csr"),
        dict(name="spmv csr power-law", op="spmv", matrix="powerlaw", n=1 << 20, nnz=1 << 24, layout="csr"),
        # a stencil-like matrix split into full diagonals and a remainder (configuration 3), and SpMV over such a hybrid
        # at an odd size
        dict(name="decompose dia+csr", op="decompose", matrix="banded", n=1 << 21, nnz=7 << 21, layout="dia+csr"),
        dict(name="spmv dia+csr odd", op="spmv", matrix="banded", n=777_777, nnz=7 * 777_777, layout="dia+csr"),
        # a FEM-like matrix to 4x4 blocks and SpMM over them (configuration 4)
        dict(name="convert bcsr", op="convert", matrix="blockfem", n=1 << 19, nnz=24 * 4 << 19, layout="bcsr"),
        dict(name="spmm bcsr 64", op="spmm", matrix="blockfem", n=1 << 19, nnz=24 * 4 << 19, layout="bcsr", cols=64),
        # the largest: a graph of 40 M entries split into ELL + COO, SpMM with 128 features over the hybrid (configuration 5)
        dict(name="decompose ell+coo", op="decompose", matrix="local", n=2_000_000, nnz=40_000_000, layout="ell+coo"),
        dict(name="spmm ell+coo 128", op="spmm", matrix="local", n=2_000_000, nnz=40_000_000, layout="ell+coo", cols=128),
        # from layout to layout (the transpose of a resident matrix) at a ragged middle size
        dict(name="csr to csc ragged", op="reconvert", matrix="powerlaw", n=200_003, nnz=3_100_007, layout="csr>csc"),
        # one step of label propagation with as many labels as the benchmark uses
        dict(name="spmm csr 1000", op="spmm", matrix="local", n=1 << 18, nnz=5_200_000, layout="csr", cols=1000),
    ]


def draw(rng):
    """One more case: any of the paths above, 41 k to 40 M entries, rows of 4 to 64 entries on average, 1 to 1000 columns."""
    op, matrix, layout = rng.choice([
        ("convert", "uniform", "csr"), ("convert", "powerlaw", "csr"), ("convert", "powerlaw", "dcsr"),
        ("convert", "local", "csc"), ("convert", "blockfem", "bcsr"),
        ("decompose", "banded", "dia+csr"), ("decompose", "local", "ell+coo"),
        ("reconvert", "powerlaw", "csr>csc"), ("reconvert", "blockfem", "dcsc>bcsr"),
        ("spmv", "uniform", "csr"), ("spmv", "powerlaw", "csr"), ("spmv", "banded", "dia+csr"), ("spmv", "local", "ell+coo"),
        ("spmm", "blockfem", "bcsr"), ("spmm", "local", "csr"), ("spmm", "local", "ell+coo"), ("spmm", "banded", "dia+csr"),
    ])

    def between(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    nnz = between(40_960, 40_000_000)
    if matrix == "banded":
        n = max(8192, nnz // len(OFFSETS))
        nnz = n * len(OFFSETS)
    elif matrix == "blockfem":
        n = 4 * max(64, nnz // (16 * BLOCKS_PER_ROW))
        nnz = n * 4 * BLOCKS_PER_ROW
    else:
        n = max(2048, int(nnz / math.exp(rng.uniform(math.log(4), math.log(64)))))
    case = dict(op=op, matrix=matrix, n=n, nnz=nnz, layout=layout)
    if op == "spmm":
        most = min(1000, 5_000_000_000 // nnz, 250_000_000 // n)
        case["cols"] = between(1, most)
    return case


# ----------------------------------------------------------------------------- matrices
@functools.lru_cache(maxsize=16)
def _lengths(n, nnz, s):
    """Lengths of n rows, about nnz in all: floor(scale * z + u) clipped to [1, longest], z ~ Zipf(s) at equally spaced
    quantiles and u evenly spread."""
    longest = min(MAX_ROW, max(4, n // 4))
    k = np.arange(1, longest + 1, dtype=np.float64)
    p = k ** -s
    p /= p.sum()
    lo, hi = 0.0, 4.0 * nnz / n + 4.0
    for _ in range(60):
        c = 0.5 * (lo + hi)
        if float((p * np.clip(c * k, 1, longest)).sum()) * n < nnz:
            lo = c
        else:
            hi = c
    i = np.arange(n)
    z = np.minimum(np.searchsorted(np.cumsum(p), (i + 0.5) / n) + 1, longest)
    return np.clip(np.floor(hi * z + (i * 0.6180339887498949) % 1.0).astype(np.int64), 1, longest)


def _exponent(matrix):
    return 2.0 if matrix == "local" else 1.8


def _generator(seed, salt=0):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(int(seed) * 1_000_003 + salt)
    return g


def _uniform(shape, g):
    v = torch.rand(shape, generator=g, device=DEVICE).mul_(2.0).sub_(1.0)
    return torch.where(v == 0.0, torch.full_like(v, 0.5), v)


def _distinct(keys, redraw, bad=None):
    """Draws the repeats in `keys` (and what `bad` finds fault with) again until there are none."""
    while True:
        order = torch.sort(keys, stable=True)
        wrong = torch.zeros(keys.numel(), dtype=torch.bool, device=DEVICE)
        wrong[order.indices[1:]] = order.values[1:] == order.values[:-1]
        if bad is not None:
            wrong |= bad(keys)
        at = torch.nonzero(wrong).flatten()
        if at.numel() == 0:
            return keys
        keys[at] = redraw(keys[at])


def _keys(case, g):
    """row * n + column of every entry, all distinct; how many there are, and how long the rows are in all, does not
    depend on the seed."""
    n, nnz, matrix = case["n"], case["nnz"], case["matrix"]

    def ints(hi, count):
        return torch.randint(0, hi, (count,), generator=g, device=DEVICE, dtype=torch.int64)

    def row_of(keys):
        return torch.div(keys, n, rounding_mode="floor")

    def same_row(keys):
        return row_of(keys) * n + ints(n, keys.numel())

    if matrix == "uniform":
        return _distinct(ints(n * n, nnz), lambda k: ints(n * n, k.numel()))
    if matrix == "banded":
        i = torch.arange(n, device=DEVICE, dtype=torch.int64)
        diagonals = [i[max(0, -o):min(n, n - o)] * (n + 1) + o for o in OFFSETS]
        offsets = torch.tensor(OFFSETS, device=DEVICE)
        extra = _distinct(ints(n * n, int(EXTRA * nnz)), lambda k: ints(n * n, k.numel()),
                          bad=lambda k: torch.isin(k - row_of(k) * (n + 1), offsets))
        return torch.cat(diagonals + [extra])
    if matrix == "blockfem":
        nb = n // 4

        def in_band(br):   # a block column within BAND_BLOCKS of every block row of br
            lo, hi = (br - BAND_BLOCKS).clamp(min=0), (br + BAND_BLOCKS).clamp(max=nb - 1)
            u = torch.rand(br.numel(), generator=g, device=DEVICE, dtype=torch.float64)
            return br * nb + lo + (u * (hi - lo + 1).double()).long().minimum(hi - lo)

        br = torch.arange(nb, device=DEVICE, dtype=torch.int64).repeat_interleave(BLOCKS_PER_ROW)
        blocks = _distinct(in_band(br), lambda k: in_band(torch.div(k, nb, rounding_mode="floor")))
        br, q = torch.div(blocks, nb, rounding_mode="floor"), torch.arange(16, device=DEVICE, dtype=torch.int64)
        return ((br * 4)[:, None] + q // 4).reshape(-1) * n + (((blocks - br * nb) * 4)[:, None] + q % 4).reshape(-1)
    length = torch.from_numpy(_lengths(n, nnz, _exponent(matrix))).to(DEVICE)
    length = length[torch.randperm(n, generator=g, device=DEVICE)]
    row = torch.repeat_interleave(torch.arange(n, device=DEVICE, dtype=torch.int64), length)
    col = ints(n, row.numel())
    if matrix == "local":
        start = torch.cumsum(length, 0) - length
        within = torch.arange(row.numel(), device=DEVICE, dtype=torch.int64) - start[row]
        near = (length.double() * LOCAL).long().clamp_(max=WINDOW)[row]
        shifted = (row + ints(2 * WINDOW + 1, row.numel()) - WINDOW).clamp_(0, n - 1)
        col = torch.where(within < near, shifted, col)
    return _distinct(row * n + col, same_row)


def _coo(case, seed):
    """Unsorted COO on the GPU."""
    g = _generator(seed)
    keys = _keys(case, g)
    keys = keys[torch.randperm(keys.numel(), generator=g, device=DEVICE)]
    row = torch.div(keys, case["n"], rounding_mode="floor")
    return row.to(torch.int32), (keys - row * case["n"]).to(torch.int32), _uniform((keys.numel(),), g)


# ----------------------------------------------------------------------------- layouts
@functools.lru_cache(maxsize=None)
def _context():
    return B.Context(DEVICE)


def _desc(layout):
    P = B.us_desc_preset
    return {"csr": lambda: P(B.US_F_CSR), "dcsr": lambda: P(B.US_F_DCSR), "csc": lambda: P(B.US_F_CSC),
            "dcsc": lambda: P(B.US_F_DCSC), "coo": lambda: P(B.US_F_COO), "dia": lambda: P(B.US_F_DIA),
            "ell": lambda: P(B.US_F_ELL), "bcsr": lambda: P(B.US_F_BCSR, 4, 4)}[layout]()


def _predicate(layout):
    if layout == "dia+csr":   # diagonals at least 90 % full
        return B.make_predicate([B.expr(B.US_E_AFFINE, -1, 1)], B.US_P_SUM_GE_FRAC_OF_CAPACITY, 9, 10)
    return B.make_predicate([B.expr(B.US_E_AFFINE, 1, 0)], B.US_P_RANK_LT_PERCENTILE, 9, 10)


def _build(ctx, n, coo, layout):
    """The resident layout (two parts for a hybrid)."""
    if "+" in layout:
        a, b = layout.split("+")
        return list(B.us_decompose(ctx, n, n, *coo, _desc(a), _desc(b), _predicate(layout)))
    return [B.us_convert(ctx, n, n, *coo, _desc(layout))]


def _arrays(part):
    """Everything a layout consists of, level by level."""
    out = [part.val()]
    for level in range(part.desc.nlevels):
        out += [a for a in (part.ptr(level), part.idx(level)) if a is not None]
    return out


# ----------------------------------------------------------------------------- the interface
def prepare(case, seed):
    n, op, layout = case["n"], case["op"], case["layout"]
    ctx = _context()
    state = {"op": op, "ctx": ctx, "n": n, "layout": layout}
    coo = _coo(case, seed)
    if op in ("convert", "decompose"):
        state["coo"] = coo
        state["descs"] = [_desc(d) for d in layout.split("+")]
        state["pred"] = _predicate(layout) if op == "decompose" else None
    elif op == "reconvert":
        src, dst = layout.split(">")
        state["src"], state["desc"] = _build(ctx, n, coo, src)[0], _desc(dst)
    else:
        g = _generator(seed, 1)
        state["parts"] = _build(ctx, n, coo, layout)
        shape = (n,) if op == "spmv" else (n, case["cols"])
        state["x"], state["y"] = _uniform(shape, g), torch.empty(shape, device=DEVICE)
    return state


def run(state):
    ctx, op, n = state["ctx"], state["op"], state["n"]
    if op in ("spmv", "spmm"):
        product = B.us_spmv if op == "spmv" else B.us_spmm
        for k, part in enumerate(state["parts"]):   # a hybrid: the second part adds to the first
            product(ctx, part, state["x"], state["y"], accumulate=k > 0)
        return state["y"]
    if op == "convert":
        parts = [B.us_convert(ctx, n, n, *state["coo"], state["descs"][0])]
    elif op == "decompose":
        parts = B.us_decompose(ctx, n, n, *state["coo"], *state["descs"], state["pred"])
    else:
        parts = [B.us_convert_formatted(ctx, state["src"], state["desc"])]
    out = [_arrays(p) for p in parts]
    for p in parts:
        p.free(wait=False)   # the arrays above stay: torch keeps the memory of a tensor that is still referred to
    return out


def work(case):
    n, nnz, op, layout = case["n"], case["nnz"], case["op"], case["layout"]
    ptr, entries = 4.0 * (n + 1), float(nnz)

    def stored(name):
        if name in ("csr", "csc", "dcsr", "dcsc"):
            return 8.0 * nnz + ptr
        if name == "bcsr":
            return 4.0 * nnz + 4.0 * nnz / 16 + ptr / 4
        if name == "dia+csr":
            return 4.0 * nnz + 8.0 * int(EXTRA * nnz) + ptr
        # ELL + COO: the entries of either part (how much padding the slab carries is the layout's, but it has to be written)
        length = _lengths(n, nnz, _exponent(case["matrix"]))
        width = int(np.sort(length)[max(0, -(-9 * n // 10) - 1)])
        return 8.0 * width * n + 12.0 * float(np.maximum(length - width, 0).sum())

    if case["matrix"] == "banded":
        entries *= 1 + EXTRA
    if op in ("convert", "decompose"):
        return {"bytes": 12.0 * entries + stored(layout), "flops": 0}
    if op == "reconvert":
        src, dst = layout.split(">")
        return {"bytes": stored(src) + stored(dst), "flops": 0}
    cols = case.get("cols", 1)
    return {"bytes": stored(layout) + 8.0 * n * cols, "flops": 2.0 * entries * cols}


def tolerance(case):
    # layouts hold coordinates, counts and copied values; products are sums of fp32 products in any order
    return {"rel": 1e-5} if case["op"] in ("spmv", "spmm") else "exact"
