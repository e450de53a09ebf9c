"""The work that a program using this library has it do: y = A x through a built handle, and the
build of a handle for a matrix that has just been assembled, on the matrix families of
``workloads`` (5-point and 27-point stencils, row templates, R-MAT graphs, lognormal rows), fp32
and fp64, from sizes where a call is all latency to matrices of a hundred million nonzeros.

Matrices are generated on the GPU with the recipes of ``workloads/generators.py`` (torch's
generator instead of numpy's, so that a hundred million nonzeros take a fraction of a second).
"""
from __future__ import annotations

import math

import torch

import paper_2504_08860_amd as H

# mean of floor(lognormal(2.5, 1.2)) and the share of R-MAT draws left when duplicates are merged
LOGNORMAL_MEAN = 24.5
RMAT_KEPT = {12: 0.82, 14: 0.87, 16: 0.91, 18: 0.94, 20: 0.96, 22: 0.97}


def _case(name, op, matrix, dtype, **size):
    return {"name": name, "op": op, "matrix": matrix, "dtype": dtype, **size}


def listed():
    return [
        # one product with a small grid operator, the matrix of the smallest configuration (the
        # smoother of a coarse multigrid level): launches and host time
        _case("laplace64_f32", "spmv", "laplace", "f32", side=64),
        # the product of an iterative solver on a 3D grid: long row segments, memory-bound
        _case("stencil128_f32", "spmv", "stencil", "f32", side=128),
        # the same on an ordinary odd grid, through the entry point that never allocates (serving loops)
        _case("stencil67_f32_static", "static", "stencil", "f32", side=67),
        # rows that repeat 1024 column patterns scattered over all of x: short row segments
        _case("template20_f32", "spmv", "template", "f32", rows=1 << 20),
        # one step of a graph iteration (PageRank and the like) on a power-law graph
        _case("rmat22_f32", "spmv", "rmat", "f32", log2=22),
        # irregular rectangular matrix, the workload that bench.py is quoted on
        _case("lognormal4M_f32", "spmv", "lognormal", "f32", rows=4_000_000, cols=1_000_000),
        # wide and ragged: fewer rows than columns, no size a multiple of anything
        _case("lognormal_wide_f32", "spmv", "lognormal", "f32", rows=150_001, cols=400_009),
        # solvers that need double precision: regular and irregular rows
        _case("stencil128_f64", "spmv", "stencil", "f64", side=128),
        _case("lognormal1M2_f64", "spmv", "lognormal", "f64", rows=1_200_007, cols=299_993),
        # a matrix that has just been assembled (time stepping, Newton): build, use once, free
        _case("build_stencil128_f32", "build", "stencil", "f32", side=128),
        _case("build_rmat20_f64", "build", "rmat", "f64", log2=20),
        _case("build_lognormal4M_f32", "build", "lognormal", "f32", rows=4_000_000, cols=1_000_000),
    ]


def draw(rng):
    """One more case: any family, product or build, either type, sizes spread over their logarithm."""
    def spread(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choice(["spmv", "spmv", "spmv", "static", "build"])
    dtype = "f32" if op == "static" else rng.choice(["f32", "f32", "f64"])
    matrix = rng.choice(["laplace", "stencil", "template", "rmat", "lognormal", "lognormal"])
    if op == "static":
        # this entry point holds 8,323,072 row segments at most
        matrix = rng.choice(["laplace", "stencil"])
    case = {"op": op, "matrix": matrix, "dtype": dtype}
    if matrix == "laplace":
        case["side"] = spread(40, 1500)
    elif matrix == "stencil":
        case["side"] = spread(12, 128)
    elif matrix == "template":
        case["rows"] = spread(4_000, 1 << 20)
    elif matrix == "rmat":
        case["log2"] = rng.choice([12, 14, 16, 18, 20, 22])
    else:
        case["rows"] = spread(3_000, 4_000_000)
        case["cols"] = min(1_000_000, max(2_000, int(case["rows"] * math.exp(rng.uniform(math.log(1 / 6), math.log(4))))))
    return case


# ------------------------------------------------------------------------------- matrices

def _from_keys(keys, n_rows, n_cols):
    """CSR arrays from int64 keys row * n_cols + column, duplicates merged."""
    keys = torch.unique(keys)
    rows = torch.div(keys, n_cols, rounding_mode="floor")
    ptr = torch.zeros(n_rows + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(torch.bincount(rows, minlength=n_rows), 0, out=ptr[1:])
    return ptr.to(torch.int32), (keys - rows * n_cols).to(torch.int32)


def _grid(side, dims, offsets):
    """CSR arrays of a stencil on a side^dims grid and the mask of the diagonal entries; the
    offsets come in ascending column order."""
    n = side**dims
    r = torch.arange(n, dtype=torch.int32, device="cuda")
    axes = [torch.div(r, side**d, rounding_mode="floor") % side for d in reversed(range(dims))]  # slowest first
    mask = torch.empty((n, len(offsets)), dtype=torch.bool, device="cuda")
    cols = torch.empty((n, len(offsets)), dtype=torch.int32, device="cuda")
    for k, off in enumerate(offsets):
        inside = torch.ones(n, dtype=torch.bool, device="cuda")
        step = 0
        for d, o in enumerate(off):
            inside &= (axes[d] + o >= 0) & (axes[d] + o < side)
            step = step * side + o
        mask[:, k] = inside
        cols[:, k] = r + step
    ptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(mask.sum(1), 0, out=ptr[1:])
    diag = torch.zeros_like(mask)
    diag[:, len(offsets) // 2] = True
    return n, n, ptr.to(torch.int32), cols[mask], diag[mask]


def _matrix(case, gen):
    """(n_rows, n_cols, csr_ptr, csr_col, csr_val, x) on the GPU."""
    dt = torch.float64 if case["dtype"] == "f64" else torch.float32
    kw = dict(device="cuda", generator=gen)
    kind = case["matrix"]
    if kind == "laplace":
        n_rows, n_cols, ptr, col, diag = _grid(case["side"], 2, [(-1, 0), (0, -1), (0, 0), (0, 1), (1, 0)])
        val = torch.where(diag, 4.0, -1.0).to(dt) + (torch.rand(col.numel(), dtype=dt, **kw) - 0.5) * 0.02
    elif kind == "stencil":
        span = (-1, 0, 1)
        n_rows, n_cols, ptr, col, diag = _grid(case["side"], 3, [(a, b, c) for a in span for b in span for c in span])
        val = torch.rand(col.numel(), dtype=dt, **kw) * 2.0 - 1.0
        val[diag] = 27.0
    elif kind == "template":
        n_rows = n_cols = case["rows"]
        templates = torch.randint(0, n_cols, (1024, 32), dtype=torch.int64, **kw)
        pick = torch.randperm(n_rows, **kw) % 1024
        cols = templates[pick]
        fresh = torch.randint(0, n_cols, cols.shape, dtype=torch.int64, **kw)
        cols = torch.where(torch.rand(cols.shape, **kw) < 0.1, fresh, cols)
        ptr, col = _from_keys((torch.arange(n_rows, device="cuda")[:, None] * n_cols + cols).ravel(), n_rows, n_cols)
        val = torch.randn(col.numel(), dtype=dt, **kw)
    elif kind == "rmat":
        n_rows = n_cols = 1 << case["log2"]
        row = torch.zeros(16 * n_rows, dtype=torch.int64, device="cuda")
        column = torch.zeros_like(row)
        for _ in range(case["log2"]):
            u = torch.rand(row.numel(), **kw)
            low = u >= 0.76
            right = ((u >= 0.57) & ~low) | (u >= 0.95)
            row.mul_(2).add_(low)
            column.mul_(2).add_(right)
        ptr, col = _from_keys(row * n_cols + column, n_rows, n_cols)
        val = 1.0 - torch.rand(col.numel(), dtype=dt, **kw)
    else:
        n_rows, n_cols = case["rows"], case["cols"]
        lens = torch.exp(torch.randn(n_rows, **kw) * 1.2 + 2.5).floor().clamp(max=min(10_000, n_cols)).to(torch.int64)
        rows = torch.repeat_interleave(torch.arange(n_rows, device="cuda"), lens)
        keys = rows * n_cols + torch.randint(0, n_cols, (rows.numel(),), dtype=torch.int64, **kw)
        ptr, col = _from_keys(keys, n_rows, n_cols)
        val = torch.randn(col.numel(), dtype=dt, **kw)
    x = torch.rand(n_cols, dtype=dt, **kw) * 2.0 - 1.0
    return n_rows, n_cols, ptr, col.contiguous(), val, x


# ------------------------------------------------------------------------------- cases

class _State:
    """What a program holds: vectors and a handle, or the assembled CSR arrays."""

    handle = None

    def __del__(self):
        if self.handle is not None:
            H.hbp_free(self.handle)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    s = _State()
    s.op, s.f64 = case["op"], case["dtype"] == "f64"
    s.n_rows, s.n_cols, s.ptr, s.col, s.val, s.x = _matrix(case, gen)
    s.y = torch.empty(s.n_rows, dtype=s.x.dtype, device="cuda")
    if s.op != "build":
        build = H.hbp_build_f64 if s.f64 else H.hbp_build
        s.handle = build(s.ptr, s.col, s.val, s.n_rows, s.n_cols)
        s.ptr = s.col = s.val = None  # the handle holds its own copy
    return s


def run(s):
    if s.op == "static":
        H.hbp_spmv_static_scratch(s.handle, s.x, s.y)
        return s.y
    spmv = H.hbp_spmv_f64 if s.f64 else H.hbp_spmv
    if s.op == "spmv":
        spmv(s.handle, s.x, s.y)
        return s.y
    build = H.hbp_build_f64 if s.f64 else H.hbp_build
    handle = build(s.ptr, s.col, s.val, s.n_rows, s.n_cols)
    spmv(handle, s.x, s.y)
    H.hbp_free(handle)
    return s.y


def _shape(case):
    """(rows, columns, expected nonzeros)"""
    kind = case["matrix"]
    if kind == "laplace":
        n = case["side"] ** 2
        return n, n, 5 * n - 4 * case["side"]
    if kind == "stencil":
        n = case["side"] ** 3
        return n, n, (3 * case["side"] - 2) ** 3
    if kind == "template":
        n = case["rows"]
        return n, n, int(32 * n * min(1.0, 1.0 - 16.0 / n))
    if kind == "rmat":
        n = 1 << case["log2"]
        return n, n, int(16 * n * RMAT_KEPT[case["log2"]])
    rows, cols = case["rows"], case["cols"]
    return rows, cols, int(LOGNORMAL_MEAN * rows)


def work(case):
    """A product reads each value with a 2-byte column (blocks are at most 32768 columns wide) and x,
    and writes y.  A build with one product reads the CSR arrays, writes values and columns of the
    layout once and reads them once."""
    rows, cols, nnz = _shape(case)
    vb = 8 if case["dtype"] == "f64" else 4
    product = (vb + 2) * nnz + vb * (rows + cols)
    if case["op"] == "build":
        return {"bytes": (4 + vb) * nnz + 4 * (rows + 1) + (vb + 2) * nnz + product, "flops": 2 * nnz}
    return {"bytes": product, "flops": 2 * nnz}


def tolerance(case):
    """Measured: rows summed in other orders (8 and 2 lanes per row of the CSR kernels) against the
    path in 64 bits differ by up to 3.0e-7 / 6e-7 on R-MAT, whose longest rows hold 10^5 nonzeros, and by
    1.4e-7 elsewhere; in fp64 by 6e-16 / 1.2e-15 and 2.9e-16."""
    if case["matrix"] == "rmat":
        return {"rel": 2.5e-15 if case["dtype"] == "f64" else 1.2e-6}
    return {"rel": 1.2e-15 if case["dtype"] == "f64" else 5e-7}
