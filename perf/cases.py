"""The library's workloads for timing and for comparing two builds of it.

Each case is one call of a public entry point as a program that uses the library makes it: matrices, workspace and
schedule are in hand, the call runs on the current stream.  The in-place calls (factorisations, solves) are handed a
fresh copy of their input, since a program keeps the original for residuals or for the next solve; that copy is part
of the pass.
"""
import math

import torch

from paper_2309_07235_amd import binding as B
from paper_2309_07235_amd import inputs

DTYPES = {"f64": torch.float64, "f32": torch.float32}
CODES = {"f64": B.DLA_F64, "f32": B.DLA_F32}
MM3_DIMS = ("ni", "nk", "nj", "nm", "nl")
MAX_N = 8192              # the largest factorisation listed


def _mm3(name, dtype, dims, tile=0):
    return {"name": name, "op": "mm3", "dtype": dtype, "tile": tile, **{k: dims[k] for k in MM3_DIMS}}


def _factor(name, op, dtype, n, nb=0):
    return {"name": name, "op": op, "dtype": dtype, "n": n, "nb": nb}


def _solve(name, op, dtype, n, nrhs):
    return {"name": name, "op": op, "dtype": dtype, "n": n, "nrhs": nrhs}


def listed():
    return [
        # the small dataset of the paper's 3mm at a tile a search proposes: two launches, latency only
        _mm3("mm3_128_tile16_f64", "f64", inputs.MM3_SMALL, tile=16),
        # the large dataset in single precision: sizes that no tile divides
        _mm3("mm3_large_f32", "f32", inputs.MM3_LARGE_PAPER_ORDER),
        # the extralarge dataset: the headline 3mm
        _mm3("mm3_extralarge_f64", "f64", inputs.MM3_EXTRALARGE),
        # a small dense system factored once: three block columns, the last one ragged
        _factor("lu_300_f64", "lu_factor", "f64", 300),
        # the mid-size Cholesky at the block size a search visits
        _factor("cholesky_1024_nb64_f64", "cholesky_factor", "f64", 1024, nb=64),
        # the headline factorisations (the paper's extralarge dataset)
        _factor("lu_4000_f64", "lu_factor", "f64", 4000),
        _factor("cholesky_4000_f64", "cholesky_factor", "f64", 4000),
        # the largest ones, one in each precision
        _factor("lu_8192_f64", "lu_factor", "f64", 8192),
        _factor("cholesky_8192_f32", "cholesky_factor", "f32", 8192),
        # one system with a block of right-hand sides, solved right after its factorisation
        _solve("lu_solve_4000x64_f64", "lu_solve", "f64", 4000, 64),
        # a program that keeps the factor and solves for one right-hand side at a time
        _solve("cholesky_solve_prepared_2000x1_f64", "cholesky_solve_prepared", "f64", 2000, 1),
        # many right-hand sides at once
        _solve("cholesky_solve_8192x1024_f32", "cholesky_solve", "f32", 8192, 1024),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(("mm3", "lu_factor", "cholesky_factor", "lu_solve", "cholesky_solve", "lu_solve_prepared",
                     "cholesky_solve_prepared"))
    dtype = rng.choice(("f64", "f32"))
    if op == "mm3":
        dims = {k: _log_uniform(rng, 64, 2400) for k in MM3_DIMS}
        # half of the calls leave the tile to the library; the smallest tiles are for the small products
        tiles = (16, 32) if max(dims.values()) <= 512 else (32, 64, 128)
        return {"op": op, "dtype": dtype, "tile": rng.choice((0, rng.choice(tiles))), **dims}
    n = _log_uniform(rng, 100, MAX_N)
    if op in ("lu_factor", "cholesky_factor"):
        # mostly the library's block size; the small one belongs to the smaller matrices, 256 is two panels of 128
        return {"op": op, "dtype": dtype, "n": n, "nb": rng.choice((0, 0, 0, 64 if n <= 2048 else 128, 256))}
    return {"op": op, "dtype": dtype, "n": n, "nrhs": _log_uniform(rng, 1, 1024)}


def _uniform(gen, rows, cols):
    """rows x cols, uniform in [-1, 1), fp64."""
    return torch.rand(rows, cols, dtype=torch.float64, device="cuda", generator=gen).mul_(2.0).sub_(1.0)


def _system(gen, n, kind):
    """M*M^T/n plus n*I (LU: diagonally dominant, stable without pivoting) or plus I (Cholesky: positive definite)."""
    m = _uniform(gen, n, n)
    a = torch.mm(m, m.t()).div_(float(n))
    a.diagonal().add_(float(n) if kind == "lu" else 1.0)
    return a


def _generator(seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return gen


def _mm3_operands(gen, case):
    ni, nk, nj, nm, nl = (case[k] for k in MM3_DIMS)
    return [_uniform(gen, r, c).to(DTYPES[case["dtype"]]) for r, c in ((ni, nk), (nk, nj), (nj, nm), (nm, nl))]


def prepare(case, seed):
    gen = _generator(seed)
    op, dtype, code = case["op"], DTYPES[case["dtype"]], CODES[case["dtype"]]
    st = {"op": op}
    if op == "mm3":
        ni, nj, nl = case["ni"], case["nj"], case["nl"]
        st["ops"] = _mm3_operands(gen, case)
        st["g"] = torch.empty((ni, nl), dtype=dtype, device="cuda")
        t = case["tile"]
        st["params"] = B.Mm3Params(*[B.GemmParams(t, t, 0, 0, 0, 0) for _ in range(3)]) if t else None
        st["ws"] = torch.empty(B.mm3_workspace_bytes(ni, nj, nl, code), dtype=torch.uint8, device="cuda")
        return st
    n, kind = case["n"], op.split("_")[0]
    a = _system(gen, n, kind).to(dtype)
    params = B.FactorParams(case["nb"], -1, B.GemmParams(), 0) if case.get("nb") else None
    fws = torch.empty(B.factor_workspace_bytes(n, code, params), dtype=torch.uint8, device="cuda")
    info = torch.zeros(1, dtype=torch.int32, device="cuda")
    factor = B.lu_factor if kind == "lu" else B.cholesky_factor
    if op in ("lu_factor", "cholesky_factor"):
        st.update(a0=a, a=torch.empty_like(a), params=params, ws=fws, info=info)
        return st
    factor(a, workspace=fws, info=info)
    st["f"] = a
    st["b0"] = _uniform(gen, n, case["nrhs"]).to(dtype)
    st["b"] = torch.empty_like(st["b0"])
    if op.endswith("_prepared"):
        st["ws"] = (B.lu_solve_prepare if kind == "lu" else B.cholesky_solve_prepare)(a, case["nrhs"])
    else:
        st["ws"] = torch.empty(B.solve_workspace_bytes(n, case["nrhs"], code), dtype=torch.uint8, device="cuda")
    return st


def run(st):
    op = st["op"]
    if op == "mm3":
        B.mm3(*st["ops"], st["g"], st["params"], workspace=st["ws"])
        return st["g"]
    if op in ("lu_factor", "cholesky_factor"):
        st["a"].copy_(st["a0"])
        getattr(B, op)(st["a"], st["params"], workspace=st["ws"], info=st["info"])
        return st["a"], st["info"]
    st["b"].copy_(st["b0"])
    getattr(B, op)(st["f"], st["b"], workspace=st["ws"])
    return st["b"]


def _lu_no_pivoting(a, nb=64):
    """L (unit, below the diagonal) and U of a in one matrix, by torch's own operations."""
    a, n = a.clone(), a.shape[0]
    for k in range(0, n, nb):
        e = min(k + nb, n)
        for j in range(k, e):
            a[j + 1:, j] /= a[j, j]
            a[j + 1:, j + 1:e] -= torch.outer(a[j + 1:, j], a[j, j + 1:e])
        if e < n:
            a[k:e, e:] = torch.linalg.solve_triangular(a[k:e, k:e], a[k:e, e:], upper=False, unitriangular=True)
            a[e:, e:] -= torch.mm(a[e:, k:e], a[k:e, e:])
    return a


def exact(case, seed):
    """run()'s outputs from the same inputs, by torch in fp64."""
    gen, op = _generator(seed), case["op"]
    if op == "mm3":
        a, b, c, d = (x.double() for x in _mm3_operands(gen, case))
        return torch.mm(torch.mm(a, b), torch.mm(c, d))
    n, kind = case["n"], op.split("_")[0]
    a = _system(gen, n, kind).to(DTYPES[case["dtype"]]).double()
    f = _lu_no_pivoting(a) if kind == "lu" else torch.linalg.cholesky(a)
    if op in ("lu_factor", "cholesky_factor"):
        return f, None
    b = _uniform(gen, n, case["nrhs"]).to(DTYPES[case["dtype"]]).double()
    if kind == "lu":
        y = torch.linalg.solve_triangular(f, b, upper=False, unitriangular=True)
        return torch.linalg.solve_triangular(f, y, upper=True)
    y = torch.linalg.solve_triangular(f, b, upper=False)
    return torch.linalg.solve_triangular(f.t(), y, upper=True)


def work(case):
    """Inputs read once, outputs written once; the textbook operation counts."""
    size = 8 if case["dtype"] == "f64" else 4
    if case["op"] == "mm3":
        ni, nk, nj, nm, nl = (case[k] for k in MM3_DIMS)
        return {"bytes": size * (ni * nk + nk * nj + nj * nm + nm * nl + ni * nl),
                "flops": 2.0 * (ni * nk * nj + nj * nm * nl + ni * nj * nl)}
    n = case["n"]
    if case["op"] == "lu_factor":
        return {"bytes": 2 * size * n * n, "flops": 2.0 * n ** 3 / 3.0}
    if case["op"] == "cholesky_factor":  # the lower triangle in, the whole matrix (zeros above) out
        return {"bytes": size * (n * (n + 1) // 2 + n * n), "flops": n ** 3 / 3.0}
    factor = n * n if case["op"].startswith("lu") else n * (n + 1) // 2
    return {"bytes": size * (factor + 2 * n * case["nrhs"]), "flops": 2.0 * n * n * case["nrhs"]}


# About four times the difference from exact(), in units of the type's rounding.  3mm: two constants.  Factors and
# solves: the sums they add up grow with n, so do their differences: rel = 4 eps (a + n / b), the largest one c times
# that.  Measured at n = 100 to 8192; in eps, rel and largest, at n = 8192: LU fp64 20 and 95, Cholesky fp64 7.4 and 61,
# fp32 12.9 and 73, solves fp64 20 and 100, fp32 28 and 105.
MM3_TOLERANCE = {"f64": (1.5e-14, 1e-13), "f32": (6e-6, 4e-5)}
GROWTH = {
    ("lu_factor", "f64"): (3, 450, 5),
    ("lu_factor", "f32"): (6, 8192, 3),
    ("cholesky_factor", "f64"): (1, 1200, 8),
    ("cholesky_factor", "f32"): (1, 700, 8),
    ("solve", "f64"): (4, 500, 5),
    ("solve", "f32"): (4, 350, 4),
}


def tolerance(case):
    op, dtype = case["op"], case["dtype"]
    if op == "mm3":
        rel, largest = MM3_TOLERANCE[dtype]
        return {"rel": rel, "max": largest}
    if (op, dtype) == ("lu_factor", "f32") and case["n"] >= 1024:
        # the diagonal, about n, outweighs what the updates take from it: a pivot is its input but for one rounding
        return {"rel": 2.4e-7, "max": 5e-7}
    a, b, c = GROWTH[op if op.endswith("_factor") else "solve", dtype]
    rel = 4.0 * torch.finfo(DTYPES[dtype]).eps * (a + case["n"] / b)
    return {"rel": rel, "max": c * rel}
