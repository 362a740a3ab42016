"""The GEMM of the library's own schedule choice, at the edges of its tiles and k-slabs.

Entries are integers small enough for every partial sum to be exact in the type, so the comparison is bit for bit
whatever the order of the sums.  What surrounds the matrices in memory is NaN.
"""
import numpy as np
import pytest

from tests.gpu_util import announce, to_host

pytestmark = pytest.mark.gpu

# (m, n, k): around one tile of 32, 64, 128 rows; k around a slab of 16 (fp64) and 32 (fp32) and around two and three
SHAPES = [(1, 1, 1), (15, 17, 2), (32, 32, 16), (33, 31, 17), (64, 32, 33), (65, 66, 32), (63, 129, 47), (130, 259, 70),
          (2100, 70, 64), (1100, 1030, 49), (2050, 1923, 31)]


@pytest.mark.parametrize("pad", [0, 1, 2, 5])
@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("op", [0, 1, 4])
def test_edges_bit_for_bit(op, dtype, pad):
    import torch
    from paper_2309_07235_amd import binding as B
    dt = getattr(torch, dtype)
    rng = np.random.default_rng(17 + op)

    def put(x):
        """x with `pad` extra columns and one extra row of NaN around it, offset by `pad` elements."""
        full = torch.full((x.shape[0] + 1, x.shape[1] + 2 * pad), float("nan"), dtype=dt, device="cuda")
        view = full[:x.shape[0], pad:pad + x.shape[1]]
        view.copy_(torch.from_numpy(x))
        return full, view

    for m, n, k in SHAPES:
        announce(f"gemm op {op} {dtype} pad {pad} {m} x {n} x {k}")
        a = rng.integers(-3, 4, (k, m) if op == 4 else (m, k)).astype(dtype)
        b, c = (rng.integers(-3, 4, s).astype(dtype) for s in ((k, n), (m, n)))
        prod = (a.T if op == 4 else a) @ b
        _, ad = put(a)
        _, bd = put(b)
        cfull, cd = put(c)
        B.dla_gemm(op, ad, bd, cd)
        got = to_host(cd)
        assert np.array_equal(got, prod if op == 0 else c - prod), (m, n, k)
        outside = cfull.clone()
        outside[:m, pad:pad + n] = float("nan")
        assert bool(torch.isnan(outside).all()), "written outside the matrix"
        assert int(torch.isnan(cfull).sum()) == cfull.numel() - m * n
