"""The diagonal-block kernel at the edges of its 16-wide stages: sizes around every count of sub-blocks it treats
differently (one, two, half a block, the full 128, a second block), and the pivot a breakdown is reported for.

The gates are the factorisation tests' own: max |x - y| / max(|y|, rms(y)) of 1e-9 in fp64 and 1e-4 in fp32 against the
oracle in fp64 on the same (rounded) input.
"""
import numpy as np
import pytest

from tests.gpu_util import announce, to_host
from tests.metrics import cholesky_rel_err, lu_rel_err

pytestmark = pytest.mark.gpu

SIZES = [1, 15, 16, 17, 32, 33, 48, 63, 64, 65, 79, 80, 96, 111, 112, 113, 127, 128, 129, 144]


def _factor(kind, A, dtype, pad):
    """Factor A inside a wider buffer of NaN; the result, info, and whether the padding is still NaN."""
    import torch
    from paper_2309_07235_amd import binding as B
    n = A.shape[0]
    full = torch.full((n, n + pad), float("nan"), dtype=getattr(torch, dtype), device="cuda")
    view = full[:, :n]
    view.copy_(torch.from_numpy(A))
    info = torch.full((1,), -7, dtype=torch.int32, device="cuda")
    (B.lu_factor if kind == "lu" else B.cholesky_factor)(view, info=info)
    return to_host(view).astype(np.float64), int(info.item()), bool(torch.isnan(full[:, n:]).all())


@pytest.mark.parametrize("pad", [0, 3])
@pytest.mark.parametrize("dtype,gate", [("float64", 1e-9), ("float32", 1e-4)])
@pytest.mark.parametrize("kind", ["lu", "chol"])
def test_sizes(kind, dtype, gate, pad):
    import oracle
    from paper_2309_07235_amd import inputs
    for n in SIZES:
        announce(f"{kind} {dtype} n {n} pad {pad}")
        A = inputs.general_dominant_matrix(n, 5) if kind == "lu" else inputs.spd_matrix(n, 5)
        A = A.astype(dtype).astype(np.float64)
        if kind == "chol":  # the upper triangle is neither read nor written through
            A[np.triu_indices(n, 1)] = np.nan
        got, info, padding_kept = _factor(kind, A, dtype, pad)
        clean = np.where(np.tri(n, dtype=bool), A, 0.0) if kind == "chol" else A
        want, _ = (oracle.lu if kind == "lu" else oracle.cholesky)(clean)
        err = (lu_rel_err if kind == "lu" else cholesky_rel_err)(got, want)
        assert info == 0 and padding_kept and err <= gate, (n, info, err)
        assert kind == "lu" or np.all(np.triu(got, 1) == 0.0)


@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("kind,value", [("lu", 0.0), ("chol", 0.0), ("chol", -1.0)])
def test_first_bad_pivot(kind, value, dtype):
    n = 150
    for p in (0, 1, 15, 16, 31, 47, 63, 64, 100, 112, 127, 128, 149):
        A = np.eye(n)
        A[p, p] = value
        A[min(p + 20, n - 1), min(p + 20, n - 1)] = value  # a later one is not the one reported
        announce(f"{kind} {dtype} pivot {p} = {value}")
        assert _factor(kind, A, dtype, 0)[1] == p + 1
