"""Solves with few right-hand sides: both passes in one launch, its workgroups waiting for each other (flow_kernel)."""
import numpy as np
import pytest

from paper_2309_07235_amd import inputs
from tests.gpu_util import announce, to_device, to_host
from tests.metrics import EPS32, EPS64, max_rel_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2309_07235_amd import binding
    return binding


def _system(kind, n, seed, dtype):
    """A factor (with an unused other triangle of ones for Cholesky) and its matrix, in fp64, representable in dtype."""
    rng = np.random.default_rng(seed)
    low = np.tril(rng.uniform(-1, 1, (n, n)), -1) / np.sqrt(n) + (np.eye(n) if kind == "lu" else np.diag(rng.uniform(1, 2, n)))
    up = np.triu(rng.uniform(-1, 1, (n, n)), 1) / np.sqrt(n) + np.diag(rng.uniform(1, 2, n))
    low, up = (x.astype(dtype).astype(np.float64) for x in (low, up))
    if kind == "lu":
        return np.tril(low, -1) + up, low, up
    return low + np.triu(np.ones((n, n)), 1), low, low.T


def _reference(low, up, rhs):
    from scipy.linalg import solve_triangular
    return solve_triangular(up, solve_triangular(low, rhs, lower=True), lower=False)


def _bound(low, up, rhs, eps):
    """Relative to the largest entries.  A pass adds up at most n products per entry and, by blocks, multiplies by inverted blocks:
    c n eps times the norms of the factors and of their inverses, which for these systems (off-diagonal entries of size
    1 / sqrt(n), pivots in [1, 2]) are small constants; 16 covers both passes.  Measured: a tenth of n eps."""
    return 16 * len(low) * eps


# one block, whole and ragged; the first blocks with a sum (4), a last block of one row and of one row less than a whole one;
# one column, a whole and a ragged column block, the most; the two widths of a workgroup (2100 x 64 takes two column blocks)
@pytest.mark.parametrize("kind", ["lu", "chol"])
@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("n,nrhs,lda,ldb", [(255, 16, 255, 16), (256, 17, 257, 19), (257, 64, 257, 64), (768, 1, 768, 1), (769, 33, 771, 33),
                                            (1023, 63, 1025, 64), (1025, 2, 1026, 7), (1281, 15, 1281, 15), (2100, 64, 2101, 65),
                                            (2305, 61, 2308, 61)])
def test_against_substitution(B, kind, dtype, n, nrhs, lda, ldb):
    import torch
    announce(f"flow {kind} {dtype} n={n} nrhs={nrhs} lda={lda} ldb={ldb}")
    d = getattr(torch, dtype)
    F, low, up = _system(kind, n, n + nrhs, dtype)
    rhs = inputs.uniform_matrix(61, 3, n, nrhs).astype(dtype).astype(np.float64)
    f = torch.full((n, lda), 3.5, dtype=d, device="cuda")
    b = torch.full((n, ldb), -7.25, dtype=d, device="cuda")
    f[:, :n] = to_device(F, d)
    b[:, :nrhs] = to_device(rhs, d)
    (B.lu_solve if kind == "lu" else B.cholesky_solve)(f[:, :n], b[:, :nrhs])
    got = to_host(b).astype(np.float64)
    eps = EPS64 if dtype == "float64" else EPS32
    assert max_rel_err(got[:, :nrhs], _reference(low, up, rhs)) <= _bound(low, up, rhs, eps)
    assert np.all(got[:, nrhs:] == -7.25)


@pytest.mark.parametrize("kind", ["lu", "chol"])
@pytest.mark.parametrize("n,nrhs,dtype", [(200, 3, "float64"), (1100, 40, "float64"), (1030, 64, "float32"), (2100, 62, "float64")])
def test_waits_that_give_up(B, kind, n, nrhs, dtype):
    """Every wait ends at once: what the launch has not finished then comes from the row by row substitution."""
    import torch
    announce(f"flow give-up {kind} {dtype} n={n} nrhs={nrhs}")
    d = getattr(torch, dtype)
    F, low, up = _system(kind, n, 7, dtype)
    rhs = inputs.uniform_matrix(62, 3, n, nrhs).astype(dtype).astype(np.float64)
    f, b = to_device(F, d), to_device(rhs, d)
    B.solve_giveup_selftest(0 if kind == "lu" else 1, f, b)
    eps = EPS64 if dtype == "float64" else EPS32
    assert max_rel_err(to_host(b).astype(np.float64), _reference(low, up, rhs)) <= _bound(low, up, rhs, eps)


@pytest.mark.parametrize("dtype,empty", [("float64", 0x7FF9D1A5C3B2E607), ("float32", 0x7FD1A5C3)])
def test_the_pattern_that_means_not_there_yet(B, dtype, empty):
    """Right-hand sides that hold the very NaN the areas are filled with, and infinities: their columns are NaN or infinite
    from there on, the others are what they are without them, and the call ends."""
    import torch
    n, nrhs = 900, 20
    announce(f"flow NaN {dtype}")
    F, low, up = _system("lu", n, 9, dtype)
    rhs = inputs.uniform_matrix(63, 3, n, nrhs).astype(dtype)
    bad = rhs.copy()
    bad[5, 3] = np.array([empty], dtype=np.uint64 if dtype == "float64" else np.uint32).view(dtype)[0]
    bad[700, 4] = np.inf
    d = getattr(torch, dtype)
    f, b, c = to_device(F, d), to_device(rhs, d), to_device(bad, d)
    B.lu_solve(f, b)
    B.lu_solve(f, c)
    clean, got = to_host(b), to_host(c)
    rest = [j for j in range(nrhs) if j not in (3, 4)]
    assert np.array_equal(got[:, rest], clean[:, rest])
    assert np.all(np.isnan(got[:, 3])) and not np.any(np.isfinite(got[700:, 4]))


def test_several_streams_at_once(B):
    """Solves on four streams, each with a workspace of its own, submitted together: every result is the lone call's."""
    import torch
    announce("flow on four streams")
    cases = []
    for i, (n, nrhs) in enumerate(((1500, 64), (2000, 1), (900, 33), (2304, 16))):
        F, _, _ = _system("lu" if i % 2 else "chol", n, 70 + i, "float64")
        f, b0 = to_device(F), to_device(inputs.uniform_matrix(71, i, n, nrhs))
        solve = B.lu_solve if i % 2 else B.cholesky_solve
        want = b0.clone()
        ws = solve(f, want)
        cases.append((solve, f, b0, want, ws, torch.cuda.Stream()))
    torch.cuda.synchronize()
    for _ in range(5):
        got = [c[2].clone() for c in cases]
        torch.cuda.synchronize()
        for b, (solve, f, b0, _, ws, st) in zip(got, cases):
            with torch.cuda.stream(st):
                for _ in range(3):  # (the last counts: each starts from a fresh copy)
                    b.copy_(b0)
                    solve(f, b, workspace=ws)
        torch.cuda.synchronize()
        for b, c in zip(got, cases):
            assert torch.equal(b, c[3])


def test_captured_and_replayed(B):
    import torch
    announce("flow in a graph")
    n, nrhs = 1100, 5
    F, _, _ = _system("lu", n, 81, "float64")
    f = to_device(F)
    rhs = [to_device(inputs.uniform_matrix(82, i, n, nrhs)) for i in range(3)]
    want = [r.clone() for r in rhs]
    ws = B.lu_solve(f, want[0])
    for w in want[1:]:
        B.lu_solve(f, w, workspace=ws)
    b = rhs[0].clone()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.lu_solve(f, b, workspace=ws)
    for r, w in zip(rhs * 2, want * 2):
        b.copy_(r)
        graph.replay()
        other = r.clone()
        B.lu_solve(f, other)  # eager work between the replays
        torch.cuda.synchronize()
        assert torch.equal(b, w) and torch.equal(other, w)


@pytest.mark.parametrize("kind", ["lu", "chol"])
@pytest.mark.parametrize("n,nrhs,dtype", [(250, 3, "float64"), (257, 1, "float32"), (1100, 40, "float64"), (1030, 64, "float32"), (2305, 61, "float64")])
def test_workgroups_that_stay_away(B, kind, n, nrhs, dtype):
    """Every eighth workgroup leaves at once: the others take over its pieces, and each piece is what it is in an ordinary call."""
    import torch
    announce(f"flow absent {kind} {dtype} n={n} nrhs={nrhs}")
    d = getattr(torch, dtype)
    F, _, _ = _system(kind, n, 17, dtype)
    f, rhs = to_device(F, d), to_device(inputs.uniform_matrix(64, 3, n, nrhs), d)
    want, got = rhs.clone(), rhs.clone()
    (B.lu_solve if kind == "lu" else B.cholesky_solve)(f, want)
    B.solve_absent_selftest(0 if kind == "lu" else 1, f, got)
    assert torch.equal(got, want)


def test_large_solves_on_several_streams(B):
    """Four solves that would each fill the card, on four streams, with factorisations beside them: they hold compute units that the
    others' next workgroups need, and all end with the lone call's result bit for bit."""
    import torch
    n = 8192
    gen = torch.Generator(device="cuda").manual_seed(5)
    f = torch.rand(n, n, dtype=torch.float64, device="cuda", generator=gen) / n + torch.eye(n, dtype=torch.float64, device="cuda")
    g0 = f[:3000, :3000].contiguous()
    cases = []
    for nrhs in (64, 33, 64, 1):
        b0 = torch.rand(n, nrhs, dtype=torch.float64, device="cuda", generator=gen)
        want = b0.clone()
        ws = B.lu_solve(f, want)
        cases.append((b0, want, ws, torch.cuda.Stream()))
    factor = g0.clone()
    B.lu_factor(factor, info=torch.zeros(1, dtype=torch.int32, device="cuda"))
    side, info = torch.cuda.Stream(), torch.zeros(1, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    for round_ in range(3):
        announce(f"flow large on four streams, pass {round_}")
        got, x = [c[0].clone() for c in cases], g0.clone()
        torch.cuda.synchronize()
        for b, (b0, _, ws, st) in zip(got, cases):
            with torch.cuda.stream(st):
                for _ in range(4):
                    b.copy_(b0)
                    B.lu_solve(f, b, workspace=ws)
        with torch.cuda.stream(side):
            for _ in range(3):
                x.copy_(g0)
                B.lu_factor(x, info=info)
        torch.cuda.synchronize()
        for b, c in zip(got, cases):
            assert torch.equal(b, c[1])
        assert int(info.item()) == 0 and torch.equal(x, factor)


@pytest.mark.parametrize("kind", ["lu", "chol"])
@pytest.mark.parametrize("nrhs", [1, 40])
def test_rounding_is_that_of_one_block_product(B, kind, nrhs):
    """An entry of a pass is mostly one term, the diagonal's.  It is rounded at its own size about 20 times (16 steps of the wave that
    holds that term, the sums of waves), half an ulp each: sqrt(20 / 12) ulp, 0.72 eps on average, so 0.93 eps, and 1.3 eps for two
    passes (measured 1.2 to 1.4).  With the next block's product behind it in the same sum there are 36, and it was 2.2 to 2.5."""
    from scipy.linalg import lu_factor, solve_triangular
    import torch
    n = 1100
    announce(f"flow rounding {kind} nrhs={nrhs}")
    m = np.random.default_rng(3).uniform(-1, 1, (n, n))
    a = m @ m.T / n + (n if kind == "lu" else 1) * np.eye(n)
    if kind == "lu":
        f, piv = lu_factor(a)
        assert np.array_equal(piv, np.arange(n))
    else:
        f = np.linalg.cholesky(a)
    f = f.astype(np.float32)
    low = np.tril(f.astype(np.float64), -1) + np.eye(n) if kind == "lu" else f.astype(np.float64)
    rhs = inputs.uniform_matrix(65, 3, n, nrhs).astype(np.float32)
    b = to_device(rhs, torch.float32)
    (B.lu_solve if kind == "lu" else B.cholesky_solve)(to_device(f, torch.float32), b)
    y = solve_triangular(low, rhs.astype(np.float64), lower=True)
    want = solve_triangular(np.triu(f.astype(np.float64)) if kind == "lu" else low.T, y, lower=False)
    got = to_host(b).astype(np.float64)
    assert np.linalg.norm(got - want) <= 1.8 * EPS32 * np.linalg.norm(want)
