"""Factorisations in 64 x 64 tiles (tile_factor_kernel, one team and two to a workgroup): edges of tiles, alignment, hand-over,
breakdown, and the line to the pipeline."""
import numpy as np
import pytest

from paper_2309_07235_amd import inputs
from tests.gpu_util import announce, to_device, to_host
from tests.metrics import EPS32, EPS64, cholesky_rel_err, lu_rel_err

gpu = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2309_07235_amd import binding
    return binding


def _factor(B, kind, H, dtype, pad, shift, nb):
    """The factor of H in a buffer with `pad` more columns and `shift` elements in front; the padding must stay as it was.
    What lies above the diagonal must not matter to Cholesky."""
    import torch
    n, d = len(H), getattr(torch, dtype)
    buf = torch.full((shift + n * (n + pad),), 7.25, dtype=d, device="cuda")
    a = buf[shift:].view(n, n + pad)
    a[:, :n] = to_device(H, d)
    if kind == "chol":
        a[:, :n] += torch.triu(torch.full((n, n), float("nan"), dtype=d, device="cuda"), 1)
    info = torch.full((1,), -7, dtype=torch.int32, device="cuda")
    (B.lu_factor if kind == "lu" else B.cholesky_factor)(a[:, :n], B.FactorParams(nb, -1, B.GemmParams(), 0), info=info)
    got = to_host(a)
    assert np.all(got[:, n:] == 7.25) and bool((buf[:shift] == 7.25).all())
    return got[:, :n].astype(np.float64), int(info.item())


# two tiles and a row, one less than three, three, a row more; the smallest the library chooses tiles for; a ring of inverses gone
# round (1025 rows: 17 tiles).  Aligned rows (64-bit: 16 elements), rows and bases that are not
@gpu
@pytest.mark.parametrize("kind", ["lu", "chol"])
@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("n,pad,shift,nb", [(129, 0, 0, 64), (191, 1, 0, 64), (192, 0, 0, 64), (193, 31, 1, 64), (257, 0, 0, 0),
                                            (320, 0, 16, 0), (321, 3, 0, 0), (1025, 7, 0, 0), (1088, 0, 0, 0)])
def test_tiles_match_the_oracle(B, oracle, kind, dtype, n, pad, shift, nb):
    announce(f"tiles {kind} {dtype} n={n} pad={pad} shift={shift} nb={nb}")
    H = inputs.general_dominant_matrix(n, 90 + n) if kind == "lu" else inputs.spd_matrix(n, 90 + n)
    H = H.astype(dtype).astype(np.float64)
    got, info = _factor(B, kind, H, dtype, pad, shift, nb)
    want, _ = (oracle.lu if kind == "lu" else oracle.cholesky)(H)
    assert info == 0
    # each part against its own scale; a factor's element is a sum of up to n products of rounded terms
    bound = 8 * n * (EPS64 if dtype == "float64" else EPS32)
    assert (lu_rel_err if kind == "lu" else cholesky_rel_err)(got, want) <= bound
    if kind == "chol":
        assert np.all(np.triu(got, 1) == 0.0)


# both sides of the line between one team and two to a workgroup (aligned rows of LU fp64), and of the line to the pipeline (which then leaves its last rows to the
# tiles), also where the caller passes the library's defaults on; against the factor of the pipeline alone
@gpu
@pytest.mark.parametrize("kind,dtype,n", [("lu", "float64", 3699), ("lu", "float64", 3700), ("lu", "float64", 7200), ("lu", "float64", 7201),
                                          ("chol", "float64", 4799), ("chol", "float64", 4800), ("chol", "float64", 7233),
                                          ("lu", "float32", 4300), ("lu", "float32", 5601), ("chol", "float32", 5401),
                                          # the step in front of the tiles carries two panels
                                          ("lu", "float64", 7300), ("lu", "float32", 5700), ("chol", "float64", 7300),
                                          ("lu", "float64", 4992), ("lu", "float64", 5008)])
def test_lines_between_the_forms(B, kind, dtype, n):
    import torch
    announce(f"tiles lines {kind} {dtype} n={n}")
    d = getattr(torch, dtype)
    gen = torch.Generator(device="cuda").manual_seed(n)
    m = torch.rand(n, n, dtype=torch.float64, device="cuda", generator=gen) * 2 - 1
    a = torch.mm(m, m.t()) / n
    a.diagonal().add_(4.0)
    if kind == "lu":
        a += (m - m.t()) / 8
    a = a.to(d)
    outs = []
    default = B.default_params(B.DLA_KERNEL_LU if kind == "lu" else B.DLA_KERNEL_CHOLESKY, n, B.DLA_F64 if dtype == "float64" else B.DLA_F32)
    for nb, lookahead in ((0, -1), (128, 2), (default.nb, -1)):
        x, info = a.clone(), torch.full((1,), -7, dtype=torch.int32, device="cuda")
        (B.lu_factor if kind == "lu" else B.cholesky_factor)(x, B.FactorParams(nb, lookahead, B.GemmParams(), 0), info=info)
        assert int(info.item()) == 0
        outs.append(x.double())
    assert torch.equal(outs[0], outs[2])
    eps = EPS64 if dtype == "float64" else EPS32
    # the sums of both are those of the same products in another order: about sqrt(n) eps apart, and no further than n eps
    assert float((outs[0] - outs[1]).norm() / outs[1].norm()) <= 0.1 * n * eps


@gpu
@pytest.mark.parametrize("kind,n,bad", [("lu", 300, 0), ("lu", 300, 64), ("lu", 300, 299), ("chol", 700, 130), ("chol", 700, 699),
                                        ("lu", 3800, 3001), ("chol", 5000, 1), ("lu", 7300, 1000), ("lu", 7300, 7000)])
def test_first_bad_pivot(B, kind, n, bad):
    import torch
    announce(f"tiles breakdown {kind} n={n} at {bad}")
    a = torch.eye(n, dtype=torch.float64, device="cuda") * 2
    a[bad, bad] = 0.0
    if n - bad > 40:
        a[bad + 33, bad + 33] = 0.0  # a later one does not count
    info = torch.full((1,), -7, dtype=torch.int32, device="cuda")
    (B.lu_factor if kind == "lu" else B.cholesky_factor)(a, info=info)
    assert int(info.item()) == bad + 1


@gpu
@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("n", [200, 1500, 4900])
def test_waits_that_give_up_are_reported(B, kind, n):
    import torch
    announce(f"tiles give-up kind={kind} n={n}")
    a = torch.eye(n, dtype=torch.float64, device="cuda")
    assert B.factor_giveup_selftest(kind, a) == -1
    info = torch.full((1,), -7, dtype=torch.int32, device="cuda")
    a = torch.eye(n, dtype=torch.float64, device="cuda") * 4
    (B.cholesky_factor if kind else B.lu_factor)(a, info=info)
    assert int(info.item()) == 0 and torch.equal(a, torch.eye(n, dtype=torch.float64, device="cuda") * (2 if kind else 4))


@gpu
def test_on_many_streams(B):
    """A program's streams share a few hardware queues with the helper streams.  Whichever stream a call is on, the workgroups
    that wait for each other run side by side, and the result is the default stream's bit for bit."""
    import torch
    cases = []
    for kind, n, dtype in (("lu", 4000, torch.float64), ("lu", 5008, torch.float64), ("chol", 5000, torch.float64), ("lu", 5008, torch.float32),
                           ("lu", 7300, torch.float64)):
        gen = torch.Generator(device="cuda").manual_seed(n)
        m = torch.rand(n, n, dtype=torch.float64, device="cuda", generator=gen) * 2 - 1
        a = torch.mm(m, m.t()) / n
        a.diagonal().add_(4.0)
        factor, a = B.lu_factor if kind == "lu" else B.cholesky_factor, a.to(dtype)
        info = torch.full((1,), -7, dtype=torch.int32, device="cuda")
        want = a.clone()
        factor(want, info=info)
        assert int(info.item()) == 0
        cases.append((factor, a, want, info, f"{kind} n={n} {dtype}"))
    for i in range(12):
        stream = torch.cuda.Stream()
        factor, a, want, info, name = cases[i % len(cases)]
        announce(f"tiles on side stream {i}: {name}")
        info.fill_(-7)
        x = a.clone()
        stream.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(stream):
            factor(x, info=info)
        stream.synchronize()
        assert int(info.item()) == 0 and torch.equal(x, want)


# the most tiles that there are room for in either type, against the library's choice at that size (a pipeline with a tail)
@gpu
@pytest.mark.parametrize("kind,dtype,n", [("lu", "float64", 8192), ("chol", "float64", 8190), ("lu", "float32", 8000), ("chol", "float32", 7999)])
def test_largest_with_block_size_64(B, kind, dtype, n):
    import torch
    announce(f"tiles largest {kind} {dtype} n={n}")
    gen = torch.Generator(device="cuda").manual_seed(n)
    m = torch.rand(n, n, dtype=torch.float64, device="cuda", generator=gen) * 2 - 1
    a = torch.mm(m, m.t()) / n
    a.diagonal().add_(4.0)
    if kind == "lu":
        a += (m - m.t()) / 8
    a = a.to(getattr(torch, dtype))
    outs = []
    for nb in (0, 64):
        x, info = a.clone(), torch.full((1,), -7, dtype=torch.int32, device="cuda")
        (B.lu_factor if kind == "lu" else B.cholesky_factor)(x, B.FactorParams(nb, -1, B.GemmParams(), 0), info=info)
        assert int(info.item()) == 0
        outs.append(x.double())
    eps = EPS64 if dtype == "float64" else EPS32
    assert float((outs[0] - outs[1]).norm() / outs[0].norm()) <= 0.1 * n * eps  # (as in test_lines_between_the_forms)
