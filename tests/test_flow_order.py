"""flow_kernel's hand-overs and order of work, as far as they can be checked on the host."""
import ctypes
import subprocess
from pathlib import Path

import numpy as np
import pytest

from paper_2309_07235_amd import build

HERE = Path(__file__).resolve().parent


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    so = tmp_path_factory.mktemp("flow") / "libflow_host.so"
    subprocess.run([build.HIPCC, "--offload-arch=gfx950", "--cuda-host-only", "-std=c++17", "-O1", "-shared", "-fPIC", "-w", "-I",
                    str(build.CSRC), str(HERE / "host" / "flow_host.hip"), "-o", str(so)], check=True)
    return ctypes.CDLL(str(so))


def test_neighbouring_waits_hand_over_in_different_slots(host):
    """A wait's slot is read behind the one barrier that the wait has; the next wait may write before a slow wave has read it, so
    it must write elsewhere.  (It went by the product's number, which a wait that finds two positions complete leaves even.)"""
    slot = np.full(200, -1, dtype=np.int32)
    host.flow_host_slots(200, slot.ctypes.data_as(ctypes.POINTER(ctypes.c_int)))
    assert set(slot) == {0, 1} and np.all(slot[1:] != slot[:-1])


def _pieces(host, n, tiles_n):
    """Per piece (pass, sum, position, rows, columns) or None, and the indices of the pieces that it waits for."""
    ints = ctypes.POINTER(ctypes.c_int)
    out = np.zeros((host.flow_host_pieces(n, tiles_n, None), 5), dtype=np.int32)
    host.flow_host_pieces(n, tiles_n, out.ctypes.data_as(ints))
    pieces = [tuple(r) if r[2] >= 0 else None for r in out.tolist()]
    blocks = (n + 255) // 256
    at = {}  # (pass, sum, position, columns) -> indices
    for i, f in enumerate(pieces):
        if f:
            at.setdefault((f[0], f[1], f[2], f[4]), []).append(i)
    needs = []
    for f in pieces:
        want = []
        if f:
            back, is_sum, p, _, ct = f
            # a sum: the blocks solved so far but for the last two; a solution: those two and its sum; both of the backward pass: Y
            for q in range(p - 2) if is_sum else range(max(p - 2, 0), p):
                want += at[back, 0, q, ct]
            if not is_sum and p > 2:
                want += at[back, 1, p, ct]
            if back:
                want += at[0, 0, blocks - 1 - p, ct]
        needs.append(want)
    return pieces, needs


@pytest.mark.parametrize("n,tiles_n", [(1, 1), (256, 1), (257, 2), (769, 1), (1030, 4), (2305, 2), (8192, 2)])
def test_a_piece_waits_only_for_pieces_before_it(host, n, tiles_n):
    pieces, needs = _pieces(host, n, tiles_n)
    there = [f for f in pieces if f]
    assert len(set(there)) == len(there) == host.flow_host_expected(n) * tiles_n
    rows = {f[:3] + (f[4],): 0 for f in there}
    for f in there:
        rows[f[:3] + (f[4],)] += 1
    blocks = (n + 255) // 256
    for (back, is_sum, p, _), count in rows.items():
        i = blocks - 1 - p if back else p
        assert count == (min(n - 256 * i, 256) + 15) // 16
    assert all(w < i for i, want in enumerate(needs) for w in want)


def _two_launches(needs, search):
    """Two launches on two streams, 8 XCDs with room for 8 workgroups each.  An XCD starts its share of either launch in order, but
    whose turn it is differs: half of them begin with the one, half with the other.  Whether both launches end.  Without `search`
    a workgroup waits for as long as it takes; with it, as the kernel does, one that waits in vain gives its piece back and takes
    the first one up to its own that nobody has."""
    count = len(needs)
    done, claimed = [set(), set()], [set(), set()]
    starts = [[list(range(x, count, 8)) for x in range(8)] for _ in range(2)]
    there = [[] for _ in range(8)]  # per XCD: [launch, workgroup, piece]
    while True:
        moved = False
        for x in range(8):
            for launch in (0, 1) if x < 4 else (1, 0):
                while len(there[x]) < 8 and starts[launch][x]:
                    wg = starts[launch][x].pop(0)
                    if wg not in claimed[launch]:  # (else another workgroup has it)
                        claimed[launch].add(wg)
                        there[x].append([launch, wg, wg])
                    moved = True
            for w in list(there[x]):
                launch, wg, piece = w
                if not all(q in done[launch] for q in needs[piece]):
                    continue
                done[launch].add(piece)
                moved = True
                if piece == wg:
                    there[x].remove(w)
                else:
                    left = [q for q in range(wg + 1) if q not in claimed[launch]]
                    if left:
                        claimed[launch].add(left[0])
                        w[2] = left[0]
                    else:
                        there[x].remove(w)
        if len(done[0]) == len(done[1]) == count:
            return True
        if not moved:
            if not search:
                return False
            for x in range(8):
                for w in there[x]:
                    launch, wg, piece = w
                    claimed[launch].discard(piece)
                    w[2] = next(q for q in range(wg + 1) if q not in claimed[launch])
                    claimed[launch].add(w[2])
                    moved |= w[2] != piece
            if not moved:
                return False


@pytest.mark.parametrize("n,tiles_n", [(1280, 1), (2048, 2), (1000, 4)])
def test_two_launches_that_keep_each_other_from_starting_both_end(host, n, tiles_n):
    _, needs = _pieces(host, n, tiles_n)
    assert not _two_launches(needs, search=False)
    assert _two_launches(needs, search=True)
