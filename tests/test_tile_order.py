"""The order in which tile_factor_kernel's workgroups take their tiles, on the host."""
import ctypes
import subprocess
from pathlib import Path

import numpy as np
import pytest

from paper_2309_07235_amd import build

HERE = Path(__file__).resolve().parent
LU, CHOL = 0, 1


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    so = tmp_path_factory.mktemp("tile") / "libtile_host.so"
    subprocess.run([build.HIPCC, "--offload-arch=gfx950", "--cuda-host-only", "-std=c++17", "-O1", "-shared", "-fPIC", "-w", "-I",
                    str(build.CSRC), str(HERE / "host" / "tile_host.hip"), "-o", str(so)], check=True)
    return ctypes.CDLL(str(so))


def _order(host, kind, nt):
    i, j = (np.full(nt * nt, -1, dtype=np.int32) for _ in range(2))
    ints = ctypes.POINTER(ctypes.c_int)
    count = host.tile_host_order(kind, nt, i.ctypes.data_as(ints), j.ctypes.data_as(ints))
    return list(zip(i[:count].tolist(), j[:count].tolist()))


@pytest.mark.parametrize("kind", [LU, CHOL])
def test_every_tile_once(host, kind):
    for nt in range(2, host.tile_host_max() + 1):
        order = _order(host, kind, nt)
        want = {(i, j) for i in range(nt) for j in range(nt if kind == LU else i + 1)} - {(0, 0)}
        assert len(order) == len(want) and set(order) == want


def _runs_through(order, kind, nt, ring, workers):
    """Whether a factorisation ends with so many workgroups beside workgroup 0.  What each waits for is what the kernel's
    workgroups wait for; nothing that is done is undone, so one order of doing what can be done stands for all."""
    up = (lambda k, j: (k, j)) if kind == LU else (lambda k, j: (j, k))  # the right operand of a product
    solved, copied, read, diag, taken = set(), set(), {}, 0, 0           # diag: blocks published
    held = []                                                            # [tile, whether it waits for its diagonal block]
    while True:
        moved = False
        if diag < nt:  # workgroup 0: block `diag` is published once the blocks beside the next one are there, and a place in the ring
            s = diag
            need = {(s + 1, s), (s + 1, s + 1)} | ({(s, s + 1)} if kind == LU else set()) if s + 1 < nt else set()
            gone = s + 1 - ring
            free = gone < 0 or s + 1 >= nt or read.get(gone, 0) >= (2 if kind == LU else 1) * (nt - 1 - gone)
            if need <= copied and free:
                diag += 1
                moved = True
        while len(held) < workers and taken < len(order):
            held.append([order[taken], False])
            taken += 1
            moved = True
        for h in list(held):
            (i, j), waits = h
            s = min(i, j)
            if not waits:
                depth = s - 1 if i == j else s
                if any((i, k) not in solved or up(k, j) not in solved for k in range(depth)):
                    continue
                if i == j or abs(i - j) == 1:
                    copied.add((i, j))
                h[1] = moved = True
            if i == j:
                held.remove(h)
            elif diag > s:
                read[s] = read.get(s, 0) + 1
                solved.add((i, j))
                held.remove(h)
                moved = True
        if diag == nt and taken == len(order) and not held:
            return True
        if not moved:
            return False


@pytest.mark.parametrize("kind,workers", [(LU, 3), (CHOL, 2)])
@pytest.mark.parametrize("nt", [2, 3, 4, 17, 18, 40])
def test_few_workgroups_are_enough(host, kind, workers, nt):
    """However few of them the other work on the card lets run: no workgroup waits for one that has not started."""
    order, ring = _order(host, kind, nt), host.tile_host_ring()
    assert _runs_through(order, kind, nt, ring, workers) and _runs_through(order, kind, nt, ring, 255)
