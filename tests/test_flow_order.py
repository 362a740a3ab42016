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
