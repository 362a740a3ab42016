"""What a call submits, and in which order the streams and events let it run (host only: a stand-in for the HIP runtime writes
the calls down; nothing is launched)."""
import json
import subprocess
import sys
from pathlib import Path

import pytest

from paper_2309_07235_amd import build

HERE = Path(__file__).resolve().parent
F64, F32 = 0, 1

# Run in a process of its own, without torch: the stand-in has to be there before the library's own runtime.
DRIVER = r"""
import ctypes, json, sys, threading
rec = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
vp, i64, ci, sz = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int, ctypes.c_size_t
class Gemm(ctypes.Structure):
    _fields_ = [(f, ci) for f in ("tile_m", "tile_n", "tile_k", "unroll_k", "wave_m", "wave_n")]
class Params(ctypes.Structure):
    _fields_ = [("nb", ci), ("lookahead", ci), ("update", Gemm), ("defer_min_rows", ci)]
lib.factor_workspace_bytes.argtypes, lib.factor_workspace_bytes.restype = [i64, ci, vp], sz
for f in (lib.lu_factor, lib.cholesky_factor):
    f.argtypes = [vp, i64, i64, ci, ctypes.POINTER(Params), vp, sz, vp, vp]
lib.dla_factor_giveup_selftest.argtypes = [ci, vp, i64, i64, ci, vp, sz, vp, vp]
lib.solve_workspace_bytes.argtypes, lib.solve_workspace_bytes.restype = [i64, i64, ci], sz
lib.lu_solve.argtypes = [vp, i64, i64, vp, i64, i64, ci, vp, sz, vp]
rec.record_text.restype = ctypes.c_char_p
def call(kind, dtype, n, nb=0, lookahead=-1, info=True, stream=0x77, giveup=False, nrhs=0):
    if nrhs:
        return lib.lu_solve(0x10000000000, n, n, 0x100000000, nrhs, nrhs, dtype, 0x20000000000, lib.solve_workspace_bytes(n, nrhs, dtype), stream)
    ws = lib.factor_workspace_bytes(n, dtype, None)
    data, scratch, status = 0x100000000, 0x200000000, 0x300000000 if info else None
    if giveup:
        return lib.dla_factor_giveup_selftest(int(kind != "lu"), data, n, n, dtype, scratch, ws, stream, status)
    f = lib.lu_factor if kind == "lu" else lib.cholesky_factor
    return f(data, n, n, dtype, Params(nb, lookahead, Gemm(), 0), scratch, ws, stream, status)
job = json.loads(sys.argv[3])
out = []
for threads in job["runs"]:  # each a list of threads, each a list of calls
    rec.record_start(ci(job.get("pause", 0)))
    rcs = [[] for _ in threads]
    def work(t):
        rec.record_thread(ci(t))
        for c in threads[t]:
            rcs[t].append(call(**c))
    ts = [threading.Thread(target=work, args=(t,)) for t in range(len(threads))]
    for t in ts: t.start()
    for t in ts: t.join()
    out.append({"rc": rcs, "text": rec.record_text().decode()})
print(json.dumps(out))
"""


@pytest.fixture(scope="module")
def record(tmp_path_factory):
    so = tmp_path_factory.mktemp("rec") / "librecorder.so"
    subprocess.run(["g++", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-std=c++17", "-O1", "-w", "-shared", "-fPIC", "-pthread",
                    str(HERE / "host" / "hip_recorder.cpp"), "-o", str(so)], check=True)

    def run(runs, pause=0):
        """Per run the calls' return codes and the list of (thread, what, stream, event, workgroups, kernel)."""
        res = subprocess.run([sys.executable, "-c", DRIVER, str(so), str(build.LIB), json.dumps({"runs": runs, "pause": pause})],
                             capture_output=True, text=True, timeout=100, check=True)
        out = []
        for r in json.loads(res.stdout):
            rows = [line.split(" ") for line in r["text"].splitlines()]
            out.append((r["rc"], [(int(t), w, st, ev, int(g), k) for t, w, st, ev, g, k in rows]))
        return out

    return run


def _behind(ops):
    """Per operation the set (bits) of launches that are complete before it starts, and that for the end of each stream."""
    done, events, before = {}, {}, []
    for i, (_, what, st, ev, _, _) in enumerate(ops):
        now = done.get(st, 0)
        before.append(now)
        if what == "W":
            done[st] = now | events.get(ev, 0)
        elif what == "L":
            done[st] = now | 1 << i
            if ev != "0":
                events[ev] = done[st]
        elif what == "R":
            events[ev] = now
    return before, done


def _call(kind, dtype, n, **more):
    return {"kind": kind, "dtype": dtype, "n": n, **more}


# every form: one block, one stream, both pipelines, tiles, and tails of tiles behind an even and an odd number of block steps
# (a step that carries two panels is then the last one, or is not)
FORMS = [_call(kind, dtype, n, **more) for kind, dtype in (("lu", F64), ("lu", F32), ("chol", F64), ("chol", F32))
         for n, more in [(100, {}), (600, {"lookahead": 0}), (600, {"info": False}), (5000, {"lookahead": 2}), (5000, {"nb": 256}), (600, {}),
                         (5000, {}), (7300, {}), (7400, {}), (7500, {}), (8000, {}), (8192, {})]]


def test_a_call_joins_all_it_has_submitted(record):
    """Whatever the caller's stream runs next is behind every kernel of the call, and so is the launch that takes the last rows in
    tiles: it works in place on what the pipeline's kernels have left."""
    for form, (rc, ops) in zip(FORMS, record([[[f]] for f in FORMS])):
        assert rc == [[0]], form
        launches = sum(1 << i for i, o in enumerate(ops) if o[1] == "L")
        assert launches, form
        before, done = _behind(ops)
        names = lambda bits: sorted({ops[i][5] for i in range(len(ops)) if bits >> i & 1})
        assert done["77"] & launches == launches, (form, names(launches & ~done["77"]))
        for i, o in enumerate(ops):
            if o[1] == "L" and "tile_" in o[5]:
                rest = sum(1 << j for j in range(i) if ops[j][1] == "L" and "tile_" not in ops[j][5])
                assert before[i] & rest == rest, (form, o[5], names(rest & ~before[i]))


def test_calls_from_several_threads_line_up(record):
    """The helper streams and events are one set for the process: whatever the kinds and types of the calls, one has submitted all
    it has before the next begins to, starts behind it on the device, and the set is made once."""
    calls = [_call("lu", F64, 600), _call("chol", F64, 700), _call("lu", F32, 1500), _call("chol", F32, 6000), _call("lu", F64, 8000),
             _call("chol", F64, 900, lookahead=2), _call("lu", F32, 4000, giveup=True), _call("chol", F64, 1000, giveup=True)]
    (rc, ops), = record([[[c] for c in calls]], pause=200)
    assert rc == [[0]] * len(calls)
    turns = [t for i, (t, *_) in enumerate(ops) if i == 0 or ops[i - 1][0] != t]
    assert sorted(turns) == list(range(len(calls))), turns
    assert sum(o[1] == "S" for o in ops) == 3 and sum(o[1] == "E" for o in ops) == 8
    before, _ = _behind([(t, w, st if st != "77" else f"77 of {t}", ev, g, k) for t, w, st, ev, g, k in ops])  # a stream per thread
    for a, t in enumerate(turns[1:]):
        first = next(i for i, o in enumerate(ops) if o[0] == t and o[1] == "L")
        rest = sum(1 << i for i, o in enumerate(ops) if o[0] == turns[a] and o[1] == "L")
        assert before[first] & rest == rest, (calls[turns[a]], calls[t])


def test_what_waits_for_each_other_is_one_launch(record):
    """The tiles' workgroups wait for the diagonal's and it for theirs: in two launches they would need two hardware queues, and
    streams share a few.  They are one launch, on the caller's stream, behind the one that clears their flags."""
    tiled = 0
    for form, (_, ops) in zip(FORMS, record([[[f]] for f in FORMS])):
        tiles = [o for o in ops if o[1] == "L" and "tile_" in o[5]]
        assert all(o[2] == "77" for o in tiles), (form, tiles)
        assert not tiles or (len(tiles) == 2 and "tile_clear_kernel" in tiles[0][5] and "tile_factor_kernel" in tiles[1][5]), (form, tiles)
        tiled += bool(tiles)
    assert tiled == 4 * 7


@pytest.mark.parametrize("kind", ["lu", "chol"])
@pytest.mark.parametrize("dtype,most", [(F64, 8192), (F32, 8000)])
def test_block_size_64_is_the_tiles_up_to_a_size(record, kind, dtype, most):
    """The line that the header states, on both sides; the diagnostic of the tiles' waits has the same."""
    runs = record([[[_call(kind, dtype, n, **more)]] for more in ({"nb": 64}, {"giveup": True}) for n in (most, most + 1)])
    tiled = [any("tile_factor_kernel" in o[5] for o in ops) for _, ops in runs]
    assert tiled == [True, False, True, False]
    assert [rc for rc, _ in runs] == [[[0]], [[0]], [[0]], [[1 if dtype == F64 else 2]]]  # (DLA_ERR_UNSUPPORTED_PARAMS; DLA_ERR_WORKSPACE)


@pytest.mark.parametrize("nrhs,most", [(64, 683 * 256), (1, 1366 * 256)])
def test_one_launch_of_passes_as_long_as_its_claims_have_room(record, nrhs, most):
    """fp32: the flags and claims of flow_kernel lie in the 512 KiB of the first block's M; a system beyond takes the launches."""
    runs = record([[[_call("lu", F32, n, nrhs=nrhs)]] for n in (most, most + 1)])
    flows = [sum("flow_kernel" in o[5] for o in ops) for _, ops in runs]
    assert flows == [1, 0] and all(rc == [[0]] for rc, _ in runs)
    assert sum(o[1] == "L" for o in runs[0][1]) == 4  # three of the pre-pass in front of it
