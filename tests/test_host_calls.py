"""What the library asks of the HIP runtime, seen by a stand-in without a device.

A child process loads ``fakes/hip_runtime.c`` in front of the library, builds
and solves small batches (no kernel runs) and prints the runtime calls.
"""
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))

CHILD = """
import ctypes as C, os, sys
C.CDLL(sys.argv[1], mode=os.RTLD_GLOBAL | os.RTLD_NOW)
sys.path.insert(0, sys.argv[2])
import numpy as np
from paper_2309_06427_amd import _lib
L = _lib.load()
mem = 4096  # no pointer is followed
stream = 0x5000
for dev, sizes, prec, pc in eval(sys.stdin.read()):
    N, nx = (np.array(v, dtype=np.int32) for v in zip(*sizes))
    p = lambda a: a.ctypes.data_as(C.POINTER(C.c_int32))
    h = C.c_void_p()
    assert L.ssp_batch_create(len(N), p(N), p(nx), p(nx // 2), dev, C.byref(h)) == 0
    assert L.ssp_build(h, pc, prec, mem, mem, mem, mem, mem, stream) == 0
    C.CDLL(None).fflush(None)
    print("solve", flush=True)
    assert L.ssp_solve(h, 1e-6, 0, mem, mem, 0, mem, mem, mem, stream) == 0
    C.CDLL(None).fflush(None)
    print("end", flush=True)
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    cc = shutil.which("gcc")
    if not cc or not os.path.isdir("/opt/rocm/include/hip"):
        pytest.skip("no gcc or no HIP headers")
    so = str(tmp_path_factory.mktemp("fake") / "fakehip.so")
    subprocess.run([cc, "-shared", "-fPIC", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(HERE, "fakes", "hip_runtime.c"), "-o", so], check=True)
    return so


def calls(fake, work):
    """The calls of each solve and, first, all calls in order, as lists of words."""
    r = subprocess.run([sys.executable, "-c", CHILD, fake, os.path.dirname(HERE)], input=repr(work),
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    lines = [l.split() for l in r.stdout.splitlines()]
    solves, cur = [], None
    for w in lines:
        if w[0] == "solve":
            cur = []
            solves.append(cur)
        elif w[0] == "end":
            cur = None
        elif cur is not None:
            cur.append(w)
    return lines, solves


FP64, REFINE = 0, 2
SYM = 2


def test_large_lds_is_allowed_on_each_device(fake):
    """A launch with more than 64 KiB of dynamic LDS needs the kernel's opt-in on the device it runs on."""
    sizes = [(60, 14), (50, 14), (40, 26), (90, 6), (30, 36)]
    lines, _ = calls(fake, [(d, sizes, p, SYM) for p in (REFINE, FP64) for d in (0, 1)])
    allowed, large = {}, 0
    for w in lines:
        if w[0] == "allow":
            allowed[w[1], w[2]] = int(w[3])
        elif w[0] == "launch" and int(w[3]) > 64 * 1024:
            large += 1
            assert allowed.get((w[1], w[2]), 0) >= int(w[3]), w
    assert large >= 8


def test_internal_streams_fork_from_and_join_into_the_callers(fake):
    """Internal streams wait for events of the caller's stream alone and only the caller's stream waits for theirs (a
    capture cannot end where they join each other); each that launches is joined after its last launch."""
    _, (calls_,) = calls(fake, [(0, [(400, 26), (30, 26), (700, 14), (90, 6), (30, 36)], REFINE, SYM)])
    caller, recorded, open_ = "0x5000", {}, set()
    launches = [w[4] for w in calls_ if w[0] == "launch"]
    assert len(set(launches)) == 5
    for w in calls_:
        if w[0] == "record":
            recorded[w[1]] = w[2]
            if w[2] != caller:
                open_.discard(w[2])
        elif w[0] == "wait":
            src = recorded[w[2]]
            assert (w[1] == caller) != (src == caller), (w, src)
        elif w[0] == "launch" and w[4] != caller:
            open_.add(w[4])
    assert not open_
    waited = {recorded[w[2]] for w in calls_ if w[0] == "wait" and w[1] == caller}
    assert set(launches) - {caller} <= waited


def test_one_state_size_stays_on_the_callers_stream(fake):
    """Long problems and, where that pays, the others on chip after them: one stream, both kernels, all problems."""
    for sizes, blocks in (([(400, 26), (300, 26), (30, 26)], [256]), ([(769, 14)] + [(100, 14)] * 18000, [256, 512])):
        _, (calls_,) = calls(fake, [(0, sizes, REFINE, SYM)])
        assert {w[0] for w in calls_} <= {"launch", "allow"}
        solves = [w for w in calls_ if w[0] == "launch" and int(w[3]) > 0]
        assert [int(w[6]) for w in solves] == blocks and {w[4] for w in solves} == {"0x5000"}


def test_solves_ask_the_runtime_for_nothing_but_launches_after_the_first(fake):
    """Once a process has run a solve of a kind, further ones, also of new handles, make launches, event records and waits
    only, as a capture needs it."""
    some = [(60, 14), (40, 26), (90, 6), (30, 36)]
    work = [(0, sizes, p, SYM) for sizes in (some, some + [(20, 9)]) for p in (REFINE, FP64)]
    _, solves = calls(fake, work * 2)
    for first, again in zip(solves[:4], solves[4:]):
        assert {w[0] for w in again} == {"launch", "record", "wait"} and len(again) >= 7
        assert {w[0] for w in first} - {"allow"} == {"launch", "record", "wait"}
