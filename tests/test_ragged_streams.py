"""The streams of a ragged batch, without a GPU: the library's host code runs
over a recording stand-in for the HIP runtime (fake_hip.cpp), and what ran on a
fork stream has to be joined back into the caller's stream, also when a later
call of the sequence fails: the caller frees or reuses its buffers in the order
of its own stream."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2606_06386_amd", "libmpdiv.so")
CALLER = "0x5000"

CALL = """
import ctypes, sys
ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
L = ctypes.CDLL(sys.argv[2])
p, n = ctypes.c_void_p(16), ctypes.c_int64(1 << 20)
args = [p, n, p, n, p, p, n, p, n, p, ctypes.c_int32(int(sys.argv[4]))]
args += [p] if sys.argv[3] == "mp_divrem_ragged" else []
status = getattr(L, sys.argv[3])(*args, ctypes.c_void_p(%s))
ctypes.CDLL(None).fflush(None)
print("status", status)
""" % CALLER


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake") / "libfakehip.so")
    subprocess.run(["g++", "-shared", "-fPIC", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-o", so,
                    os.path.join(ROOT, "tests", "fake_hip.cpp")], check=True, timeout=120)
    return so


def _calls(fake, entry="mp_divrem_ragged", count=4096, **env):
    """(status, [(what, stream, event, ok, kernel)]) of one call"""
    out = subprocess.run([sys.executable, "-c", CALL, fake, LIB, entry, str(count)], capture_output=True, text=True,
                         timeout=60, env={**os.environ, **env}, check=True).stdout.splitlines()
    calls, kernel = [], None
    for line in out[:-1]:
        if line.startswith("#"):
            what, a, b, ok = line[1:].split()
            calls.append((what, a, b, ok == "ok", kernel))
        kernel = None if line.startswith("#") else line
    assert out[-1].startswith("status ")
    return int(out[-1].split()[1]), calls


def _unjoined(calls):
    """fork streams with work that no later event of theirs brings back to the caller's stream"""
    left = set()
    for i, (what, s, e, ok, _) in enumerate(calls):
        if s == CALLER or not ok or what not in ("launch", "wait"):
            continue
        done = [j for j, c in enumerate(calls) if j > i and c[0] == "record" and c[1] == s and c[3]]
        if not any(c[0] == "wait" and c[1] == CALLER and c[2] == calls[j][2] and c[3]
                   for j in done for c in calls[j + 1:]):
            left.add(s)
    return left


def test_class_kernels_fork_and_join(fake):
    status, calls = _calls(fake)
    assert status == 0
    launches = [c for c in calls if c[0] == "launch"]
    assert len(launches) == 5 and len({c[1] for c in launches}) == 4 and launches[0][1] == CALLER
    assert not _unjoined(calls)


def test_forks_are_joined_when_a_call_fails(fake):
    """Each launch, attribute call and wait of the sequence fails in turn (a
    record that fails leaves nothing to wait for)."""
    _, good = _calls(fake)
    for n, (what, s, *_rest) in enumerate(good, 1):
        if what == "record":
            continue
        status, calls = _calls(fake, FAKE_HIP_FAIL=str(n))
        assert status == 3, (n, what, status)
        if not (what == "wait" and s == CALLER):          # (the join itself)
            assert not _unjoined(calls), f"call {n} ({what} on {s}) fails: {_unjoined(calls)} not joined"


@pytest.mark.parametrize("entry,count,env,kernels", [
    ("mp_divrem_ragged", 512, {}, 1), ("mp_divrem_ragged", 513, {"FAKE_HIP_CAPTURE": "1"}, 5),
    ("mp_divrem_ragged_static", 512, {}, 1), ("mp_divrem_ragged_static", 513, {}, 5)])
def test_batches_that_stay_on_the_callers_stream(fake, entry, count, env, kernels):
    """One launch up to two instances per compute unit (of 256); and in order on
    the caller's stream without a workspace, or if it is captured before the
    library has seen it."""
    status, calls = _calls(fake, entry, count, **env)
    assert status == 0 and {c[0] for c in calls} == {"attribute", "launch"}
    launches = [c for c in calls if c[0] == "launch"]
    assert len(launches) == kernels and {c[1] for c in launches} == {CALLER}
    assert ("k_ragged_direct" in launches[0][4]) == (kernels == 1)
