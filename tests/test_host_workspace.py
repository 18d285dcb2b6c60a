"""Host code of the library without a GPU: what a call allocates, clears and launches, through a stand-in
for the HIP runtime (host_runtime_stub.cpp) in a process of its own."""
import json
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.environ.get("QGEMM_LIB") or os.path.join(ROOT, "paper_2504_12984_amd", "libqgemm.so")

PRELUDE = """
import ctypes as C, json, re, sys
stub, lib = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL), C.CDLL(sys.argv[2])
stub.stub_take_log.restype = lib.qg_last_error.restype = C.c_char_p
class T(C.Structure): _fields_ = [(n, C.c_int32) for n in ("kind", "bits", "ebits", "mbits")]
P, I, L = C.c_void_p, C.c_int, C.c_int64
lib.qgemm.argtypes = lib.qgemm_noalloc.argtypes = [P, P, P, P, T, I, I, I, L, L, L, L, P, P]
lib.qgemm_a8.argtypes = [P, P, P, P, P, T, I, I, L, L, L, L, P, P]
lib.qgemm_codebook.argtypes = [P, P, P, P, I, I, I, L, L, L, L, P, P]
A = 0x10000                                                    # any aligned address: nothing is read
def log(): return stub.stub_take_log().decode().splitlines()
LOADED = log()
def call(rc):
    lines = log()
    def ints(word): return [int(s.split()[1]) for s in lines if s.startswith(word + " ")]
    launches = [s.split()[1:] for s in lines if s.startswith("launch ")]
    kernel = lambda name: re.search("([a-z0-9]+(?:_[a-z0-9]+)*_kernel)", re.sub("^_ZN2qg[0-9]+", "", name)).group(1)
    return dict(rc=rc, malloc=ints("malloc"), memset=ints("memset"),
                launches=[(kernel(n), n, int(x), int(y)) for n, x, y, _ in launches])
def a8(M, K, N, kind=0, bits=4, zeros=True, group=128, stream=1):
    return call(lib.qgemm_a8(A, A, A, A, A if zeros else None, T(kind, bits, 0, 0), 0, 0, group, M, N, K, A, stream))
def linear(M, K, N, bits=4, group=128, stream=1, entry=None):
    return call((entry or lib.qgemm)(A, A, A, None, T(0, bits, 0, 0), 0, 0, 0, group, M, N, K, A, stream))
def codebook(M, K, N, bits, stream=1):
    return call(lib.qgemm_codebook(A, A, A, A, bits, 0, 0, 128, M, N, K, A, stream))
out = []
"""


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("stub") / "libstub.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "host_runtime_stub.cpp")], check=True)
    return so


def _run(stub, code):
    r = subprocess.run([sys.executable, "-c", PRELUDE + code + "\nprint(json.dumps(out))", stub, LIB], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    return json.loads(r.stdout)


def _kernels(call):
    return [k for k, *_ in call["launches"]]


def test_a_failed_allocation_does_not_fail_a_call_that_needs_none(stub):
    # eight-bit codebook, 1024 rows: no buffer for the de-quantised weight, so the fused kernel; then calls without a workspace
    calls = _run(stub, "stub.stub_set(1, 0, 0)\nout = [codebook(1024, 4096, 4096, 8), linear(16, 8192, 2048), linear(16, 4096, 28672)]")
    assert calls[0]["rc"] == 0 and calls[0]["malloc"] and _kernels(calls[0]) == ["large_kernel"], calls[0]
    assert calls[1]["rc"] == -3 and calls[1]["launches"] == []        # splits K: refused, nothing enqueued
    assert calls[2]["rc"] == 0 and _kernels(calls[2]) == ["decode_kernel"], calls[2]


def test_no_workspace_is_made_on_a_capturing_stream(stub):
    # not even where the capture mode allows it: the memset would be recorded, and the wait for a strip's other slabs
    # in the tiled kernel would read counters that nothing has cleared
    calls = _run(stub, "stub.stub_set(0, 1, 0)\nout = [linear(16, 8192, 2048), linear(300, 8192, 8192), linear(200, 8192, 2048)]")
    for c in calls:
        assert c["rc"] == -3 and c["malloc"] == [] and c["memset"] == [] and c["launches"] == [], c
    calls = _run(stub, "linear(16, 8192, 2048)\nstub.stub_set(0, 1, 0)\nout = [linear(16, 8192, 2048), linear(300, 8192, 8192)]")
    for c in calls:                                           # one eager call on the stream before: served
        assert c["rc"] == 0 and c["malloc"] == [] and c["memset"] == [] and c["launches"], c


@pytest.mark.parametrize("state", ["stub.stub_set(1, 0, 0)", "stub.stub_set(0, 1, 0)", "stub.stub_set(0, 1, 1)\nstub.stub_set(1, 0, 1)",
                                   "[linear(16, 8192, 2048, stream=16 * i + 160) for i in range(32)]"],
                         ids=["no_memory", "capture", "unanswered_query", "all_pairs_taken"])
def test_int8_calls_that_would_split_k_do_without_a_workspace(stub, state):
    # the tiled kernel alone, unsplit (the fourth template argument), whatever the blocks of 64 rows would have needed
    calls = _run(stub, state + "\nout = [a8(M, K, N, group=64) for M, K, N in ((1000, 8192, 2048), (300, 8192, 4096), (131200, 16384, 512))]")
    for c in calls:
        assert c["rc"] == 0 and c["memset"] == [] and set(_kernels(c)) == {"a8_large_kernel"}, c
        assert all("ELb0ELb0ELb1E" in name for _, name, _, _ in c["launches"]), c
    assert len(calls[2]["launches"]) == 2                     # two blocks of rows, the last one short
    calls = _run(stub, "out = [a8(M, K, N, group=64) for M, K, N in ((1000, 8192, 2048), (300, 8192, 4096))]")
    for c in calls:                                           # and split where a workspace is there
        assert c["rc"] == 0 and all("ELb0ELb1ELb1E" in name for _, name, _, _ in c["launches"]), c


def test_workspace_sizes(stub):
    # partial sums, counters, and slots for what the automatic plans split: fewer than 512 strips x slabs of 8 KiB
    size, cleared = (36 << 20) + 65536, (4 << 20) + 65536
    loaded, first, second = _run(stub, "out = [LOADED, linear(16, 8192, 2048), linear(32, 8192, 2048, entry=lib.qgemm_noalloc)]")
    assert [int(s.split()[2]) for s in loaded if "scratch" in s] == [size]
    assert first["malloc"] == [size] and first["memset"] == [cleared] and second["malloc"] == []
    most = max(c["launches"][0][2] * (c["launches"][0][3] - 1) for c in _run(
        stub, "out = [f(M, K, 64 * n) for f in (linear, a8) for M in (1, 17) for K in (2048, 4096, 8192, 16384) for n in (1, 8, 31, 63, 64, 127, 128, 129, 191, 255, 256)]"))
    assert 128 <= most < 512


@pytest.mark.parametrize("entry", ["lib.qgemm", "lib.qgemm_noalloc"])
def test_forced_slabs_beyond_the_slots_are_cleared_ahead_of_the_kernel(stub, entry):
    calls = _run(stub, "lib.qg_set_knob(1, 8)\nout = [linear(M, 8192, N, entry=%s) for M, N in ((16, 8192), (16, 16384), (32, 8192), (48, 16384))]" % entry)
    assert [_kernels(c) for c in calls] == [["decode_kernel"], ["clear_kernel", "decode_kernel"], ["clear_kernel", "decode_kernel"], ["decode_kernel"]]
    assert calls[1]["launches"][0][2] == 7 * 256 * 4096 // 16 // 256 and all(c["rc"] == 0 for c in calls)


def test_int8_calls_that_do_not_split_k_take_no_workspace(stub):
    # more tiles than a workspace has counters for, and more with every call: nothing to allocate
    calls = _run(stub, "out = [a8(200, 8192, 2048)] + [a8(M, 8192, 28672) for M in (1000, 4700, 4900, 9000)] + [a8(2400, 8192, 57344)]")
    assert len(calls[0]["malloc"]) == 1                       # this one splits K
    for c in calls[1:]:
        assert c["rc"] == 0 and c["malloc"] == [] and c["memset"] == [] and _kernels(c)[-1] == "a8_large_kernel", c


def test_a_forced_height_that_int8_tiles_do_not_have_changes_nothing(stub):
    calls = "[a8(M, K, N) for M, K, N in ((65, 8192, 28672), (300, 8192, 8192), (1000, 8192, 28672), (2000, 4096, 8192))]"
    got = _run(stub, f"out = {calls}\nlib.qg_set_knob(2, 256)\nout += {calls}\nlib.qg_set_knob(2, 64)\nout += {calls}")
    launches = [c["launches"] for c in got]
    assert launches[:4] == launches[4:8] and all(_kernels(c) == ["a8_large_kernel"] for c in got[1:4])
    assert all("Li64E" in n for c in got[9:] for _, n, _, _ in c["launches"])
