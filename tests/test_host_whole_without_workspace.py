"""Calls of the tiled kernels for which no workspace is to be had (no memory, a capturing stream): those that the first fit of the
plan left whole run whole, whatever today's fit would split; the others stay refused; int8 calls never need one."""
import pytest

from test_host_workspace import _kernels, _run, stub  # noqa: F401

NONE = {"no_memory": "stub.stub_set(1, 0, 0)", "capture": "stub.stub_set(0, 1, 0)"}


@pytest.mark.parametrize("state", list(NONE))
def test_calls_that_were_left_whole_run_whole(stub, state):  # noqa: F811
    calls = "out = [linear(200, 5120, 13824), linear(160, 4096, 14336), codebook(1024, 4096, 4096, 8)]"
    for c in _run(stub, NONE[state] + "\n" + calls):
        assert c["rc"] == 0 and c["memset"] == [] and _kernels(c)[-1] == "large_kernel", c      # (ahead of it: de-quantised where its buffer was to be had)
    assert any(c["malloc"] for c in _run(stub, calls)[:2])                  # split where there is a workspace


@pytest.mark.parametrize("state", list(NONE))
def test_calls_that_were_split_stay_refused(stub, state):  # noqa: F811
    for c in _run(stub, NONE[state] + "\nout = [linear(300, 8192, 8192), linear(128, 8192, 2048), linear(64, 8192, 28672)]"):
        assert c["rc"] == -3 and c["launches"] == [], c


@pytest.mark.parametrize("state", list(NONE))
def test_int8_rows_beyond_one_block(stub, state):  # noqa: F811
    for c in _run(stub, NONE[state] + "\nout = [a8(M, 8192, 8192) for M in (65, 70, 96, 300)]"):
        assert c["rc"] == 0 and set(_kernels(c)) == {"a8_large_kernel"}, c
