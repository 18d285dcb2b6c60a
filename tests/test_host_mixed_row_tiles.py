"""Host logic: which row tiles a call of the tiled kernels launches, and how many -- for the shapes of test_gpu_mixed_row_tiles.py and
test_gpu_cut_row_tiles.py, whose results are the same whatever the tiles.  The 16-bit kernel is forced (knob 0), as there.

A launch of 128-row tiles and 64-row ones has 8 * (ceil(full / 8) + ceil(half / 8)) workgroups: an XCD gets a run of either kind."""
import re

import pytest

from test_host_workspace import _run, stub  # noqa: F401


def _tiles(call):
    """[(row-tile height, workgroups)] of a call's launches of the tiled kernels"""
    assert call["rc"] == 0, call
    return [(int(re.search(r"large_kernelI(?:Li\d+E){2,3}?Li(64|128|256)E", n).group(1)), x) for k, n, x, _ in call["launches"]
            if k in ("large_kernel", "a8_large_kernel")]


def _grid(full, half=0):
    return 8 * ((full + 7) // 8 + (half + 7) // 8)


U = "T(0, %d, 0, 0)"


def _calls(stub, calls, path=2):
    return _run(stub, f"lib.qg_set_knob(0, {path})\nout = [" + ", ".join(calls) + "]")


def _qgemm(t, M, K, N, group=128, act=0, scale=0):
    return f"call(lib.qgemm(A, A, A, None, {t}, 0, {act}, {scale}, {group}, {M}, {N}, {K}, A, 1))"


# (columns, rows, 128-row tiles, 64-row tiles): a last row tile of 64 rows, halves of 128-row tiles, both
@pytest.mark.parametrize("N,M,full,half", [
    (16384, 257, 128, 64), (16448, 320, 130, 65), (16384, 600, 256, 128), (16448, 700, 256, 203), (16384, 705, 256, 256),
    (16448, 1100, 512, 146), (16384, 1600, 768, 64)])
def test_heights(stub, N, M, full, half):
    for t in (U % 3, U % 4, U % 5):
        c, = _calls(stub, [_qgemm(t, M, 256, N)])
        assert _tiles(c) == [(128, _grid(full, half))], _tiles(c)


def test_second_launch(stub):
    plain, cut = _calls(stub, [_qgemm("T(1, 4, 0, 0)", 1300, 8192, 16384), _qgemm("T(1, 4, 0, 0)", 769, 4096, 20480)])
    assert _tiles(plain) == [(256, _grid(252)), (128, _grid(220, 22))]
    assert _tiles(cut) == [(256, _grid(256)), (128, _grid(0, 208))]


# types with constants or LDS of their own: a 128-row tile and the 64 rows behind it both in 64-row tiles; two rounds of
# 128-row tiles and the last ones as halves
@pytest.mark.parametrize("N,M,full,half", [(16448, 129, 0, 195), (16448, 961, 512, 16)])
def test_cut_of_other_types(stub, N, M, full, half):
    calls = [_qgemm("T(2, 6, 3, 2)", M, 256, N), _qgemm("T(2, 5, 2, 2)", M, 256, N), _qgemm("T(2, 4, 2, 1)", M, 256, N, group=32, act=1, scale=2),
             _qgemm("T(2, 8, 4, 3)", M, 256, N, group=32, act=1, scale=2), _qgemm(U % 4, M, 256, N, group=32), _qgemm(U % 8, M, 256, N, group=32),
             f"codebook({M}, 256, {N}, 4)", f"codebook({M}, 256, {N}, 8)"]
    for c in _calls(stub, calls):
        assert _tiles(c) == [(128, _grid(full, half))], (c["launches"], _tiles(c))
    dense, = _calls(stub, [_qgemm(U % 5, M, 256, N)], path=4)
    assert _tiles(dense) == [(128, _grid(full, half))]


def test_e3m2_is_cut_as_the_types_with_a_quick_convert(stub):
    # M = 257, K = 8192, N = 28672: 146 us in tiles of 128 and 64 rows, 198 in 256-row ones, which e2m2 takes
    e2m1, e3m2, e4m3, e2m2 = _calls(stub, [_qgemm(f"T(2, {b}, {e}, {m})", 257, 8192, 28672) for b, e, m in ((4, 2, 1), (6, 3, 2), (8, 4, 3), (5, 2, 2))])
    assert _tiles(e3m2) == _tiles(e2m1) == _tiles(e4m3) == [(128, _grid(224, 112))]
    assert _tiles(e2m2) == [(256, _grid(224))]


def test_only_the_8_bit_table_leaves_a_cu_one_workgroup(stub):
    # M = 300, K = 8192, N = 28672, 6 bits: 208 us in tiles of 128 and 64 rows, 298 in 256-row ones; 8 bits: 311 and 286
    calls = _calls(stub, [f"codebook(300, 8192, 28672, {bits})" for bits in (5, 6, 7, 8)])
    assert [_tiles(c) for c in calls] == 3 * [[(128, _grid(224, 112))]] + [[(256, _grid(224))]]
    # bf16, M = 1000: 520 us in 256-row tiles, 550 with lower ones behind 64 columns of them
    bf16 = "call(lib.qgemm_codebook(A, A, A, A, 6, 1, 1, 128, %d, 28672, 8192, A, 1))"
    assert [_tiles(c) for c in _calls(stub, [bf16 % 300, bf16 % 1000])] == [[(128, _grid(224, 112))], [(256, _grid(448))]]


@pytest.mark.parametrize("N,M,full,half", [
    (16384, 257, 128, 64), (16448, 320, 130, 65), (16384, 600, 256, 128), (16448, 700, 256, 203), (16448, 1100, 512, 146), (16384, 1600, 768, 64)])
def test_heights_int8(stub, N, M, full, half):
    for bits in (4, 5, 8):
        c, = _calls(stub, [f"a8({M}, 256, {N}, bits={bits}, group={(64, 128)[M % 3 == 0]})"])
        assert _tiles(c) == [(128, _grid(full, half))], _tiles(c)
