"""Tiled kernels, K in slabs, tile height forced to 128: a last row tile of more than 64 rows is a 128-row tile with rows past M (of up to 64 rows
it is a 64-row one: test_gpu_tiled_slabs.py, test_gpu_a8_row_tiles.py).  Alone and behind another, one row past the half, one short of a
whole; slabs that meet in the kernel and, from four on, in a second one.  Inputs, references and tolerances are those two files'."""
import pytest

import test_gpu_a8_row_tiles as a8
import test_gpu_tiled_slabs as f16

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _reset_knobs():
    yield
    from paper_2504_12984_amd import binding as B
    for k in range(4):
        B.qg_set_knob(k, 0)


@pytest.mark.parametrize("splitk", [2, 3, 4, 6])
@pytest.mark.parametrize("M", [65, 100, 200, 255])
def test_slabs_of_whole_row_tiles(M, splitk):
    f16.test_slabs_meet(128, M, splitk)


@pytest.mark.parametrize("splitk", [2, 3, 5, 8])
@pytest.mark.parametrize("M", [65, 100, 200, 255])
@pytest.mark.parametrize("kind,bits,zeros", [("u", 4, "in"), ("i", 8, None), ("u", 7, "beyond")])
def test_slabs_of_whole_row_tiles_int8(kind, bits, zeros, M, splitk):
    a8.test_row_tiles_and_slabs(kind, bits, zeros, 128, M, splitk)
