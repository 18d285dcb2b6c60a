"""The tiled int8-activation kernel (qgemm_a8 on many rows) against the oracle's int8 leg, at the
edges of its tiles: row counts around 128, strips that leave wavefronts idle, one to several chunks,
every code width and scale group, forced K-slabs, sums at the ends of their range, and many groups.  Tolerance as for every int8 case (see test_gpu_a8.py); the
one-hot test there runs this kernel too (256 rows)."""
import numpy as np
import pytest
import torch

from paper_2504_12984_amd import workloads as WL
from gpu_util import assert_c_close, bits_of
from test_gpu_a8 import A8Case, _case, _reset_knobs, I, U  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N", [(65, 128, 64), (127, 256, 320), (128, 384, 256), (129, 1024, 192), (257, 640, 576)])
@pytest.mark.parametrize("bits", range(1, 9))
def test_tile_edges(bits, M, K, N):
    from paper_2504_12984_amd import binding as B
    B.qg_set_knob(0, 2)
    kind, group = (U, I)[(bits + M) % 2], {0: 128, 1: 64, 2: K}[(bits + N // 64) % 3]
    zero = "random" if (bits + K // 128) % 3 else None
    P = A8Case(_case(f"a8l_{bits}_{M}", M, K, N, kind, bits, group, act="f16" if M % 2 else "bf16", zero=zero, zero_hi=255, seed=41000 + M + bits))
    got = P.gpu()
    assert_c_close(got, P.ref(), P.case.name)
    assert np.array_equal(bits_of(got), bits_of(P.gpu()))


@pytest.mark.parametrize("splitk", [2, 3, 7])
@pytest.mark.parametrize("bits,group", [(4, 128), (8, 64), (5, 256), (3, 1792)])
def test_forced_slabs(splitk, bits, group):
    from paper_2504_12984_amd import binding as B
    B.qg_set_knob(0, 2); B.qg_set_knob(1, splitk)
    P = A8Case(_case(f"a8l_split_{bits}_{splitk}", 200, 1792, 320, U, bits, group, seed=41100 + bits))
    got = P.gpu()
    assert_c_close(got, P.ref(), P.case.name)
    assert np.array_equal(bits_of(got), bits_of(P.gpu()))


@pytest.mark.parametrize("bits", [1, 4, 8])
@pytest.mark.parametrize("a,code,zero", [(-128, "max", 0), (-128, "min", 255), (127, "max", 255)])
def test_sums_at_the_ends_of_their_range(bits, a, code, zero):
    # a chunk's sum reaches 128 * 128 * 2^(bits-1) * 2^(8-bits) = 2^21, a row sum 2^14 per chunk
    case = _case(f"a8l_ends_{bits}", 130, 512, 128, U, bits, 256, act="bf16", zero=None, seed=41200)
    inp = WL.make_inputs(case)
    inp["A"][:] = a
    inp["codes"][:] = (1 << bits) - 1 if code == "max" else 0
    inp["zeros"] = np.full((2, 128), zero, dtype=np.uint8)
    P = A8Case(case, inp)
    P.B.qg_set_knob(0, 2)
    assert_c_close(P.gpu(), P.ref(), case.name)


def test_more_rows_than_one_launch_takes():
    # 1024 groups; one launch here (test_gpu_a8_zero_points.py has a test of the same name that needs two)
    case = _case("a8l_blocks", 2051, 65536, 64, U, 2, 64, seed=41300)
    P = A8Case(case)
    rows = np.array([0, 1, 2046, 2047, 2048, 2049, 2050])
    assert_c_close(P.gpu()[torch.from_numpy(rows).cuda()], P.ref(rows=rows), case.name)


def test_capture_without_a_workspace_falls_back():
    # a stream that has no workspace yet may be under capture: nothing may be allocated there
    case = _case("a8l_capture", 256, 256, 128, U, 4, 128, seed=41400)
    P = A8Case(case)
    want = P.gpu()
    out = torch.zeros_like(want)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        call = P.B.BoundQgemmA8(P.d_A, P.d_as, P.d_packed, P.d_scales, P.d_zeros, P.wtype, case.group, case.N, out)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            call()
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert_c_close(out, P.ref(), case.name)
