"""K-slabs of the streaming kernels meeting in a tree of exchanges: even and odd numbers of slabs, every
number of sums per thread, calls of other shapes in between (the slots have to be empty again), sums that are
infinite or not a number, and a captured graph.  Tolerance: see test_gpu_tiled_slabs.py."""
import numpy as np
import pytest
import torch

from paper_2504_12984_amd import workloads as WL
from gpu_util import Prepared, assert_c_close, bits_of
from test_gpu_a8 import A8Case, _case
from test_gpu_tiled_slabs import _check, _reset_knobs  # noqa: F401

pytestmark = pytest.mark.gpu


def _knobs(*values):
    from paper_2504_12984_amd import binding as B
    for k, v in enumerate(values):
        B.qg_set_knob(k, v)


@pytest.mark.parametrize("M,variants", [(1, (10, 11, 12, 14, 15, 16)), (16, (10, 11, 12, 14, 15, 16)), (17, (21, 26)), (32, (21, 26))])
def test_every_arrangement_and_number_of_slabs(M, variants):
    case = WL.Case(f"tree_{M}", M, 2432, 256, WL.KIND_UINT, 3, group=128, act="f16" if M % 2 else "bf16",
                   scale_dtype="f16", zero=3, seed=54000 + M)
    P = Prepared(case)
    for variant in variants:
        for splitk in (2, 3, 5, 8, 19):
            _knobs(1, splitk, 0, variant)
            first = P.gpu_c()
            _check(P, first, f"{case.name} {variant} in {splitk}")
            assert np.array_equal(bits_of(first), bits_of(P.gpu_c())), (variant, splitk)


def test_more_slots_than_the_workspace_has():
    # forced slabs: slots where the partial sums of other calls lie, cleared ahead of the kernel
    from paper_2504_12984_amd import binding as B
    P = Prepared(WL.Case("tree_many", 32, 2048, 8192, WL.KIND_UINT, 4, group=128, zero=8, seed=54050))
    Q = Prepared(WL.Case("tree_few", 16, 8192, 512, WL.KIND_UINT, 4, group=128, zero=8, seed=54051))
    R = Prepared(WL.Case("tree_tiles", 200, 8192, 512, WL.KIND_UINT, 4, group=128, zero=8, seed=54052))      # leaves partial sums behind
    a8 = A8Case(_case("a8_tree_many", 32, 2048, 8192, WL.KIND_UINT, 4, 128, zero=8, seed=54053))
    others = [bits_of(Q.gpu_c()), bits_of(R.gpu_c())]
    out = torch.empty(32, 8192, dtype=torch.float16, device="cuda")
    for splitk in (5, 16):
        _knobs(0, splitk)
        _check(P, P.gpu_c(), f"{splitk} slabs")
        assert_c_close(a8.gpu(), a8.ref(), a8.case.name)
        B.qgemm_noalloc(P.d_A, P.d_packed, P.d_scales, P.d_zeros, P.wtype, 128, 8192, out)
        assert np.array_equal(bits_of(out), bits_of(P.gpu_c()))
        _knobs(0, 0)
        for X, want in zip((Q, R), others):
            assert np.array_equal(bits_of(X.gpu_c()), want)


def test_automatic_splits_and_other_shapes_in_between():
    cases = [Prepared(WL.Case(f"tree_auto_{i}", M, K, N, WL.KIND_INT, b, group=128, zero=None, seed=54100 + i))
             for i, (M, K, N, b) in enumerate([(1, 4096, 512, 3), (16, 8192, 128, 4), (5, 2048, 1024, 8), (32, 4096, 192, 4), (64, 4096, 512, 4)])]
    want = [bits_of(P.gpu_c()) for P in cases]
    for P in cases:
        _check(P, P.gpu_c(), P.case.name)
    for _ in range(3):
        for P, w in zip(cases, want):
            assert np.array_equal(bits_of(P.gpu_c()), w), P.case.name


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf")])
def test_sums_that_are_not_finite(bad):
    P = Prepared(WL.Case("tree_nan", 7, 1024, 128, WL.KIND_UINT, 4, group=128, zero="random", seed=54200))
    _knobs(1, 1)
    clean = bits_of(P.gpu_c())
    A = P.d_A.clone()
    A[3, 900] = bad
    A.view(torch.int16)[5, 10] = -1                        # every bit set: a NaN of either format
    want = P.gpu_c(A).float().cpu()
    for splitk in (2, 4):
        _knobs(1, splitk)
        got = P.gpu_c(A).float().cpu()
        assert torch.equal(torch.isnan(got), torch.isnan(want)) and torch.equal(torch.isposinf(got), torch.isposinf(want))
        assert torch.equal(torch.isneginf(got), torch.isneginf(want))
        again = P.gpu_c()
        _check(P, again, "after")
        rows = [0, 1, 2, 4, 6]
        assert np.array_equal(bits_of(got.half())[rows], bits_of(again)[rows])      # the other rows are untouched
    _knobs(1, 1)
    assert np.array_equal(bits_of(P.gpu_c()), clean)


@pytest.mark.parametrize("M", [1, 16, 31, 64])
@pytest.mark.parametrize("splitk", [2, 3, 7])
def test_int8_activations(M, splitk):
    for K in (896, 2432):                                  # four and eight wavefronts per strip
        P = A8Case(_case(f"a8_tree_{M}_{splitk}", M, K, 192, WL.KIND_UINT, 5, 128, zero=9, seed=54300 + M))
        _knobs(3, splitk)
        got = P.gpu()
        assert_c_close(got, P.ref(), P.case.name)
        assert np.array_equal(bits_of(got), bits_of(P.gpu()))


def test_in_a_captured_graph():
    from paper_2504_12984_amd import binding as B
    P = Prepared(WL.Case("tree_graph", 16, 8192, 512, WL.KIND_UINT, 4, group=128, zero=8, seed=54400))
    assert B.qg_plan(P.wtype, 128, 16, 512, 8192)["splitk"] > 1
    side, out = torch.cuda.Stream(), torch.empty(16, 512, dtype=torch.float16, device="cuda")
    call = lambda: B.qgemm(P.d_A, P.d_packed, P.d_scales, P.d_zeros, P.wtype, 128, 512, out=out)      # noqa: E731
    with torch.cuda.stream(side):
        call()
    torch.cuda.synchronize()
    want = bits_of(out)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        call()
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(bits_of(out), want)
        assert np.array_equal(bits_of(P.gpu_c()), want)    # eager work between the replays
