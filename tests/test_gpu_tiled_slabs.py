"""K-slabs of the tiled kernel: two or three meet inside the kernel (the wavefront that arrives last
adds the others' sums to its own), four and more in a second kernel.  At the edges: rows past M in the last
tile, strips that leave wavefronts idle, a short odd last slab, both row tiles, rounding routes.

Tolerance: the sums are fp32, so |C - ref| <= u |ref| + K 2^-24 sum |a w| with u = 2^-11 (fp16) or 2^-8
(bf16) for the one rounding to the output type (and 2^-24 for fp16 results below its normal range)."""
import numpy as np
import pytest
import torch

from paper_2504_12984_amd import workloads as WL
from gpu_util import Prepared, bits_of, to_f64

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _reset_knobs():
    yield
    from paper_2504_12984_amd import binding as B
    for k in range(4):
        B.qg_set_knob(k, 0)


def _check(P, got, what):
    c = P.case
    W, _ = P.oracle_w()
    ref = P.A64 @ W
    u = 2.0 ** -11 if c.act == "f16" else 2.0 ** -8
    bound = u * np.abs(ref) + c.K * 2.0 ** -24 * (np.abs(P.A64) @ np.abs(W)) + 2.0 ** -24
    bad = np.argwhere(~(np.abs(to_f64(got) - ref) <= bound))
    assert len(bad) == 0, f"{what}: {len(bad)} outside, first at {tuple(bad[0])}"


@pytest.mark.parametrize("splitk", [2, 3, 4, 6, 9])
@pytest.mark.parametrize("bm,M", [(64, 1), (64, 65), (64, 200), (128, 130), (128, 257)])
def test_slabs_meet(bm, M, splitk):
    from paper_2504_12984_amd import binding as B
    act = "f16" if (splitk + M) % 2 else "bf16"
    case = WL.Case(f"slabs_{bm}_{M}_{splitk}", M, 2432, 320, WL.KIND_UINT, 4 + splitk % 3, group=(64, 128, 2432)[splitk % 3],
                   act=act, scale_dtype=act, zero="random", zero_hi=15, seed=52000 + M)
    P = Prepared(case)
    for k, v in enumerate((2, splitk, bm)):
        B.qg_set_knob(k, v)
    first = P.gpu_c()
    _check(P, first, case.name)
    assert np.array_equal(bits_of(first), bits_of(P.gpu_c()))          # counters left clean, fixed order of the slabs


def test_slabs_in_a_captured_graph():
    from paper_2504_12984_amd import binding as B
    P = Prepared(WL.Case("slabs_graph", 100, 4096, 512, WL.KIND_INT, 4, group=128, zero=None, seed=52500))
    side = torch.cuda.Stream()
    out = torch.empty(100, 512, dtype=torch.float16, device="cuda")
    for splitk in (2, 8):
        for k, v in enumerate((2, splitk, 64)):
            B.qg_set_knob(k, v)
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
            assert np.array_equal(bits_of(out), want), splitk
            P.gpu_c()                                                  # eager work between the replays
