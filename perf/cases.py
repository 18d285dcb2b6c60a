"""The timed cases of the library: what a program that serves a low-bit model asks of it.

Every case is a plain dict:

    path    "linear"    16-bit activations times a low-bit weight (qgemm)
            "a8"        int8 activations with one fp32 scale per row (qgemm_a8)
            "codebook"  codes that index a table of fp16 levels (qgemm_codebook)
            "load"      a weight on its way in: codes -> canonical stream -> device layout
    w       weight type: u1..u8, i1..i8, f3..f8 (e1m1, e2m1, e2m2, e3m2, e3m3, e4m3), cb1..cb8
    act     "f16" | "bf16": activations, results (for "a8": results)
    scale   "f16" | "bf16", or "e8m0": one power-of-two byte per 32 rows
    group   rows of the weight per scale; 0 = one scale per output column
    zeros   a zero-point per (group, column), or none
    M, K, N rows of activations, and the weight's shape
    layers  weights of this shape that one pass goes through, one after the other, as the
            layers of a model: a decode step meets every weight cold, because all the others
            came in between
    block   instead of one shape the four projections of a transformer layer with hidden
            size K and inner size N: K -> 1.5 K, K -> K, K -> 2 N, N -> K
    bound   calls whose arguments were checked once (the Bound* objects a decode loop keeps);
            otherwise the plain functions
"""
from __future__ import annotations

import math

import torch

from paper_2504_12984_amd import binding as B

_DT = {"f16": torch.float16, "bf16": torch.bfloat16}
_FLOAT = {3: (1, 1), 4: (2, 1), 5: (2, 2), 6: (3, 2), 7: (3, 3), 8: (4, 3)}


def _case(name, path, w, M, K, N, act="f16", scale="f16", group=128, zeros=False, layers=1, block=False, bound=True):
    c = {"path": path, "w": w, "act": act, "scale": scale, "group": group, "zeros": zeros,
         "M": M, "K": K, "N": N, "layers": layers, "block": block, "bound": bound}
    return {"name": name, **c} if name else c


def listed():
    return [
        # One token through one small projection by the plain call: all launch and host latency.
        _case("one_row_512", "linear", "u4", 1, 512, 512, zeros=True, bound=False),
        # Two whole layers of one decode step for one sequence: short and long K, narrow and wide N.
        _case("decode_block_u3_m1", "linear", "u3", 1, 4096, 14336, zeros=True, layers=2, block=True),
        # Batched decode on the large projection of a 70B-class model, symmetric int4.
        _case("decode_i4_m16", "linear", "i4", 16, 8192, 28672, layers=2),
        # Per-channel 6-bit floats with bf16 activations, one sequence, square projections.
        _case("decode_f6_m1_channel", "linear", "f6", 1, 8192, 8192, act="bf16", group=0, layers=4),
        # Continuous batching with a few dozen sequences; a row count that is no tile's multiple.
        _case("rows45_u4_g64", "linear", "u4", 45, 8192, 8192, group=64, zeros=True, layers=3),
        # A large decode batch / a short prompt, again ragged.
        _case("rows300_u4", "linear", "u4", 300, 8192, 8192, zeros=True, layers=2),
        # The largest: prefill of 4096 tokens on the widest projection.
        _case("prefill_u6_m4096", "linear", "u6", 4096, 8192, 57344, act="bf16", scale="bf16", group=64, zeros=True,
              bound=False),
        # Block-scaled 4-bit floats (one exponent per 32 rows), an odd prompt length.
        _case("prefill_mxf4_m1000", "linear", "f4", 1000, 8192, 28672, act="bf16", scale="e8m0", group=32, bound=False),
        # int8 activations: batched decode, and a prompt.
        _case("a8_decode_i4_m16", "a8", "i4", 16, 8192, 28672, layers=2),
        _case("a8_prefill_u4_m1000", "a8", "u4", 1000, 8192, 28672, zeros=True, bound=False),
        # Codebook weights in batched decode.
        _case("codebook4_m16", "codebook", "cb4", 16, 8192, 28672, layers=2),
        # A checkpoint's weight made ready: an odd code width, straddling bytes.
        _case("load_u5", "load", "u5", 1, 8192, 28672, zeros=False),
    ]


# ---- drawn cases --------------------------------------------------------------------------------
def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _mult(rng, lo, hi, step):
    """A multiple of `step`, log-uniform over [lo, hi]; half of the time a round one (a power of two of steps)."""
    v = _log(rng, lo, hi)
    if rng.random() < 0.5:
        v = 2.0 ** round(math.log2(v))
    return max(lo, min(hi, int(round(v / step)) * step))


_MNK = {"linear": 4096 * 8192 * 57344, "codebook": 2048 * 8192 * 28672, "a8": 1000 * 8192 * 28672}


def draw(rng):
    path = rng.choices(["linear", "a8", "codebook", "load"], [8, 3, 2, 1])[0]
    K = _mult(rng, 512, 16384, 128)
    N = _mult(rng, 512, 57344, 64)
    while K * N > 8192 * 28672:
        N = max(512, N // 2 // 64 * 64)
    act = rng.choice(["f16", "bf16"])
    scale = "f16" if act == "f16" else rng.choice(["f16", "bf16"])
    if path == "load":
        w = rng.choice(["u", "i"]) + str(rng.randint(1, 8)) if rng.random() < 0.7 else "f" + str(rng.randint(3, 8))
        return _case(None, "load", w, 1, K, N)
    if path == "codebook":
        w = "cb" + str(rng.choice([2, 3, 4, 4, 4, 5, 6, 8]))
    elif path == "a8":
        w = rng.choice(["u", "i"]) + str(rng.choice([2, 3, 4, 4, 4, 5, 6, 8, 8]))
    else:
        w = rng.choice(["u", "u", "i", "f"])
        w += str(rng.randint(3, 8) if w == "f" else rng.choice([1, 2, 3, 4, 4, 4, 5, 6, 7, 8]))
        if w in ("f4", "f8") and rng.random() < 0.5:
            act, scale = "bf16", "e8m0"
    groups = [g for g in (128, 128, 128, 64, 256, 0) if g == 0 or K % g == 0]
    if path == "linear":
        groups.append(32)
    group = 32 if scale == "e8m0" else rng.choice(groups)
    zeros = w[0] == "u" and rng.random() < 0.7
    # rows: half decode batches, the rest up to the longest prompt the largest listed case allows
    most = _MNK[path] // (K * N)
    M = int(_log(rng, 1, 65)) if rng.random() < 0.5 else int(_log(rng, 33, max(34, min(8192, most))))
    M = max(1, min(M, most))
    layers = 1
    if M <= 64:
        layers = max(1, min(6, round(128e6 / (K * N * _bits(w) / 8))))
    return _case(None, path, w, M, K, N, act, scale, group, zeros, layers, False, M <= 64)


# ---- inputs -------------------------------------------------------------------------------------
def _bits(w):
    return int(w.lstrip("uifcb"))


def _wtype(w):
    bits = _bits(w)
    if w.startswith("cb"):
        return B.WType(B.QG_CODEBOOK, bits)
    if w[0] == "f":
        return B.WType(B.QG_FLOAT, bits, *_FLOAT[bits])
    return B.WType(B.QG_UINT if w[0] == "u" else B.QG_INT, bits)


def _shapes(case):
    K, N = case["K"], case["N"]
    one = [(K, 3 * K // 2), (K, K), (K, 2 * N), (N, K)] if case["block"] else [(K, N)]
    return one * case["layers"]


def _scale_rows(case, K):
    return K // case["group"] if case["group"] else 1


def _codes(case, K, N, gen):
    bits = _bits(case["w"])
    codes = torch.randint(0, 1 << bits, (K, N), dtype=torch.uint8, device="cuda", generator=gen)
    if case["w"] == "f8":          # the one not-a-number of e4m3 (either sign) is no weight
        codes = torch.where((codes & 0x7F) == 0x7F, codes ^ 1, codes)
    return codes


def _activations(case, K, gen):
    A = torch.randn(case["M"], K, device="cuda", generator=gen)
    if case["path"] == "a8":
        return torch.clamp(torch.round(A * 40.0), -127, 127).to(torch.int8)
    return A.to(_DT[case["act"]])


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    t = _wtype(case["w"])
    if case["path"] == "load":
        return {"case": case, "t": t, "codes": _codes(case, case["K"], case["N"], gen)}
    layout = B.QG_LAYOUT_TILE128x64_I8 if case["path"] == "a8" else B.QG_LAYOUT_TILE128x64
    act, calls, inputs = _DT[case["act"]], [], {}
    for K, N in _shapes(case):
        if K not in inputs:        # layers of one width read the same kind of activations
            inputs[K] = _activations(case, K, gen)
        A = inputs[K]
        packed = B.repack(B.qg_pack_codes(_codes(case, K, N, gen), t.bits), t, K, N, layout=layout)
        rows = _scale_rows(case, K)
        if case["scale"] == "e8m0":
            scales = torch.randint(117, 125, (rows, N), dtype=torch.uint8, device="cuda", generator=gen)
        else:
            scales = (0.005 + 0.015 * torch.rand(rows, N, device="cuda", generator=gen)).to(_DT[case["scale"]])
        zeros = None
        if case["zeros"]:
            zeros = torch.randint(0, 1 << t.bits, (rows, N), dtype=torch.uint8, device="cuda", generator=gen)
        group, M = case["group"], case["M"]
        args = [A, packed, scales, zeros, t, group, N]
        if case["path"] == "a8":
            a_scale = 0.02 + 0.01 * torch.rand(M, device="cuda", generator=gen)
            args = [A, a_scale, packed, scales, zeros, t, group, N]
            plain, held = B.qgemm_a8, B.BoundQgemmA8
        elif case["path"] == "codebook":
            levels = torch.randn(1 << t.bits, device="cuda", generator=gen).clamp(-3, 3).sort().values.half()
            args = [A, packed, levels, scales, t.bits, group, N]
            plain, held = B.qgemm_codebook, B.BoundQgemmCodebook
        else:
            plain, held = B.qgemm, B.BoundQgemm
        if case["bound"]:
            calls.append((held(*args, torch.empty(M, N, dtype=act, device="cuda")), (), {}))
        else:
            calls.append((plain, tuple(args), {"out_dtype": act} if case["path"] == "a8" else {}))
    return {"case": case, "calls": calls}


def run(state):
    case = state["case"]
    if case["path"] == "load":
        stream = B.qg_pack_codes(state["codes"], state["t"].bits)
        return {"stream": stream, "packed": B.repack(stream, state["t"], case["K"], case["N"])}
    return [fn(*args, **kw) for fn, args, kw in state["calls"]]


# ---- what a pass cannot do without --------------------------------------------------------------
def work(case):
    bits, M = _bits(case["w"]), case["M"]
    if case["path"] == "load":     # codes in, stream out, stream in, packed out
        n = case["K"] * case["N"]
        return {"bytes": n + 3 * (n * bits // 8), "flops": 0}
    nbytes = flops = 0
    for K, N in _shapes(case):
        rows = _scale_rows(case, K)
        nbytes += K * N * bits // 8 + rows * N * (1 if case["scale"] == "e8m0" else 2) + (rows * N if case["zeros"] else 0)
        nbytes += M * K * (1 if case["path"] == "a8" else 2) + 2 * M * N + (4 * M if case["path"] == "a8" else 0)
        nbytes += (2 << bits) if case["path"] == "codebook" else 0
        flops += 2 * M * N * K
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # The path against the same contraction of its de-quantised weights in 64 bits shows the one
    # rounding to the output type and nothing else: 2-norm of the difference over that of the result
    # 2.1e-4 (fp16) and 1.66e-3 (bf16) at every shape tried, largest difference 4.8e-4 and 3.9e-3.
    # Four times that; what a "load" returns is bytes.
    if case["path"] == "load":
        return "exact"
    return {"rel": 8e-4, "max": 2e-3} if case["act"] == "f16" else {"rel": 7e-3, "max": 1.6e-2}
