"""Timed cases of the integer GEMM library, through its tensor entry points.

``listed()`` names twelve cases and ``draw(rng)`` gives more of the same
ranges; ``prepare`` makes a case's device tensors (and packs the weights where
the program would keep them packed), ``run`` is one call of the library,
``work`` the bytes and operations that call cannot do without, and ``exact``
the same result from plain torch in float64 and int64.

Four kinds of call:
  gemm      gemm_i16 / gemm_i8: C += A.B, int32 C with wraparound
  packed_b  gemm_packed_b: the same with the weights B packed beforehand
  srs       gemm_srs: int16 C, the product of each block of kc shifted,
            rounded, saturated and added
  conv      conv2d: NHWC convolution, int32 output
"""
from __future__ import annotations

import torch

import paper_2302_07594_amd as ig


def _gemm(name, dtype, m, n, k, **more):
    c = {"kind": "gemm", "dtype": dtype, "m": m, "n": n, "k": k}
    c.update(more)
    if name:
        c["name"] = name
    return c


def _conv(name, dtype, batch, hw, c, k, f, stride, pad, dil=1):
    d = {"kind": "conv", "dtype": dtype, "batch": batch, "h": hw, "w": hw, "c": c, "k": k,
         "f": f, "stride": stride, "pad": pad, "dil": dil}
    if name:
        d["name"] = name
    return d


def listed():
    return [
        # The smallest call: a cube that fits a few tiles; latency and the
        # host path count.
        _gemm("i16_256cube", "i16", 256, 256, 256),
        # One decode step of eight sequences through an MLP projection of a
        # 7B-class decoder: the weights are read once, nothing is reused.
        _gemm("i8_decode_8x11008x4096", "i8", 8, 11008, 4096),
        # Prefill of 512 tokens through an attention projection of the same
        # decoder.
        _gemm("i8_prefill_512x4096x4096", "i8", 512, 4096, 4096),
        # Prefill in int16 with the weights packed once and kept, as a server
        # holds them.
        _gemm("i16_packed_b_256x11008x4096", "i16", 256, 11008, 4096, kind="packed_b"),
        # The large square product in int16, the headline of the benchmark.
        _gemm("i16_4096cube", "i16", 4096, 4096, 4096),
        # The largest call: the large square product in int8.
        _gemm("i8_8192cube", "i8", 8192, 8192, 8192),
        # Odd sizes in int8, rows at any byte address (vocabulary slices,
        # pruned layers).
        _gemm("i8_ragged_1000x3001x1777", "i8", 1000, 3001, 1777),
        # Odd sizes in int16.
        _gemm("i16_ragged_777x1111x2049", "i16", 777, 1111, 2049),
        # A 3x3 layer of a 50-layer residual CNN at batch 32, int16.
        _conv("i16_conv_b32_56x56x64_3x3", "i16", 32, 56, 64, 64, 3, 1, 1),
        # The 3x3 stride-2 layer that opens the next stage, int8, batch 32.
        _conv("i8_conv_b32_56x56x128_3x3s2", "i8", 32, 56, 128, 128, 3, 2, 1),
        # The int16-output update on the paper's own shape, one block of k.
        _gemm("i16_srs_4096x4096x290", "i16", 4096, 4096, 290, kind="srs", kc=290, shift=0,
              half_up=False),
        # The int16-output update of a quantised int8 layer: 1024 tokens, the
        # sum over all of k requantised once with rounding.
        _gemm("i8_srs_1024x4096x1024", "i8", 1024, 4096, 1024, kind="srs", kc=0, shift=7,
              half_up=True),
    ]


# No drawn case has more than these (the largest listed cases do more).
_MAX_MACS = 5.0e10
_MAX_BYTES = 2.5e8


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def _extent(rng, lo, hi, whole):
    """An extent in [lo, hi], spread over its logarithm: any whole number, or
    a multiple of 64 where the case has whole tiles."""
    v = _log_int(rng, lo, hi)
    return max(64, (v + 32) // 64 * 64) if whole else v


def _draw_gemm(rng, kind):
    dtype = rng.choice(("i8", "i16"))
    if kind == "gemm" and rng.random() < 0.3:
        # decode: a few rows, any count, over weights of whole 64s
        m = _log_int(rng, 1, 48)
        n, k = _extent(rng, 1024, 12288, True), _extent(rng, 1024, 8192, True)
        return _gemm(None, dtype, m, n, k)
    if kind == "packed_b":
        # tokens of any number, weights of whole 64s
        m = _log_int(rng, 32, 2048)
        n, k = _extent(rng, 1024, 12288, True), _extent(rng, 512, 8192, True)
        return _gemm(None, dtype, m, n, k, kind=kind)
    whole = rng.random() < 0.5
    m, n, k = (_extent(rng, 64, 6144, whole) for _ in range(3))
    if kind == "srs":
        kc = rng.choice((0, 0, 256, 512, 290))
        # up to the shift that brings a long sum back into 16 bits
        shift = rng.randint(0, 24 if dtype == "i16" else 12)
        return _gemm(None, dtype, m, n, k, kind=kind, kc=kc, shift=shift,
                     half_up=rng.random() < 0.5)
    return _gemm(None, dtype, m, n, k)


def _draw_conv(rng):
    dtype = rng.choice(("i8", "i16"))
    f = rng.choice((1, 3, 3, 5, 7))
    stride = rng.choice((1, 1, 2))
    dil = 2 if f == 3 and rng.random() < 0.2 else 1
    hw = _log_int(rng, 7, 112)
    if rng.random() < 0.2:
        c = rng.choice((1, 3, 4))  # an image or a stem
    else:
        c = rng.choice((16, 24, 32, 48, 64, 96, 128, 256, 512, 30, 75, 200))
    k = rng.choice((16, 32, 64, 96, 128, 256, 512, 40, 91, 255))
    return _conv(None, dtype, _log_int(rng, 1, 32), hw, c, k, f, stride, dil * (f // 2), dil)


def draw(rng):
    while True:
        kind = rng.choice(("gemm", "gemm", "gemm", "packed_b", "srs", "srs", "conv", "conv"))
        case = _draw_conv(rng) if kind == "conv" else _draw_gemm(rng, kind)
        w = work(case)
        if 2.0e6 <= w["flops"] / 2 <= _MAX_MACS and w["bytes"] <= _MAX_BYTES:
            return case


def _out_hw(case):
    def extent(size):
        span = size + 2 * case["pad"] - case["dil"] * (case["f"] - 1) - 1
        return span // case["stride"] + 1
    return extent(case["h"]), extent(case["w"])


def _uniform(gen, lo, hi, shape, dtype):
    return torch.randint(lo, hi + 1, shape, generator=gen, device="cuda",
                         dtype=torch.int32).to(dtype)


def _normal(gen, sigma, lo, hi, shape, dtype):
    x = torch.empty(shape, device="cuda").normal_(0.0, sigma, generator=gen)
    return x.round_().clamp_(lo, hi).to(dtype)


def _inputs(case, seed):
    """(A or X, B or W, C or Y) on the GPU, from the seed alone. Activations
    are uniform over the type's range (for convolutions over [0, 255] in
    int16 and [0, 127] in int8, as after a ReLU), weights a clipped rounded
    normal, C uniform. Square products, and those of 4096 rows and more, are
    not a layer's: their B is uniform over the type's range like A."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    wide = case["dtype"] == "i16"
    dt, lo, hi = (torch.int16, -32768, 32767) if wide else (torch.int8, -128, 127)
    if case["kind"] == "conv":
        oh, ow = _out_hw(case)
        x = _uniform(gen, 0, 255 if wide else 127,
                     (case["batch"], case["h"], case["w"], case["c"]), dt)
        w = _normal(gen, 32.0 if wide else 20.0, lo, hi,
                    (case["f"], case["f"], case["c"], case["k"]), dt)
        y = _uniform(gen, -(1 << 20), 1 << 20, (case["batch"], oh, ow, case["k"]), torch.int32)
        return x, w, y
    m, n, k = case["m"], case["n"], case["k"]
    a = _uniform(gen, lo, hi, (m, k), dt)
    if m == n or m >= 4096:
        b = _uniform(gen, lo, hi, (k, n), dt)
    else:
        b = _normal(gen, 5120.0 if wide else 20.0, lo, hi, (k, n), dt)
    if case["kind"] == "srs":
        c = _uniform(gen, -32768, 32767, (m, n), torch.int16)
    else:
        c = _uniform(gen, -(1 << 20), 1 << 20, (m, n), torch.int32)
    return a, b, c


def prepare(case, seed):
    a, b, c = _inputs(case, seed)
    state = {"case": case, "a": a, "b": b, "c": c}
    if case["kind"] == "packed_b":
        state["b"] = ig.pack_b(b)  # the server keeps only the packed weights
    return state


def run(state):
    case, a, b, c = state["case"], state["a"], state["b"], state["c"]
    kind = case["kind"]
    if kind == "gemm":
        return ig.gemm_i16(a, b, c) if case["dtype"] == "i16" else ig.gemm_i8(a, b, c)
    if kind == "packed_b":
        return ig.gemm_packed_b(a, b, c)
    if kind == "srs":
        return ig.gemm_srs(a, b, c, kc=case["kc"], shift=case["shift"],
                           round_half_up=case["half_up"])
    return ig.conv2d(a, b, c, stride=(case["stride"],) * 2, pad=(case["pad"],) * 2,
                     dil=(case["dil"],) * 2)


def work(case):
    """Each operand read once, C (or Y) read and written once; a multiply-add
    counts as two operations."""
    es = 2 if case["dtype"] == "i16" else 1
    if case["kind"] == "conv":
        oh, ow = _out_hw(case)
        m, n, k = case["batch"] * oh * ow, case["k"], case["f"] ** 2 * case["c"]
        a_bytes = es * case["batch"] * case["h"] * case["w"] * case["c"]
    else:
        m, n, k = case["m"], case["n"], case["k"]
        a_bytes = es * m * k
    c_bytes = 2 if case["kind"] == "srs" else 4
    return {"bytes": a_bytes + es * k * n + 2 * c_bytes * m * n, "flops": 2 * m * n * k}


def tolerance(case):
    return "exact"


def _product(a, b):
    # |sum| <= k 2^30 < 2^53: float64 holds every partial sum exactly.
    return (a.double() @ b.double()).to(torch.int64)


def exact(case, seed):
    a, b, c = _inputs(case, seed)
    if case["kind"] == "conv":
        f, oh, ow = case["f"], *_out_hw(case)
        cols = torch.nn.functional.unfold(a.double().permute(0, 3, 1, 2).contiguous(), f,
                                          dilation=case["dil"], padding=case["pad"],
                                          stride=case["stride"])
        # unfold orders a column (channel, filter row, filter column)
        w = b.permute(2, 0, 1, 3).reshape(-1, case["k"]).contiguous().double()
        y = torch.stack([col.t().contiguous() @ w for col in cols]).to(torch.int64)
        return (c.to(torch.int64) + y.reshape(c.shape)).to(torch.int32)
    if case["kind"] != "srs":
        return (c.to(torch.int64) + _product(a, b)).to(torch.int32)
    k = case["k"]
    kc = case["kc"] if 0 < case["kc"] < k else k
    half = (1 << case["shift"]) >> 1 if case["half_up"] else 0
    out = c.to(torch.int64)
    for p in range(0, k, kc):
        t = (_product(a[:, p:p + kc], b[p:p + kc]) + half) >> case["shift"]
        out += t.clamp_(-32768, 32767)
    return out.to(torch.int16)
