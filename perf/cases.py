"""The calls this library is used for, as cases that can be timed and checked.

A case names an entry point, the shape of one weight matrix and the quantisation options; `prepare` makes what a
program holds before the call (quantised weights, activations, workspace), `run` is the call, `exact` the same
result from plain torch in 64 bits.  Weights are Gaussian and quantised on the device with lutq_quantize, as a
program that loads a dense checkpoint does; the shapes are the linear layers of LLaMA-2-13B and LLaMA-3-8B/70B and
the N = K = 8192 matrix of the paper's kernel study.

`op` of a case:
  matmul    lutq_matmul, one shared table
  static    lutq_matmul_static (the library's built-in scratch)
  step      one decode token through the linear layers of `layers` transformer layers, replayed as one HIP graph
  channel   lutq_matmul_channel, one table per output row
  pairs     lutq_matmul_pairs, a codebook of 256 pairs (4-bit layout)
  quads     lutq_matmul_quads, a codebook of 256 quads (2-bit layout)
  quantize  lutq_quantize, dense weights (`src`: f32, or the 16-bit dtype) to scales and packed indices
  dequant   lutq_dequant, packed weights back to a dense 16-bit matrix
"""
import math

import numpy as np
import torch

import lutq_inputs as gen
import paper_2407_10960_amd as lutq

# q/k/v, o, gate/up, down of LLaMA-3-8B: (N, K)
LAYER = ((6144, 4096), (4096, 4096), (28672, 4096), (4096, 14336))


def _case(name, op, m, n, k, bits, group, dtype, lut="nf", **more):
    return dict(name=name, op=op, m=m, n=n, k=k, bits=bits, group=group, dtype=dtype, lut=lut, **more)


def listed():
    return [
        # the smallest call of a decode step: one token through the attention output projection
        _case("decode_o_w4_m1", "matmul", 1, 4096, 4096, 4, 128, "f16"),
        # one decode token through four layers' linear layers (16 weight matrices, more than the caches hold),
        # captured once and replayed: how a serving loop runs it
        _case("decode_step_4_layers_w4_m1", "step", 1, 0, 0, 4, 128, "f16", layers=4),
        # decode of a few sequences, or the check of a few drafted tokens, on the largest layer of the 70B model
        _case("decode_70b_gate_up_w4_bf16_m4", "matmul", 4, 57344, 8192, 4, 64, "bf16"),
        # small serving batch, 3 bits, a learned table
        _case("batch_8b_qkv_w3_bf16_m8", "matmul", 8, 6144, 4096, 3, 128, "bf16", lut="learned"),
        # a batch and a matrix that fill no power of two: LLaMA-2-13B down
        _case("batch_13b_down_w4_m13", "matmul", 13, 5120, 13824, 4, 128, "f16"),
        # the largest batch of the paper's study on its square matrix, small groups
        _case("batch_sq_w4_g32_m32", "matmul", 32, 8192, 8192, 4, 32, "f16"),
        # batched decode of 64 sequences, long K
        _case("batch_8b_down_w4_m64", "matmul", 64, 4096, 14336, 4, 128, "f16"),
        # a prompt chunk of 128 tokens through the largest layer of the 8B model
        _case("prompt_8b_gate_up_w4_m128", "matmul", 128, 28672, 4096, 4, 128, "f16"),
        # a ragged prompt chunk at 3 bits, bf16
        _case("prompt_70b_o_w3_bf16_m100", "matmul", 100, 8192, 8192, 3, 64, "bf16"),
        # one table per output row, a serving batch
        _case("channel_8b_gate_up_w4_m16", "channel", 16, 28672, 4096, 4, 128, "f16", lut="learned"),
        # quantising a bf16 checkpoint matrix on the device: 70B down
        _case("quantize_70b_down_w4_bf16", "quantize", 0, 8192, 28672, 4, 64, "bf16", src="bf16"),
        # dense weights back for a long prompt that a dense product then runs on
        _case("dequant_8b_gate_up_w4", "dequant", 0, 28672, 4096, 4, 128, "f16"),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    op = rng.choices(("matmul", "static", "channel", "pairs", "quads", "quantize", "dequant"),
                     (60, 5, 8, 5, 5, 10, 7))[0]
    bits = 4 if op == "pairs" else 2 if op == "quads" else rng.choices((4, 3, 2), (5, 3, 2))[0]
    group = rng.choice((32, 64, 128, 256))
    dtype = rng.choice(("f16", "bf16"))
    step = max(group, 128 if bits == 4 else 256)
    k = step * max(1, round(_log(rng, 1024, 28672) / step))
    # rows in units of 16, not of a power of two; the product is at most 8B gate+up (quantiser, dense) or twice that
    most = (1.2e8 if op in ("quantize", "dequant") else 2.4e8) / k
    n = 16 * max(1, round(_log(rng, 1024, min(57344, most)) / 16))
    m = 0 if op in ("quantize", "dequant") else min(128, max(1, round(_log(rng, 0.75, 140))))
    c = _case("", op, m, n, k, bits, group, dtype, rng.choice(("nf", "learned")))
    if op == "quantize":
        c["src"] = rng.choice(("f32", dtype))
    del c["name"]
    return c


def _dt(dtype):
    return torch.float16 if dtype == "f16" else torch.bfloat16


def _gen(seed, salt):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 1009 + salt)
    return g


def _randn(seed, salt, *shape, dtype=torch.float32):
    return torch.randn(shape, generator=_gen(seed, salt), device="cuda", dtype=dtype)


def _table(case, seed):
    """The table the weights are quantised to."""
    if case["lut"] == "nf":
        t = torch.from_numpy(gen.normal_float_table(case["bits"])).cuda()
    else:                                       # a learned table: ascending, any spacing, about the unit range
        t = torch.sort(_randn(seed, 3, 1 << case["bits"]).double()).values
        t = t / t.abs().max()
    return t.to(_dt(case["dtype"]))


def _weights(case, seed, salt, n, k):
    """Dense Gaussian weights: fp32 where `src` says so, else the 16-bit type."""
    w = _randn(seed, salt, n, k, dtype=torch.float32).mul_(0.02)
    return w if case.get("src") == "f32" else w.to(_dt(case["dtype"]))


def _activations(case, seed, salt, k):
    return _randn(seed, salt, case["m"], k).to(_dt(case["dtype"]))


def _codebook(case, seed):
    """What the indices of a call that does not use the quantiser's own table select."""
    op, dt = case["op"], _dt(case["dtype"])
    if op == "channel":
        return _randn(seed, 4, case["n"], 1 << case["bits"]).to(dt)
    if op in ("pairs", "quads"):
        return _randn(seed, 4, 256, 2 if op == "pairs" else 4).to(dt)
    return _table(case, seed)


def _quantised(case, seed, salt, n, k, table):
    bits, group = case["bits"], case["group"]
    w = _weights(case, seed, salt, n, k)
    scales = torch.empty((n, k // group), dtype=table.dtype, device="cuda")
    packed = torch.empty(lutq.lutq_packed_bytes(n, k, bits, group), dtype=torch.uint8, device="cuda")
    lutq.lutq_quantize(w, table, bits, group, scales, packed)
    return packed, scales


def prepare(case, seed):
    op, bits, group, n, k = case["op"], case["bits"], case["group"], case["n"], case["k"]
    dt = _dt(case["dtype"])
    table = _table(case, seed)
    s = {"op": op, "bits": bits, "group": group, "table": table}
    if op == "quantize":
        s["W"] = _weights(case, seed, 16, n, k)
        s["scales"] = torch.empty((n, k // group), dtype=dt, device="cuda")
        s["packed"] = torch.empty(lutq.lutq_packed_bytes(n, k, bits, group), dtype=torch.uint8, device="cuda")
        return s
    if op == "step":
        s["calls"] = []
        workspace = lutq.new_workspace(*LAYER[0], bits, group)
        for i in range(case["layers"] * len(LAYER)):
            n, k = LAYER[i % len(LAYER)]
            packed, scales = _quantised(case, seed, 16 + i, n, k, table)
            y = torch.empty((case["m"], n), dtype=dt, device="cuda")
            s["calls"].append((_activations(case, seed, 512 + i, k), packed, scales, table, bits, group, y, workspace))
        # captured once, replayed for every token (the first launch of each call outside the capture)
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            for c in s["calls"]:
                lutq.lutq_matmul(*c)
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            for c in s["calls"]:
                lutq.lutq_matmul(*c)
        return s
    s["packed"], s["scales"] = _quantised(case, seed, 16, n, k, table)
    if op == "dequant":
        s["W"] = torch.empty((n, k), dtype=dt, device="cuda")
        return s
    s["X"] = _activations(case, seed, 512, k)
    s["Y"] = torch.empty((case["m"], n), dtype=dt, device="cuda")
    s["lut"] = _codebook(case, seed)
    if op != "static":
        s["workspace"] = lutq.new_workspace(n, k, bits, group)
    return s


def run(s):
    op, bits, group = s["op"], s["bits"], s["group"]
    if op == "matmul":
        return lutq.lutq_matmul(s["X"], s["packed"], s["scales"], s["lut"], bits, group, s["Y"], s["workspace"])
    if op == "step":
        s["graph"].replay()
        return [c[6] for c in s["calls"]]
    if op == "static":
        return lutq.lutq_matmul_static(s["X"], s["packed"], s["scales"], s["lut"], bits, group, s["Y"])
    if op == "channel":
        return lutq.lutq_matmul_channel(s["X"], s["packed"], s["scales"], s["lut"], bits, group, s["Y"], s["workspace"])
    if op == "pairs":
        return lutq.lutq_matmul_pairs(s["X"], s["packed"], s["scales"], s["lut"], group, s["Y"], s["workspace"])
    if op == "quads":
        return lutq.lutq_matmul_quads(s["X"], s["packed"], s["scales"], s["lut"], group, s["Y"], s["workspace"])
    if op == "quantize":
        return lutq.lutq_quantize(s["W"], s["table"], bits, group, s["scales"], s["packed"])
    return lutq.lutq_dequant(s["packed"], s["scales"], s["table"], bits, group, s["W"])


def _matrices(case):
    return [LAYER[i % len(LAYER)] for i in range(case["layers"] * len(LAYER))] if case["op"] == "step" else [(case["n"], case["k"])]


def work(case):
    nbytes = flops = 0
    for n, k in _matrices(case):
        quantised = n * k * case["bits"] // 8 + n * (k // case["group"]) * 2
        if case["op"] == "quantize":
            nbytes += n * k * (4 if case["src"] == "f32" else 2) + quantised
        elif case["op"] == "dequant":
            nbytes += quantised + n * k * 2
        else:
            nbytes += quantised + case["m"] * (n + k) * 2
            if case["op"] == "channel":
                nbytes += n * (2 << case["bits"])
            flops += 2 * case["m"] * n * k
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["op"] in ("quantize", "dequant"):
        return "exact"
    # Sums are fp32; what another order of summation changes is which way an output rounds, at most by one unit in the
    # last place of the 16-bit type (2^-10 and 2^-7 of the value's binade), and its fp32 error where the sum cancels.
    # Measured against 64 bits: rel 2.1e-4 (fp16) and 1.7e-3 (bf16), which is the rounding itself.
    return {"rel": 8e-4, "max": 4e-3} if case["dtype"] == "f16" else {"rel": 6e-3, "max": 3e-2}


def _indices(w, scales16, table, group):
    """The lowest index of the nearest table entry to w / scale, in 64 bits; w: some rows of the dense matrix."""
    n, k = w.shape
    s = scales16.double().repeat_interleave(group, dim=1)
    u = torch.where(s == 0, torch.zeros_like(s), w.double() / s)
    best = (u - table[0]).abs()
    idx = torch.zeros((n, k), dtype=torch.int64, device=w.device)
    for c in range(1, table.numel()):
        d = (u - table[c]).abs()
        less = d < best
        best = torch.where(less, d, best)
        idx = torch.where(less, torch.full_like(idx, c), idx)
    return idx


def _exact_rows(case, seed, salt, n, k, table16, book):
    """For some rows at a time: (first row, absmax in 64 bits, weights in 64 bits rounded once to the 16-bit type)."""
    op, group, dt = case["op"], case["group"], _dt(case["dtype"])
    dense = _weights(case, seed, salt, n, k)
    table = table16.double()
    rows = max(1, (1 << 24) // k)
    for r0 in range(0, n, rows):
        w = dense[r0:r0 + rows]
        absmax = w.double().abs().reshape(w.shape[0], k // group, group).amax(dim=2)
        if op == "quantize":
            yield r0, absmax, None
            continue
        s16 = absmax.float().to(dt)
        q = _indices(w, s16, table, group)
        if op == "channel":
            v = torch.gather(book[r0:r0 + rows].double(), 1, q)
        elif op in ("pairs", "quads"):
            d, bits = (2, 4) if op == "pairs" else (4, 2)
            q = q.reshape(w.shape[0], k // d, d)
            code = sum(q[:, :, i] << (bits * i) for i in range(d))
            v = book.double()[code].reshape(w.shape[0], k)
        else:
            v = table[q]
        yield r0, None, v * s16.double().repeat_interleave(group, dim=1)


def exact(case, seed):
    dt, table = _dt(case["dtype"]), _table(case, seed)
    out = []
    for i, (n, k) in enumerate(_matrices(case)):
        salt = 16 + i
        book = _codebook(case, seed) if case["op"] != "step" else table
        if case["op"] == "quantize":
            return [torch.cat([a for _, a, _ in _exact_rows(case, seed, salt, n, k, table, book)]), None]
        if case["op"] == "dequant":
            w = torch.empty((n, k), dtype=torch.float64, device="cuda")
            for r0, _, v in _exact_rows(case, seed, salt, n, k, table, book):
                w[r0:r0 + v.shape[0]] = v
            return w
        x = _activations(case, seed, 512 + i, k).double()
        y = torch.empty((case["m"], n), dtype=torch.float64, device="cuda")
        for r0, _, v in _exact_rows(case, seed, salt, n, k, table, book):
            y[:, r0:r0 + v.shape[0]] = x @ v.float().to(dt).double().t()
        out.append(y)
    return out if case["op"] == "step" else out[0]
