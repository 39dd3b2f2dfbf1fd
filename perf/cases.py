"""The work users of this library have it do, as cases that can be timed.

A case is a dict of plain values; ``prepare`` builds what a user's program holds before the call
(device inputs, the plans), ``run`` makes one pass through the public entry points of
``paper_2605_29843_amd.harp``.  Sizes are the layer widths of the Llama families that this
repository's workloads and shape sweeps use, under the two schedule families they use: "r2"
(radix-2 stages, the remaining odd factor last) and "g8" (the greedy radix-8 schedule, the paper's
default).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2605_29843_amd import harp, inputs as gi

# the radix-2 schedule of every width (the greedy one comes from harp_greedy_schedule)
RADIX2 = {
    2048: [2] * 11,
    3072: [2] * 10 + [3],
    4096: [2] * 12,
    5120: [2] * 10 + [5],
    8192: [2] * 13,
    11008: [2] * 8 + [43],
    13824: [2] * 9 + [3, 3, 3],
    14336: [2] * 11 + [7],
    28672: [2] * 12 + [7],
}
WIDTHS = tuple(RADIX2)

def schedule(d: int, family: str) -> list[int]:
    return list(RADIX2[d]) if family == "r2" else harp.harp_greedy_schedule(d, 8, 8)


def listed() -> list[dict]:
    return [
        # one token of decode in a serving loop (buffers kept): latency, not bandwidth
        dict(name="decode_4096_r2", op="apply", d=4096, n=1, family="r2", dtype="bf16"),
        # a small decode batch on a feed-forward width under the paper's default schedule
        dict(name="decode_14336_g8", op="apply", d=14336, n=6, family="g8", dtype="bf16"),
        # prefill on the hidden width of the 7B / 8B models, both schedule families
        dict(name="prefill_4096_r2", op="apply", d=4096, n=2048, family="r2", dtype="bf16"),
        dict(name="prefill_4096_g8", op="apply", d=4096, n=2048, family="g8", dtype="bf16"),
        # prefill in front of a 7B down projection: 43 is left over as one large radix
        dict(name="prefill_11008_r2", op="apply", d=11008, n=2048, family="r2", dtype="bf16"),
        # rotating back (X U^T) a ragged batch on the 8B feed-forward width
        dict(name="back_14336_g8", op="apply_transpose", d=14336, n=777, family="g8", dtype="bf16"),
        # rotating back the largest activations: the 70B feed-forward width
        dict(name="back_28672_r2", op="apply_transpose", d=28672, n=4096, family="r2", dtype="bf16"),
        # calibration statistics in float32 on the 13B hidden width, a ragged number of rows
        dict(name="calib_5120_r2_f32", op="apply", d=5120, n=1001, family="r2", dtype="f32"),
        # change of basis of a 70B up projection before quantization
        dict(name="rotate_28672x8192_g8", op="rotate", d_out=28672, d_in=8192, family="g8", dtype="bf16"),
        # the way back for a dequantized 7B down projection
        dict(name="unrotate_4096x11008_r2", op="unrotate", d_out=4096, d_in=11008, family="r2",
             dtype="bf16"),
        # one fitting step's backward pass on a batch of activations
        dict(name="grad_4096_r2", op="grad", d=4096, n=2048, family="r2", dtype="bf16"),
        # the same in float32 with the rows of a weight matrix as the batch (layerwise fitting)
        dict(name="grad_11008_g8_f32", op="grad", d=11008, n=1537, family="g8", dtype="f32"),
    ]


def _rows(rng, lo: int, hi: int) -> int:
    """Log-uniform row count; every other one is odd whatever the range."""
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return max(lo, n | 1 if rng.random() < 0.5 else n)


def draw(rng) -> dict:
    op = rng.choice(["apply", "apply", "apply", "apply_transpose", "apply_transpose", "rotate",
                     "unrotate", "grad"])
    family = rng.choice(["r2", "g8"])
    dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
    if op in ("rotate", "unrotate"):
        # any two widths as the sides of a weight matrix, up to the size of the largest listed one
        d_out, d_in = rng.choice(WIDTHS), rng.choice(WIDTHS)
        while d_out * d_in > 28672 * 8192:
            d_out, d_in = rng.choice(WIDTHS), rng.choice(WIDTHS)
        if d_out * d_in > 1 << 27:
            dtype = "bf16"          # the largest matrices stay within the largest listed case
        return dict(op=op, d_out=d_out, d_in=d_in, family=family, dtype=dtype)
    d = rng.choice(WIDTHS)
    # training batches are not single rows; the cap keeps a draw below the largest listed case
    lo, cap = (64, 1 << 24) if op == "grad" else (1, 1 << 27)
    return dict(op=op, d=d, n=_rows(rng, lo, min(8192, cap // d)), family=family, dtype=dtype)


def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _generator(seed: int):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _activations(n: int, d: int, g, rng) -> torch.Tensor:
    """Student-t(3) entries with 1 % of the channels 20 times as large."""
    x = torch.randn(n, d, device="cuda", generator=g)
    chi2 = sum(torch.randn(n, d, device="cuda", generator=g).square_() for _ in range(3))
    x *= torch.rsqrt(chi2 / 3.0)
    channels = rng.choice(d, size=math.ceil(0.01 * d), replace=False)
    x[:, torch.from_numpy(channels).cuda()] *= 20.0
    return x


def _processor(d: int, family: str, rng) -> tuple:
    """(d, radices, blocks, signs) of one processor."""
    radices = schedule(d, family)
    return d, radices, gi.make_blocks(d, radices, "orth", rng), gi.make_signs(d, rng)


def _inputs(case: dict, seed: int) -> dict:
    """Processors as numpy arrays, the matrices on the device; the same for every caller."""
    rng, g, dt = np.random.default_rng(seed), _generator(seed), _dtype(case)
    if case["op"] in ("rotate", "unrotate"):
        out = {"U": _processor(case["d_out"], case["family"], rng),
               "V": _processor(case["d_in"], case["family"], rng)}
        w = torch.randn(case["d_out"], case["d_in"], device="cuda", generator=g)
        out["W"] = w.mul_(0.02).to(dt)
        return out
    n, d = case["n"], case["d"]
    out = {"processor": _processor(d, case["family"], rng)}
    out["X"] = _activations(n, d, g, rng).to(dt)
    if case["op"] == "grad":
        out["G"] = (torch.randn(n, d, device="cuda", generator=g) * 0.05).to(dt)
    return out


def prepare(case: dict, seed: int) -> dict:
    inp = _inputs(case, seed)
    state = {"op": case["op"]}
    if case["op"] in ("rotate", "unrotate"):
        state["plan_U"], state["plan_V"] = harp.Plan(*inp["U"]), harp.Plan(*inp["V"])
        state["W"] = inp["W"]
        return state
    state["plan"], state["X"] = harp.Plan(*inp["processor"]), inp["X"]
    if case["op"] == "grad":
        state["G"] = inp["G"]
    elif case["n"] <= 64:
        state["Y"] = torch.empty_like(state["X"])      # a serving loop keeps its output buffer
    return state


def run(state: dict):
    op = state["op"]
    if op == "apply":
        return harp.harp_apply(state["plan"], state["X"], state.get("Y"))
    if op == "apply_transpose":
        return harp.harp_apply_transpose(state["plan"], state["X"], state.get("Y"))
    if op == "rotate":
        return harp.harp_rotate_weight(state["plan_U"], state["plan_V"], state["W"])
    if op == "unrotate":
        return harp.harp_rotate_weight_inverse(state["plan_U"], state["plan_V"], state["W"])
    dK, dX = harp.harp_grad_blocks(state["plan"], state["X"], state["G"])
    return dK + [dX]


def _parameters(d: int, radices) -> int:
    """Bytes of the free rotation parameters of a processor (sum of d (b - 1) / 2 floats)."""
    return sum(4 * d * (b - 1) // 2 for b in radices)


def work(case: dict) -> dict:
    es = 2 if case["dtype"] == "bf16" else 4
    if case["op"] in ("rotate", "unrotate"):
        do, di = case["d_out"], case["d_in"]
        ru, rv = schedule(do, case["family"]), schedule(di, case["family"])
        return {"bytes": 2 * do * di * es + _parameters(do, ru) + _parameters(di, rv),
                "flops": 2 * do * di * (sum(ru) + sum(rv))}
    n, d, rad = case["n"], case["d"], schedule(case["d"], case["family"])
    if case["op"] == "grad":
        # X and G in, dX and the dense block gradients out; forward, backward and outer products
        return {"bytes": 3 * n * d * es + _parameters(d, rad) + sum(4 * d * b for b in rad),
                "flops": 3 * 2 * n * d * sum(rad)}
    return {"bytes": 2 * n * d * es + _parameters(d, rad), "flops": 2 * n * d * sum(rad)}


def tolerance(case: dict) -> dict:
    """About four times what the path shows against the same maps evaluated in float64: bfloat16
    results carry one rounding (0.0017 in the 2-norm, half a unit in the last place at the most
    plus the half-precision intermediates), float32 ones the sums of up to 13 stages."""
    if case["dtype"] == "bf16":
        return {"rel": 7e-3, "max": 2e-2}
    return {"rel": 1e-6, "max": 2e-5}


def _stage(x: torch.Tensor, K: torch.Tensor, b: int, s: int, transpose: bool) -> torch.Tensor:
    """One stride stage on the rows of x: y[r'] = sum_r x[r] K[c][r][r'] over every digit group."""
    n, d = x.shape
    v, k = x.view(n, d // (b * s), b, s), K.view(d // (b * s), s, b, b)
    if transpose:
        k = k.transpose(2, 3)
    y = torch.zeros_like(v)
    for r in range(b):
        for q in range(b):
            y[:, :, q, :].addcmul_(v[:, :, r, :], k[:, :, r, q])
    return y.view(n, d)


def _on_device(processor) -> tuple:
    """(blocks, radices, strides, signs) in float64 on the device."""
    d, radices, blocks, signs = processor
    K = [torch.from_numpy(np.asarray(k, dtype=np.float64)).cuda() for k in blocks]
    strides = [math.prod(radices[:t]) for t in range(len(radices))]
    return K, radices, strides, torch.from_numpy(signs.astype(np.float64)).cuda()


def _rows_times_U(x: torch.Tensor, processor, transpose: bool) -> torch.Tensor:
    K, rad, st, sg = _on_device(processor)
    order = range(len(rad) - 1, -1, -1) if transpose else range(len(rad))
    x = x if transpose else x * sg
    for t in order:
        x = _stage(x, K[t], rad[t], st[t], transpose)
    return x * sg if transpose else x


def exact(case: dict, seed: int):
    """The outputs of ``run`` in float64 from the definition, stage by stage."""
    inp, op = _inputs(case, seed), case["op"]
    if op in ("rotate", "unrotate"):
        back = op == "unrotate"
        w = _rows_times_U(inp["W"].double(), inp["V"], back)
        return _rows_times_U(w.t().contiguous(), inp["U"], back).t().contiguous()
    if op != "grad":
        return _rows_times_U(inp["X"].double(), inp["processor"], op == "apply_transpose")
    K, rad, st, sg = _on_device(inp["processor"])
    xs = [inp["X"].double() * sg]
    for t in range(len(rad)):
        xs.append(_stage(xs[t], K[t], rad[t], st[t], False))
    g, dK = inp["G"].double(), [None] * len(rad)
    n, d = g.shape
    for t in range(len(rad) - 1, -1, -1):
        b, s = rad[t], st[t]
        x4, g4 = xs[t].view(n, d // (b * s), b, s), g.view(n, d // (b * s), b, s)
        dK[t] = torch.stack([torch.stack([(x4[:, :, r, :] * g4[:, :, q, :]).sum(0).reshape(-1)
                                          for q in range(b)], -1) for r in range(b)], -2)
        g = _stage(g, K[t], b, s, True)
    return dK + [g * sg]
