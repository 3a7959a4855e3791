"""Performance cases: the calls a program makes to this framework, with inputs, work and 64-bit results.

A case is a dict of plain values.  ``kind`` names the entry point:

* ``sgemm``    -- ``sgemm`` with no tile and no workspace given (the library
  chooses, the wrapper allocates), C updated in place;
* ``consumer`` -- ``sgemm_consumer``: the sgemm with its bias + relu consumer;
* ``backward`` -- ``sgemm_backward``: the five gradients of one product;
* ``train``    -- ``sgemm_fn`` and ``torch.autograd.grad`` through it;
* ``grouped``  -- replay of a captured ``GroupedPlan`` (no autotuning);
* ``stream``   -- a streaming session: open, push every item, pop every
  result, close.

``prec`` is the arithmetic ('fp32', 'bf16', 'bf16x3'); storage is float32.
``pad`` > 0 makes every operand a view into rows that are longer by ``pad``.
Sizes of products run from 16 to 8192 a side, of batches' and streams'
instances from 32 to 2048, as in the tests and the benchmark.
"""
from __future__ import annotations

import math
import random

import torch

import paper_1611_00860_amd as hp
from paper_1611_00860_amd.autograd import sgemm_fn

# Multiply-adds of the largest product of each precision.
MOST = {"fp32": 4096 ** 3, "bf16": 8192 ** 3, "bf16x3": 4096 ** 3}
# Products whose matrices together exceed this many floats are not drawn.
MOST_FLOATS = 3 * 8192 ** 2


def listed():
    return [
        # The smallest product: the two-level graph's own small configuration,
        # where the call's latency is what a program waits for.
        dict(name="sgemm_fp32_128", kind="sgemm", prec="fp32", m=128, n=128, k=128,
             alpha=1.0, beta=0.5, dist="uniform", pad=0),
        # A handful of rows against a wide matrix: a small batch through a layer.
        dict(name="sgemm_fp32_16x4096x4096", kind="sgemm", prec="fp32", m=16, n=4096, k=4096,
             alpha=1.0, beta=0.0, dist="uniform", pad=0),
        # Sizes that no tile, slab or vector width divides.
        dict(name="sgemm_fp32_1000x1003x777", kind="sgemm", prec="fp32", m=1000, n=1003, k=777,
             alpha=1.5, beta=1.0, dist="uniform", pad=0),
        # The large FP32 workload, accumulating into C.
        dict(name="sgemm_fp32_4096", kind="sgemm", prec="fp32", m=4096, n=4096, k=4096,
             alpha=1.0, beta=1.0, dist="uniform", pad=0),
        # An ordinary BF16 product, not a multiple of the tiles.
        dict(name="sgemm_bf16_1500x1100x900", kind="sgemm", prec="bf16", m=1500, n=1100, k=900,
             alpha=1.0, beta=0.0, dist="uniform", pad=0),
        # The largest product of the precision workload.
        dict(name="sgemm_bf16_8192", kind="sgemm", prec="bf16", m=8192, n=8192, k=8192,
             alpha=1.0, beta=0.0, dist="uniform", pad=0),
        # Split precision on values of widely different magnitude.
        dict(name="sgemm_bf16x3_3000x2500x2000", kind="sgemm", prec="bf16x3", m=3000, n=2500, k=2000,
             alpha=1.0, beta=0.0, dist="loguniform", pad=0),
        # A layer's forward with its activation: fewer rows than columns.
        dict(name="consumer_512x4096x1024", kind="consumer", prec="fp32", m=512, n=4096, k=1024,
             alpha=1.0, beta=0.0, dist="uniform", pad=0),
        # Gradients of an ordinary product of uneven sides.
        dict(name="backward_fp32_1000x1200x800", kind="backward", prec="fp32", m=1000, n=1200, k=800,
             alpha=0.7, beta=0.3, dist="uniform", pad=0),
        # Forward and backward of the differentiation workload in BF16.
        dict(name="train_bf16_4096x4096x1024", kind="train", prec="bf16", m=4096, n=4096, k=1024,
             alpha=0.7, beta=0.3, dist="uniform", pad=0),
        # Many uneven products in one launch: the batching workload.
        dict(name="grouped_512", kind="grouped", prec="fp32", count=512, low=32, high=2048, multiple=16,
             shapes=3),
        # The same kind of products as a stream of items through one session.
        dict(name="stream_256", kind="stream", prec="fp32", count=256, low=32, high=1024, multiple=16,
             shapes=3, capacity=256),
    ]


def _log(rng, low, high):
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def _size(rng, low, high):
    """A size spread over the logarithm of the range: any integer, or rounded to what programs often have."""
    step = rng.choice((1, 1, 4, 8, 16, 64, 128))
    x = _log(rng, low, high)
    return min(high, max(low, (x + step // 2) // step * step))


def draw(rng: random.Random):
    kind = rng.choice(("sgemm", "sgemm", "sgemm", "sgemm", "sgemm", "consumer", "backward", "train", "grouped",
                       "stream"))
    if kind in ("grouped", "stream"):
        c = dict(kind=kind, prec="fp32", count=_log(rng, 16, 256), low=32,
                 high=rng.choice((256, 512, 1024)), multiple=rng.choice((1, 4, 16)),
                 shapes=rng.randrange(1 << 20))
        if kind == "stream":
            c["capacity"] = rng.choice((64, 256))
        return c
    prec = "fp32" if kind == "consumer" else rng.choice(("fp32", "fp32", "bf16", "bf16x3"))
    passes = {"sgemm": 1, "consumer": 1, "backward": 2, "train": 3}[kind]
    while True:
        m, n, k = (_size(rng, 16, 8192) for _ in range(3))
        if m * n * k * passes <= MOST[prec] and m * k + k * n + passes * m * n <= MOST_FLOATS:
            break
    return dict(kind=kind, prec=prec, m=m, n=n, k=k, alpha=rng.choice((1.0, 0.7, 1.5)),
                beta=rng.choice((0.0, 0.5, 1.0)), dist=rng.choice(("uniform", "uniform", "loguniform")),
                pad=rng.choice((0, 0, 0, 0, 0, 4, 3)))


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _matrix(gen, rows, cols, dist="uniform", pad=0):
    """rows x cols float32 on the GPU: U[-1, 1], or magnitude 2**U(-8, 8) with a random sign."""
    u = torch.rand(rows, cols + pad, device="cuda", generator=gen)
    if dist == "loguniform":
        sign = torch.rand(rows, cols + pad, device="cuda", generator=gen)
        u = torch.exp2(u * 16 - 8).copysign_(sign - 0.5)
    else:
        u = u.mul_(2).sub_(1)
    return u[:, :cols] if pad else u


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _operands(case, seed):
    """A, B, C, then the upstream gradient and the bias where the kind has one."""
    gen = _generator(seed)
    m, n, k, dist, pad = case["m"], case["n"], case["k"], case["dist"], case["pad"]
    ops = {"A": _matrix(gen, m, k, dist, pad), "B": _matrix(gen, k, n, dist, pad),
           "C": _matrix(gen, m, n, "uniform", pad)}
    if case["kind"] in ("backward", "train"):
        ops["G"] = _matrix(gen, m, n, "uniform", pad if case["kind"] == "backward" else 0)
    if case["kind"] == "consumer":
        ops["bias"] = _matrix(gen, 1, n)[0]
    return ops


def _instances(case):
    """(m, n, k, alpha, beta) of every instance: part of the case, not of its inputs."""
    rng = random.Random(case["shapes"])
    step, low, high = case["multiple"], case["low"], case["high"]
    dims = [[min(high, max(low, (_log(rng, low, high) + step // 2) // step * step)) for _ in range(3)]
            for _ in range(case["count"])]
    return [(m, n, k, rng.uniform(0.5, 2.0), rng.uniform(0.0, 1.0)) for m, n, k in dims]


def _batch(case, seed):
    """The instances' (A, B, C, alpha, beta), and the array that holds every C (each 256-byte aligned)."""
    gen = _generator(seed)
    instances = _instances(case)
    starts, total = [], 0
    for m, n, _, _, _ in instances:
        starts.append(total)
        total += (m * n + 63) // 64 * 64
    results = _matrix(gen, 1, total)[0]
    items = [(_matrix(gen, m, k), _matrix(gen, k, n), results[at:at + m * n].view(m, n), alpha, beta)
             for (m, n, k, alpha, beta), at in zip(instances, starts)]
    return items, results


def prepare(case, seed):
    kind = case["kind"]
    state = {"case": case}
    if kind == "grouped":
        items, state["out"] = _batch(case, seed)
        As, Bs, Cs, alphas, betas = (list(x) for x in zip(*items))
        state["plan"] = hp.GroupedPlan(As, Bs, Cs, alphas, betas)
        state["graph"] = state["plan"].capture()
        return state
    if kind == "stream":
        items, state["out"] = _batch(case, seed)
        state["packed"] = [hp.SgemmStream.pack(*x) for x in items]
        # The resident kernel runs beside the caller's stream: the items'
        # data has to be there before the first push.
        torch.cuda.current_stream().synchronize()
        return state
    state.update(_operands(case, seed))
    if kind == "consumer":
        state["D"] = torch.empty(case["m"], case["n"], device="cuda")
    if kind == "train":
        for name in ("A", "B", "C"):
            state[name].requires_grad_(True)
    return state


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "sgemm":
        return hp.sgemm(state["A"], state["B"], state["C"], case["alpha"], case["beta"], prec=case["prec"])
    if kind == "consumer":
        C = state["C"] if case["beta"] != 0.0 else None
        return hp.sgemm_consumer(state["A"], state["B"], C, case["alpha"], case["beta"], op="bias_relu",
                                 bias=state["bias"], D=state["D"])
    if kind == "backward":
        g = hp.sgemm_backward(state["A"], state["B"], state["C"], state["G"], case["alpha"], case["beta"],
                              prec=case["prec"])
        return {name: g[name] for name in ("dA", "dB", "dC_in", "dalpha", "dbeta")}
    if kind == "train":
        A, B, C = state["A"], state["B"], state["C"]
        out = sgemm_fn(A, B, C, case["alpha"], case["beta"], case["prec"])
        dA, dB, dC = torch.autograd.grad(out, (A, B, C), state["G"])
        return {"out": out.detach(), "dA": dA, "dB": dB, "dC_in": dC}
    if kind == "grouped":
        state["graph"].launch()
        return state["out"]
    # stream: results come in push order; a full ring is drained by popping.
    with hp.SgemmStream(capacity=case["capacity"]) as stream:
        for packed in state["packed"]:
            if stream.in_flight == case["capacity"]:
                stream.pop()
            stream.push_packed(packed)
        while stream.in_flight:
            stream.pop()
    return state["out"]


# ---------------------------------------------------------------------------
# Work and exact results
# ---------------------------------------------------------------------------
def work(case):
    if case["kind"] in ("grouped", "stream"):
        dims = _instances(case)
        return {"bytes": sum(4 * (m * k + k * n + 2 * m * n) for m, n, k, _, _ in dims),
                "flops": sum(2 * m * n * k for m, n, k, _, _ in dims)}
    m, n, k = case["m"], case["n"], case["k"]
    forward = m * k + k * n + (2 if case["beta"] != 0.0 else 1) * m * n
    # Backward: A, B, G read once, dA, dB, dC_in written (and C_in read for dbeta).
    grads = 2 * (m * k + k * n) + 2 * m * n
    if case["kind"] == "consumer":
        return {"bytes": 4 * (forward + n), "flops": 2 * m * n * k}
    if case["kind"] == "backward":
        return {"bytes": 4 * (grads + m * n), "flops": 4 * m * n * k}
    if case["kind"] == "train":
        return {"bytes": 4 * (forward + grads), "flops": 6 * m * n * k}
    return {"bytes": 4 * forward, "flops": 2 * m * n * k}


def exact(case, seed):
    if case["kind"] in ("grouped", "stream"):
        items, results = _batch(case, seed)
        out = results.double()
        for A, B, C, alpha, beta in items:
            at = C.storage_offset()
            out[at:at + C.numel()] = (alpha * (A.double() @ B.double()) + beta * C.double()).reshape(-1)
        return out
    x = {name: t.double() for name, t in _operands(case, seed).items()}
    A, B, C, alpha, beta = x["A"], x["B"], x["C"], case["alpha"], case["beta"]
    if case["kind"] == "backward":
        G = x["G"]
        return {"dA": alpha * (G @ B.t()), "dB": alpha * (A.t() @ G), "dC_in": beta * G,
                "dalpha": (G * (A @ B)).sum(), "dbeta": (G * C).sum()}
    out = alpha * (A @ B) + beta * C
    if case["kind"] == "train":
        G = x["G"]
        return {"out": out, "dA": alpha * (G @ B.t()), "dB": alpha * (A.t() @ G), "dC_in": beta * G}
    return torch.relu(out + x["bias"]) if case["kind"] == "consumer" else out
