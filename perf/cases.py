"""Measured cases: the products a transformer program has this library compute.

Each case is one pass through the public entry points of
``paper_2309_08978_amd`` on operands that already lie on the GPU, the way a
serving program calls them: weights and output buffers are kept, fixed layer
shapes are tuned once beforehand (``tune`` true), attention shapes that follow
the sequence length are not (``tune`` false), because the length changes from
request to request and from step to step.

Kinds of case

``linear``     C[M, N] = A[M, K] . B[K, N], activations times a weight
               (M = 1 is the decode step)
``linear_q4``  y[N] = x[K] . W for a 4-bit weight with one fp16 scale per
               output and group of inputs
``attention``  the two products of one attention layer over ``heads`` (batch
               times heads): scores[q, s] = Q[q, d] . K^T[d, s], then
               out[q, d] = P[q, s] . V[s, d] with given probabilities P.
               ``cache`` > 0: K^T and V are views of the first ``s`` positions
               of cache buffers that hold ``cache`` positions
``dtype``      ``f32`` or ``f16`` operands; results are fp32

Values: activations N(0, 1), weights N(0, 0.02), probabilities the row softmax
of N(0, 1) logits (causal where ``causal`` is true), 4-bit codes uniform,
scales uniform in [0.002, 0.01).
"""
from __future__ import annotations

import math

import torch

import paper_2309_08978_amd as nj

_DT = {"f32": torch.float32, "f16": torch.float16}


def _linear(name, M, K, N, dtype):
    return {"name": name, "kind": "linear", "M": M, "K": K, "N": N, "dtype": dtype, "tune": True}


def _attention(name, heads, q, s, d, dtype, causal, cache=0, tune=False):
    return {"name": name, "kind": "attention", "heads": heads, "q": q, "s": s, "d": d, "dtype": dtype,
            "causal": causal, "cache": cache, "tune": tune}


def listed():
    return [
        # the smallest call: one small projection, bound by latency and launches
        _linear("proj_64x768x768_f32", 64, 768, 768, "f32"),
        # second feed-forward product of a base-size encoder layer over a short
        # sequence: few output tiles, a long sum
        _linear("bart_ffn_down_f32", 128, 3072, 768, "f32"),
        # first feed-forward product of a large encoder layer, 4 sequences of 256
        _linear("t5_ffn_up_f32", 1024, 1024, 4096, "f32"),
        # vocabulary head of a 7B decoder over a 512-token prompt: the largest call
        _linear("llama_prefill_lm_head_f32", 512, 4096, 32000, "f32"),
        # feed-forward product of the same prompt in half precision
        _linear("llama_prefill_gate_f16", 512, 4096, 11008, "f16"),
        # decode step: one token through the smallest and the longest linears
        _linear("llama_decode_o_f16", 1, 4096, 4096, "f16"),
        _linear("llama_decode_down_f32", 1, 11008, 4096, "f32"),
        # decode step on 4-bit weights
        {"name": "llama_decode_gate_q4", "kind": "linear_q4", "K": 4096, "N": 11008, "group": 128, "tune": True},
        # attention of the large encoder layer: a fixed length, tuned
        _attention("t5_attention_f32", 64, 256, 256, 64, "f32", False, tune=True),
        # attention over a sequence of odd length (an encoder's request as it came)
        _attention("ragged_attention_f32", 12, 197, 197, 64, "f32", False),
        # causal prompt attention of odd length in half precision
        _attention("ragged_prefill_attention_f16", 32, 333, 333, 128, "f16", True),
        # decode attention: one query against a partly filled cache
        _attention("decode_attention_f16", 32, 1, 1023, 128, "f16", False, cache=2048),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: widths of base- to 7B-size layers,
    1 to 1024 rows, sequences of 16 to 1024, odd sizes among them."""
    pick = rng.random()
    dtype = rng.choice(["f32", "f16"])
    if pick < 0.35:
        # prompt or encoder linear: the rows are whatever the request has; widths
        # are multiples of 8, as layer widths are
        M = _log_int(rng, 16, 1024)
        K = 8 * _log_int(rng, 512 // 8, 11008 // 8)
        N = 8 * _log_int(rng, 512 // 8, 32000 // 8)
        while M * K * N > 512 * 4096 * 32000:
            N = max(512, N // 2 // 8 * 8)
            M = max(16, M // 2)
        return {"kind": "linear", "M": M, "K": K, "N": N, "dtype": dtype, "tune": True}
    if pick < 0.55:
        return {"kind": "linear", "M": 1, "K": 8 * _log_int(rng, 512 // 8, 11008 // 8),
                "N": 8 * _log_int(rng, 512 // 8, 32000 // 8), "dtype": dtype, "tune": True}
    if pick < 0.7:
        group = rng.choice([32, 64, 128])
        return {"kind": "linear_q4", "K": group * _log_int(rng, max(4, 512 // group), 11008 // group),
                "N": 8 * _log_int(rng, 512 // 8, 32000 // 8), "group": group, "tune": True}
    d = rng.choice([64, 128])
    if pick < 0.9:
        s = _log_int(rng, 16, 1024)
        return {"kind": "attention", "heads": rng.choice([12, 16, 32, 64]), "q": s, "s": s, "d": d, "dtype": dtype,
                "causal": rng.random() < 0.5, "cache": 0, "tune": rng.random() < 0.3}
    return {"kind": "attention", "heads": rng.choice([12, 16, 32, 64]), "q": 1, "s": _log_int(rng, 16, 2048), "d": d,
            "dtype": dtype, "causal": False, "cache": 2048, "tune": False}


def _inputs(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * (seed + 1) + 17)

    def normal(*shape, scale=1.0):
        t = torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)
        return t if scale == 1.0 else t.mul_(scale)

    if case["kind"] == "linear":
        dt = _DT[case["dtype"]]
        return normal(case["M"], case["K"]).to(dt), normal(case["K"], case["N"], scale=0.02).to(dt)
    if case["kind"] == "linear_q4":
        K, N, group = case["K"], case["N"], case["group"]
        x = normal(K).to(torch.float16)
        words = torch.randint(-(1 << 31), 1 << 31, (N, -(-K // 8)), generator=g, device="cuda", dtype=torch.int64)
        scales = torch.rand((N, -(-K // group)), generator=g, device="cuda") * 0.008 + 0.002
        return x, words.to(torch.int32), scales.to(torch.float16)
    dt = _DT[case["dtype"]]
    h, q, s, d = case["heads"], case["q"], case["s"], case["d"]
    room = max(case["cache"], s)
    Q = normal(h, q, d).to(dt)
    Kt = normal(h, d, room).to(dt)[:, :, :s]
    logits = normal(h, q, s)
    if case["causal"]:
        logits = logits.masked_fill(torch.ones((q, s), dtype=torch.bool, device="cuda").triu(1), float("-inf"))
    P = torch.softmax(logits, dim=-1).to(dt)
    V = normal(h, room, d).to(dt)[:, :s, :]
    return Q, Kt, P, V


def prepare(case, seed):
    ops = _inputs(case, seed)
    code = nj.NNJIT_F16 if case.get("dtype") == "f16" else nj.NNJIT_F32
    if case["kind"] == "linear":
        if case["tune"]:
            nj.check(nj.nnjit_tune(case["M"], case["N"], case["K"], code))
        out = (torch.empty((case["M"], case["N"]), dtype=torch.float32, device="cuda"),)
    elif case["kind"] == "linear_q4":
        if case["tune"]:
            nj.check(nj.nnjit_tune_gemv_q4(case["N"], case["K"], case["group"]))
        out = (torch.empty((case["N"],), dtype=torch.float32, device="cuda"),)
    else:
        h, q, s, d = case["heads"], case["q"], case["s"], case["d"]
        if case["tune"]:
            nj.check(nj.nnjit_tune_batched(h, q, s, d, code))
            nj.check(nj.nnjit_tune_batched(h, q, d, s, code))
        out = (torch.empty((h, q, s), dtype=torch.float32, device="cuda"),
               torch.empty((h, q, d), dtype=torch.float32, device="cuda"))
    return {"case": case, "in": ops, "out": out}


def run(state):
    case, ops, out = state["case"], state["in"], state["out"]
    if case["kind"] == "linear":
        return nj.matmul(ops[0], ops[1], out[0])
    if case["kind"] == "linear_q4":
        return nj.gemv_q4(ops[0], ops[1], ops[2], case["group"], case["N"], out[0])
    scores = nj.batched_matmul(ops[0], ops[1], out[0])
    return scores, nj.batched_matmul(ops[2], ops[3], out[1])


def work(case):
    if case["kind"] == "linear_q4":
        K, N, group = case["K"], case["N"], case["group"]
        return {"bytes": K * 2 + N * (-(-K // 8)) * 4 + N * (-(-K // group)) * 2 + N * 4, "flops": 2 * K * N}
    e = 2 if case["dtype"] == "f16" else 4
    if case["kind"] == "linear":
        M, K, N = case["M"], case["K"], case["N"]
        return {"bytes": (M * K + K * N) * e + M * N * 4, "flops": 2 * M * K * N}
    h, q, s, d = case["heads"], case["q"], case["s"], case["d"]
    return {"bytes": h * ((q * d + d * s + q * s + s * d) * e + (q * s + q * d) * 4), "flops": 4 * h * q * s * d}


def tolerance(case):
    """fp32 sums of exact products: the rounding of a sum of K terms, taken in
    any order, grows at most like sqrt(K).  Four times the errors measured
    against fp64: 1.8e-8 sqrt(K) where fp32 operands are summed one or two
    terms at a time, 6.4e-9 sqrt(K) where fp16 operands are summed 8 or 16
    terms at a time, 1.8e-9 sqrt(K) where many lanes share one sum (M = 1)."""
    if case["kind"] == "attention":
        K, c = max(case["d"], case["s"]), 7e-8 if case["dtype"] == "f32" else 3e-8
    elif case["kind"] == "linear_q4" or case["M"] == 1:
        K, c = case["K"], 1e-8
    else:
        K, c = case["K"], 7e-8 if case["dtype"] == "f32" else 3e-8
    return {"rel": 2e-7 + c * math.sqrt(K)}


def exact(case, seed):
    ops = _inputs(case, seed)
    if case["kind"] == "linear":
        return ops[0].double() @ ops[1].double()
    if case["kind"] == "linear_q4":
        x, words, scales = ops
        K, N, group = case["K"], case["N"], case["group"]
        shifts = torch.arange(0, 32, 4, device="cuda", dtype=torch.int32)
        q = ((words.unsqueeze(-1) >> shifts) & 15).reshape(N, -1)[:, :K].double() - 8.0
        w = q * scales.double().repeat_interleave(group, dim=1)[:, :K]
        return w @ x.double()
    Q, Kt, P, V = (t.double().contiguous() for t in ops)
    return torch.bmm(Q, Kt), torch.bmm(P, V)
