"""The work that a user of this library has it do, as cases that can be timed and compared.

A case is one call sequence of the draft layer's training through the public binding:

  steps     the training order: k forward calls (step j needs the output of step j - 1), then k
            backward calls in descending order with the fp32 carry between them
  all       all steps in one forward and one backward call (recomputation, benchmarks)
  final     the last step alone, forward without a workspace and backward (the setting of the paper's
            attention micro-benchmark)
  docsteps  a packed batch whose documents take different numbers of steps
  loss      the in-place backward of the log-softmax loss over the logits of all steps
  proj      what stands around the attention: the Q/K/V projection with the rotary embedding, and
            the output projection

Inputs are seeded Gaussians drawn on the GPU (the attention never sees the content of a corpus, only
its lengths and head geometry), as in paper_2603_18567_amd/workloads.py.
"""
import math
import random

import torch

from paper_2603_18567_amd import TttAttnRunner
from paper_2603_18567_amd import binding as B
from paper_2603_18567_amd.workloads import custom_workload, varlen_doc_lens

DEV = "cuda:0"
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
ATTENTION = ("steps", "all", "final", "docsteps")


def _attn(kind, dtype, tokens, doc_lo, doc_hi, hq, hkv, d, k, doc_seed=0):
    """Documents: lengths uniform in [doc_lo, doc_hi] until `tokens` are full (doc_lo = doc_hi = a
    divisor of tokens: equal documents)."""
    return dict(kind=kind, dtype=dtype, tokens=tokens, doc_lo=doc_lo, doc_hi=doc_hi, doc_seed=doc_seed, hq=hq, hkv=hkv, d=d, k=k)


def _loss(dtype, rows, vocab):
    return dict(kind="loss", dtype=dtype, rows=rows, vocab=vocab)


def _proj(tokens, hidden_in, hq, hkv, out_features):
    return dict(kind="proj", dtype="bf16", tokens=tokens, hidden_in=hidden_in, hq=hq, hkv=hkv, out_features=out_features)


def listed():
    cases = {
        # the fp32 configuration that everything is first checked with: latency and launches
        "tiny_f32": _attn("all", "f32", 128, 128, 128, 4, 4, 64, 3),
        # a small draft layer on a short ragged batch, trained step by step: many small calls
        "small_steps_d64": _attn("steps", "bf16", 500, 40, 180, 8, 2, 64, 4, doc_seed=23),
        # the Llama-3.1-8B-shaped draft layer at a short training length, in the training order
        "steps_2k": _attn("steps", "bf16", 2048, 2048, 2048, 32, 8, 128, 7),
        # the benchmark's workload: the paper's micro-benchmark length, all steps in one call
        "all_4k": _attn("all", "bf16", 4096, 4096, 4096, 32, 8, 128, 7),
        # a packed batch of documents in the training order
        "steps_varlen_16k": _attn("steps", "bf16", 16384, 256, 4096, 32, 8, 128, 7, doc_seed=1237),
        # the Qwen3-235B-A22B-shaped draft layer (16 query heads per kv head), two long sequences
        "all_2x8k_g16": _attn("all", "bf16", 16384, 8192, 8192, 64, 4, 128, 7),
        # the last step alone at the short end of the micro-benchmark's sweep
        "final_1k": _attn("final", "bf16", 1024, 1024, 1024, 32, 8, 128, 7),
        # a packed batch whose documents take between 1 and 12 steps
        "docsteps_16k": _attn("docsteps", "bf16", 16384, 256, 4096, 32, 8, 128, 12, doc_seed=1237),
        # logits of one training batch over all steps: 4096 tokens x 7 steps, draft vocabulary
        "loss_draft_vocab": _loss("f32", 28672, 32000),
        # one step's logits over a full vocabulary (a draft model without a reduced vocabulary)
        "loss_full_vocab": _loss("bf16", 4096, 151936),
        # projections of the draft layer (token embedding and target hidden state side by side)
        "proj_4k": _proj(4096, 8192, 32, 8, 4096),
        # the same layer on a short ragged batch: the weights outweigh the activations
        "proj_200": _proj(200, 8192, 32, 8, 4096),
    }
    return [dict(case, name=name) for name, case in cases.items()]


def _log_uniform(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("steps", "steps", "all", "all", "final", "docsteps", "loss", "loss", "proj", "proj"))
    if kind == "loss":
        return _loss(rng.choice(("f32", "bf16")), _log_uniform(rng, 64, 8192), _log_uniform(rng, 1000, 152000))
    if kind == "proj":
        hq, hkv = rng.choice(((32, 8), (64, 4), (16, 16), (24, 8), (12, 2)))
        return _proj(_log_uniform(rng, 16, 8192), 64 * rng.randint(16, 128), hq, hkv, 128 * rng.randint(8, 48))
    limit = max(work(c)["flops"] for c in listed() if c["kind"] in ATTENTION)
    while True:
        f32 = rng.random() < 0.15
        tokens = _log_uniform(rng, 100, 700) if f32 else _log_uniform(rng, 128, 16384)
        if rng.random() < 0.5:
            lo = hi = tokens
        else:
            hi = _log_uniform(rng, 64, min(tokens, 4096))
            lo = max(1, hi // rng.choice((2, 4, 16)))
        hq, hkv = rng.choice(((32, 8), (64, 4), (16, 16), (24, 8), (12, 2), (8, 1), (8, 2)))
        case = _attn(kind, "f32" if f32 else "bf16", tokens, lo, hi, hq, hkv, rng.choice((64, 128, 128)), rng.randint(1, 12),
                     doc_seed=rng.randint(1, 10 ** 6))
        if work(case)["flops"] <= limit:
            return case


def _documents(case):
    lens = varlen_doc_lens(case["tokens"], case["doc_lo"], case["doc_hi"], case["doc_seed"])
    rng = random.Random(case["doc_seed"] + 1)
    steps = [rng.randint(1, case["k"]) if case["kind"] == "docsteps" else case["k"] for _ in lens]
    return lens, steps


def _workload(case):
    lens, _ = _documents(case)
    return custom_workload(case["kind"], case["dtype"], lens, case["hq"], case["hkv"], case["d"], case["k"], 0)


def prepare(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    dtype = DTYPES[case["dtype"]]

    def randn(*shape, mult=1.0):
        x = torch.randn(shape, generator=gen, device=DEV)
        return (x * mult if mult != 1.0 else x).to(dtype)

    if case["kind"] == "loss":
        n, v = case["rows"], case["vocab"]
        z = randn(n, v, mult=3.0)
        p = torch.rand(n, v, generator=gen, device=DEV).pow_(6)
        p = p.div_(p.sum(1, keepdim=True)).to(dtype)
        return dict(case=case, z=z, p=p, g=torch.randn(n, generator=gen, device=DEV))
    if case["kind"] == "proj":
        t, h, hq, hkv, f = (case[x] for x in ("tokens", "hidden_in", "hq", "hkv", "out_features"))
        d, n_pos = 128, 4096
        angle = torch.arange(n_pos, device=DEV)[:, None] * 10000.0 ** (-torch.arange(d // 2, device=DEV) / (d // 2))
        return dict(case=case, x=randn(t, h), w=randn((hq + 2 * hkv) * d, h, mult=h ** -0.5), cos=angle.cos(), sin=angle.sin(),
                    pos=torch.randint(0, n_pos, (t,), generator=gen, device=DEV, dtype=torch.int32),
                    q=torch.empty(t, hq, d, dtype=dtype, device=DEV), k=torch.empty(t, hkv, d, dtype=dtype, device=DEV),
                    v=torch.empty(t, hkv, d, dtype=dtype, device=DEV),
                    o=randn(t, hq, d), wo=randn(f, hq * d, mult=(hq * d) ** -0.5), out=torch.empty(t, f, dtype=dtype, device=DEV))
    wl = _workload(case)
    t, hq, hkv, d = wl.T, wl.hq, wl.hkv, wl.d
    q, k, v, d_o = ([randn(t, h, d) for _ in range(wl.k)] for h in (hq, hkv, hkv, hq))
    run = TttAttnRunner(q, k, v, wl.cu_seqlens, wl.scale, DEV)
    run.alloc_grads()
    if case["kind"] == "docsteps":   # rows of steps that a document does not take keep their contents
        for ts in (run.o, run.lse, run.dq, run.dk, run.dv):
            for x in ts:
                x.zero_()
    return dict(case=case, run=run, d_o=d_o, doc_steps=_documents(case)[1])


def run(state):
    kind = state["case"]["kind"]
    if kind == "loss":
        B.ttt_loss_bwd_inplace(state["z"], state["p"], state["g"])
        return state["z"]
    if kind == "proj":
        B.ttt_qkv_rope_fwd(*(state[x] for x in ("x", "w", "cos", "sin", "pos", "q", "k", "v")))
        B.ttt_o_proj_fwd(state["o"], state["wo"], state["out"])
        return {x: state[x] for x in ("q", "k", "v", "out")}
    r, d_o = state["run"], state["d_o"]
    first = 0
    if kind == "steps":
        for j in range(r.K):
            r.forward(j, j + 1)
        for j in reversed(range(r.K)):
            r.backward(d_o, j, j + 1, accumulate=True)
    elif kind == "all":
        r.forward()
        r.backward(d_o)
    elif kind == "docsteps":
        r.forward_docsteps(state["doc_steps"])
        r.backward_docsteps(d_o, state["doc_steps"])
    else:
        first = r.K - 1
        B.ttt_attn_fwd_static(r.params(first, r.K), r.q, r.k, r.v, r.cu_dev, r.cu_host, r.o, r.lse)
        r.backward(d_o, first, r.K)
    return {"o": r.o[first:], "lse": r.lse[first:], "dq": r.dq[first:], "dk": r.dk, "dv": r.dv}


def work(case):
    e = 4 if case["dtype"] == "f32" else 2
    if case["kind"] == "loss":
        n, v = case["rows"], case["vocab"]
        return {"bytes": 3 * n * v * e + 4 * n, "flops": 6 * n * v}
    if case["kind"] == "proj":
        t, h, f, n_q = case["tokens"], case["hidden_in"], case["out_features"], case["hq"] * 128
        n_kv = 2 * case["hkv"] * 128
        return {"bytes": e * (t * (h + n_q + n_kv) + (n_q + n_kv) * h + t * (n_q + f) + n_q * f), "flops": 2 * t * ((n_q + n_kv) * h + n_q * f)}
    # visible pairs times query heads: the causal prefix of each step and the later blocks' own keys;
    # rows of Q, O, dO, dQ and of K, V, dK, dV
    lens, steps = _documents(case)
    pairs = q_rows = kv_rows = 0
    for n, s in zip(lens, steps):
        taken = (s - 1,) if case["kind"] == "final" else range(s)
        pairs += sum(n * (n + 1) // 2 + n * j for j in taken)
        q_rows += n * len(taken)
        kv_rows += n * s
    q_el, kv_el = q_rows * case["hq"] * case["d"], kv_rows * case["hkv"] * case["d"]
    return {"bytes": 4 * e * (q_el + kv_el) + 4 * q_rows * case["hq"], "flops": 14 * case["d"] * case["hq"] * pairs}


def tolerance(case):
    """Three to four times what a pass differs from the same operation in 64 bits: the largest seen were, in bf16,
    2.9e-3 (2-norm) and 0.28 (one element of dK, where thousands of rounded p and ds cancel) for the
    attention, 1.9e-3 and 3.9e-3 (one rounding) for the others; in fp32 6.0e-7 and 1.2e-5 for the
    attention, 1.1e-7 and 7.0e-7 for the loss."""
    attention = case["kind"] in ATTENTION
    if case["dtype"] == "bf16":
        return {"rel": 1.1e-2, "max": 0.9} if attention else {"rel": 7.5e-3, "max": 1.6e-2}
    return {"rel": 2.4e-6, "max": 5e-5} if attention else {"rel": 4.4e-7, "max": 2.8e-6}
