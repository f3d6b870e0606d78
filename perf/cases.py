"""Performance cases of the attention forward: the calls that users of this library make, each through a
public entry point, with its inputs, its minimal work, its tolerance and a 64-bit reference.

A case is a dict of plain values:
  kind     "prefill" (``forward``), "split" (``forward(n_split="auto")``), "decode"
           (``forward(decode=True, n_split="auto")``), "noalloc" (``fa_fwd_decode_noalloc`` into buffers
           the program keeps, as a serving loop calls it) or "unfused" (``forward_unfused``)
  B, Hq, Hkv, Sq, Sk, dqk, dv, causal, lse   sizes and options (lse: the call also returns the
           log-sum-exp)
Inputs are i.i.d. N(0, 1) in bfloat16, the regime of normalised activations, as in ``workloads``.
"""

from __future__ import annotations

import math

import torch

import paper_2609_21264_amd as fa
import workloads

HEAD_DIMS = ((64, 64), (128, 128), (192, 128))


def _case(name, kind, B, Hq, Hkv, Sq, Sk, dqk, dv, causal, lse=False):
    return {"name": name, "kind": kind, "B": B, "Hq": Hq, "Hkv": Hkv, "Sq": Sq, "Sk": Sk, "dqk": dqk, "dv": dv,
            "causal": causal, "lse": lse}


def listed():
    return [
        # One head over a short sequence: the smallest call, where launch and host latency count.
        _case("single_head_256", "prefill", 1, 1, 1, 256, 256, 64, 64, False),
        # An encoder layer's batch at BERT-base's shape.
        _case("bert_base_512", "prefill", 8, 12, 12, 512, 512, 64, 64, False),
        # GPT-2 Small's attention layer at one of the paper's sweep lengths.
        _case("gpt2_small_2048", "prefill", 1, 12, 12, 2048, 2048, 64, 64, True),
        # Long-context prefill with 64-wide heads and a 7:1 group (Qwen2.5-0.5B's shape, Table 6).
        _case("qwen25_32k", "prefill", 1, 14, 2, 32768, 32768, 64, 64, True),
        # Llama-style GQA prefill, with the log-sum-exp that a training step or a later merge keeps.
        _case("llama_gqa_8k", "prefill", 1, 32, 8, 8192, 8192, 128, 128, True, True),
        # DeepSeek-style wide-head prefill, d_qk = 192 and d_v = 128, no sharing of K/V heads.
        _case("wide_head_4k", "prefill", 1, 128, 128, 4096, 4096, 192, 128, True),
        # The flagship benchmark: 128K tokens of context.
        _case("llama_gqa_128k", "prefill", 1, 32, 8, 131072, 131072, 128, 128, True),
        # A chunk of a prompt against a cache that is longer than it: ragged lengths, 7:1 group, a batch.
        _case("chunk_777_of_5001", "prefill", 2, 28, 4, 777, 5001, 128, 128, True, True),
        # One new token against a 128K cache.
        _case("decode_128k", "decode", 1, 32, 8, 1, 131072, 128, 128, False),
        # A serving step: one token for each of 16 requests against caches of an odd length, without
        # allocation.
        _case("serve_b16_4099", "noalloc", 16, 32, 8, 1, 4099, 128, 128, True),
        # A short chunk (a prompt's last piece, or draft tokens) against a long cache in split mode.
        _case("split_100_of_32k", "split", 1, 32, 8, 100, 32768, 128, 128, True),
        # The layer-by-layer baseline at a 7B model's prefill.
        _case("unfused_4k", "unfused", 1, 32, 32, 4096, 4096, 128, 128, True),
    ]


def _log(rng, lo, hi):
    """An integer of [lo, hi], uniform over its logarithm (so odd and even alike)."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the listed ranges: kinds, head dimensions, group sizes, lengths, batches and
    options at random, scaled down in heads and batch until it costs no more than the largest listed
    cases of its kind."""
    kind = rng.choice(["prefill", "prefill", "prefill", "split", "decode", "noalloc", "unfused"])
    dqk, dv = rng.choice(HEAD_DIMS)
    hkv, group, batch = rng.choice([1, 2, 4, 8, 12, 16]), rng.choice([1, 1, 2, 4, 7, 8]), rng.choice([1, 1, 2, 3, 8])
    causal, lse = rng.random() < 0.6, rng.random() < 0.4
    if kind == "prefill":
        sk = _log(rng, 128, 65536)
        sq = sk if rng.random() < 0.6 else _log(rng, 64, sk)
        limit = 4e12  # flops
    elif kind == "split":
        sq, sk, limit = _log(rng, 16, 512), _log(rng, 4096, 131072), 5e11
    elif kind == "unfused":
        sk = _log(rng, 256, 8192)
        sq, limit = sk, 3e11
    else:
        sq, sk, batch = rng.choice([1, 1, 1, 2, 4]), _log(rng, 512, 131072), rng.choice([1, 4, 16, 64])
        hkv = max(hkv, 2)
        limit = 7e8  # bytes, below
    c = _case("", kind, batch, hkv * group, hkv, sq, sk, dqk, dv, causal, lse)
    del c["name"]
    cost = "bytes" if kind in ("decode", "noalloc") else "flops"
    while work(c)[cost] > limit and (c["B"] > 1 or c["Hkv"] > 1):
        if c["B"] > 1:
            c["B"] = (c["B"] + 1) // 2
        else:
            c["Hkv"] = (c["Hkv"] + 1) // 2
            c["Hq"] = c["Hkv"] * group
    return c


def prepare(case, seed):
    """The inputs on the GPU, and for a serving loop the output buffers and part count that it keeps."""
    c = case
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    shapes = ((c["B"], c["Hq"], c["Sq"], c["dqk"]), (c["B"], c["Hkv"], c["Sk"], c["dqk"]),
              (c["B"], c["Hkv"], c["Sk"], c["dv"]))
    q, k, v = (torch.randn(s, dtype=torch.bfloat16, device="cuda", generator=g) for s in shapes)
    state = {"case": c, "q": q, "k": k, "v": v}
    if c["kind"] == "noalloc":
        state["o"] = torch.empty((c["B"], c["Hq"], c["Sq"], c["dv"]), dtype=torch.bfloat16, device="cuda")
        state["lse"] = (torch.empty((c["B"], c["Hq"], c["Sq"]), dtype=torch.float32, device="cuda")
                        if c["lse"] else None)
        n_cu = torch.cuda.get_device_properties("cuda").multi_processor_count
        state["parts"] = fa.fa_fwd_decode_parts(n_cu, c["B"], c["Hq"], c["Hkv"], c["Sq"], c["Sk"])
    return state


def run(state):
    """One call; returns [O] or [O, LSE]."""
    c, q, k, v = state["case"], state["q"], state["k"], state["v"]
    kind, causal, lse = c["kind"], c["causal"], c["lse"]
    if kind == "noalloc":
        o, ls = state["o"], state["lse"]
        st = fa.fa_fwd_decode_noalloc(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(),
                                      ls.data_ptr() if lse else None, c["B"], c["Hq"], c["Hkv"], c["Sq"], c["Sk"],
                                      c["dqk"], c["dv"], 1.0 / math.sqrt(c["dqk"]), causal, state["parts"],
                                      torch.cuda.current_stream().cuda_stream)
        if st != fa.FA_OK:
            raise fa.FaError(st)
        return [o, ls] if lse else [o]
    if kind == "prefill":
        out = fa.forward(q, k, v, causal=causal, return_lse=lse)
    elif kind == "split":
        out = fa.forward(q, k, v, causal=causal, return_lse=lse, n_split="auto")
    elif kind == "decode":
        out = fa.forward(q, k, v, causal=causal, return_lse=lse, n_split="auto", decode=True)
    else:
        out = fa.forward_unfused(q, k, v, causal=causal, return_lse=lse)
    return list(out) if lse else [out]


def _workload(c):
    return workloads.Workload(name="", B=c["B"], Hq=c["Hq"], Hkv=c["Hkv"], Sq=c["Sq"], Sk=c["Sk"], dqk=c["dqk"],
                              dv=c["dv"], causal=c["causal"], scale=1.0 / math.sqrt(c["dqk"]), seed=0)


def work(case):
    """Bytes: Q, K, V read once and O (and LSE) written once; the layer-by-layer path also writes and
    reads its scores and probabilities, which is what that path is. Flops: the two products over the
    visible pairs."""
    w = _workload(case)
    flops = 2.0 * workloads.visible_scores(w) * (w.dqk + w.dv)
    if case["kind"] == "unfused":
        nbytes = sum(workloads.unfused_algorithmic_bytes(w).values())
        if not case["lse"]:
            nbytes -= 4 * w.B * w.Hq * w.Sq
    else:
        nbytes = workloads.algorithmic_bytes(w, with_lse=case["lse"])
    return {"bytes": float(nbytes), "flops": flops}


def tolerance(case):
    """About four times the distance from the 64-bit result measured over the listed and drawn cases:
    P and O are rounded to bfloat16 (2^-9 relative each), the layer-by-layer path's scores too."""
    return {"rel": 2e-2 if case["kind"] == "unfused" else 1e-2}


def exact(case, seed):
    """softmax(Q K^T / sqrt(d)) V and its log-sum-exp in float64, head by head and over blocks of query
    rows; None where the float64 products would take too long."""
    c = case
    if work(c)["flops"] > 2e13:
        return None
    s = prepare(c, seed)
    q, k, v = s["q"], s["k"], s["v"]
    B, Hq, Hkv, Sq, Sk = (c[n] for n in ("B", "Hq", "Hkv", "Sq", "Sk"))
    o = torch.empty((B, Hq, Sq, c["dv"]), dtype=torch.float64, device="cuda")
    lse = torch.empty((B, Hq, Sq), dtype=torch.float64, device="cuda")
    block = max(1, (1 << 27) // max(Sk, 1))
    for b in range(B):
        for g in range(Hkv):
            kt = k[b, g].double().t().contiguous()
            vd = v[b, g].double()
            for h in range(g * (Hq // Hkv), (g + 1) * (Hq // Hkv)):
                for r0 in range(0, Sq, block):
                    r1 = min(Sq, r0 + block)
                    n = min(Sk, max(0, r1 + Sk - Sq)) if c["causal"] else Sk
                    if n == 0:
                        o[b, h, r0:r1] = 0
                        lse[b, h, r0:r1] = -math.inf
                        continue
                    x = q[b, h, r0:r1].double() @ kt[:, :n].contiguous()
                    x *= 1.0 / math.sqrt(c["dqk"])
                    if c["causal"]:
                        last = torch.arange(r0, r1, device="cuda") + (Sk - Sq)
                        x.masked_fill_(torch.arange(n, device="cuda")[None, :] > last[:, None], -math.inf)
                    m = torch.logsumexp(x, dim=1)
                    lse[b, h, r0:r1] = m
                    x -= torch.where(m == -math.inf, torch.zeros_like(m), m)[:, None]
                    o[b, h, r0:r1] = x.exp_() @ vd[:n]
    return [o, lse] if c["lse"] else [o]
