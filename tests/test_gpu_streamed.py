"""GPU tests of the instances chosen by the size of the data: the layer-by-layer operators and the decode
kernel load and store non-temporally when their data is large, the softmax kernel has an instance per row
length, and a decode call of a single part writes its result without the merge."""

import pytest
import torch

import paper_2609_21264_amd as fa
import test_gpu_lbl as lbl
import workloads as W
from oracle import naive_attention
from parity import compare, to_f64

pytestmark = pytest.mark.gpu


def _bits(t):
    return t.view(torch.int16 if t.dtype == torch.bfloat16 else torch.int32)


@pytest.mark.parametrize("B,Hq,Hkv,Sq,Sk,dqk,dv,causal", [
    (2, 14, 14, 2100, 2100, 64, 64, False),
    (1, 56, 8, 2050, 2050, 128, 128, True),
    (1, 24, 24, 1000, 4300, 192, 128, True),
    # the softmax instances of the shorter rows, and sweeps over few key tiles that start anywhere in them
    (1, 900, 900, 1000, 100, 64, 64, False),
    (2, 1000, 125, 301, 300, 64, 64, True),
    (1, 180, 90, 701, 700, 128, 64, False),
    (1, 360, 45, 690, 701, 64, 128, True),
    (1, 40, 40, 1501, 1500, 192, 128, False),
    (1, 80, 80, 1499, 1497, 64, 64, True),
])
def test_streamed_spill_equals_cached(B, Hq, Hkv, Sq, Sk, dqk, dv, causal):
    """The whole problem in one chunk (its visible scores exceed 160 MiB: streamed) against chunks of one
    group of heads (below it: cached). The operators do the same arithmetic in the same order, so the
    results are the same bits; the cached path is checked against the oracle in test_gpu_lbl."""
    visible = sum(max(0, min(Sk, i + 1 + Sk - Sq)) if causal else Sk for i in range(Sq)) * 2 * Hq
    assert B * visible > 160 << 20 and B * Hq * -(-Sq // 128) >= 192 and visible // Hkv < 100 << 20
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    q, k, v = (torch.randn(s, dtype=torch.bfloat16, device="cuda", generator=g)
               for s in ((B, Hq, Sq, dqk), (B, Hkv, Sk, dqk), (B, Hkv, Sk, dv)))
    whole = fa.forward_unfused(q, k, v, causal=causal, return_lse=True)
    rows = Sq * (Hq // Hkv)
    ws = torch.empty(rows * fa.fa_lbl_ld(Sk) * 2, dtype=torch.uint8, device="cuda")
    parts = fa.forward_unfused(q, k, v, causal=causal, return_lse=True, workspace=ws)
    for a, b in zip(whole, parts):
        assert torch.equal(_bits(a), _bits(b))


@pytest.mark.parametrize("causal", [False, True], ids=["full", "causal"])
@pytest.mark.parametrize("sk", [1, 8, 505, 512, 513, 1024, 1025, 2047, 2049, 4096, 4097, 8192, 8193])
def test_softmax_row_lengths(sk, causal):
    """Both sides of every row length at which the softmax kernel changes its instance; the causal rows
    end inside the last 64-chunk steps. Checks and tolerances of the operator's own test."""
    w = W.small(f"row length {sk}", Hq=1, Hkv=1, Sq=5, Sk=sk, causal=causal, seed=900 + sk)
    lbl.test_softmax_operator(w, True)


def _decode(q, k, v, causal, parts):
    B, Hq, Sq, dqk = q.shape
    _, Hkv, Sk, dv = v.shape
    o = torch.full((B, Hq, Sq, dv), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((B, Hq, Sq), float("nan"), dtype=torch.float32, device="cuda")
    fa.forward(q, k, v, causal=causal, return_lse=True, out=o, lse=lse, n_split=parts, decode=True)
    return o, lse


@pytest.mark.parametrize("w", [
    W.small("one part gqa4 d128", dqk=128, dv=128, B=2, Hq=8, Hkv=2, Sq=3, Sk=300, causal=True, seed=91),
    W.small("one part d64 two column blocks", Hq=20, Hkv=2, Sq=4, Sk=129, causal=False, seed=92),
    W.small("one part d192", dqk=192, dv=128, Hq=3, Hkv=3, Sq=1, Sk=1000, causal=True, seed=93),
    W.small("one part rows without keys", dqk=128, dv=128, Hq=2, Hkv=1, Sq=9, Sk=4, causal=True, seed=94),
], ids=lambda w: w.name)
def test_single_part_decode(w):
    """Against the fp64 oracle, and the same bits as two parts of which the second is empty where the keys
    fit one tile (the merge of one part with an empty one returns that part)."""
    q, k, v = (x.cuda() for x in W.make_inputs(w))
    o, lse = _decode(q, k, v, w.causal, 1)
    o64, lse64 = naive_attention(to_f64(q), to_f64(k), to_f64(v), w.scale, w.causal)
    compare(to_f64(o), lse.cpu().double().numpy(), o64, lse64, w.name)
    if w.Sk <= 128:
        o2, lse2 = _decode(q, k, v, w.causal, 2)
        assert torch.equal(_bits(o), _bits(o2)) and torch.equal(_bits(lse), _bits(lse2))


@pytest.mark.parametrize("d,dv", [(64, 64), (128, 128), (192, 128)])
def test_single_part_decode_rows_without_a_sum(d, dv):
    """Rows whose sum is not a number (a NaN in Q, scores that overflow) and rows without a visible key have
    LSE = -inf and O = 0, whether one part writes the result or the merge does (the second of two parts is
    empty: the keys fit one tile). A NaN in V stays in its column, and O and LSE of the other rows too are
    the same bits either way."""
    w = W.small(f"rows without a sum d{d}", dqk=d, dv=dv, Hq=6, Hkv=2, Sq=2, Sk=1, causal=True, seed=95)
    for sk in (1, 100):
        q, k, v = (x.cuda() for x in W.make_inputs(w.with_(Sk=sk)))
        q[0, 1, 1, 3] = float("nan")
        q[0, 4, 1], k[0, 1, 0] = 3e38, 1.0  # finite; their product overflows
        v[0, 0, 0, 5] = float("nan")
        one, two = _decode(q, k, v, True, 1), _decode(q, k, v, True, 2)
        for a, b in zip(one, two):
            assert torch.equal(a.isnan(), b.isnan())
            assert torch.equal(_bits(a)[~a.isnan()], _bits(b)[~b.isnan()])
        o, lse = one
        empty = torch.zeros(6, 2, dtype=torch.bool, device="cuda")
        empty[1, 1] = empty[4, 1] = True
        empty[:, 0] = sk == 1  # causal: row 0 of 2 sees no key of 1
        assert bool((lse[0][empty] == -float("inf")).all()) and bool((o[0][empty] == 0).all())
        assert bool(lse[0][~empty].isfinite().all())


@pytest.mark.parametrize("B,Hq,Hkv,Sq,Sk,dqk,dv,parts", [
    (9, 16, 8, 1, 3999, 128, 128, 2),
    (17, 8, 8, 2, 4100, 64, 64, 1),
    (5, 12, 12, 1, 3700, 192, 128, 3),
])
def test_streamed_decode_equals_cached(B, Hq, Hkv, Sq, Sk, dqk, dv, parts):
    """The whole batch (K and V above 128 MiB: streamed) against each request alone (below it), bit for
    bit: the arithmetic does not depend on the batch."""
    assert B * Hkv * Sk * (dqk + dv) * 2 > 128 << 20
    g = torch.Generator(device="cuda")
    g.manual_seed(6)
    q, k, v = (torch.randn(s, dtype=torch.bfloat16, device="cuda", generator=g)
               for s in ((B, Hq, Sq, dqk), (B, Hkv, Sk, dqk), (B, Hkv, Sk, dv)))
    o, lse = _decode(q, k, v, True, parts)
    for b in range(B):
        ob, lb = _decode(q[b:b + 1], k[b:b + 1], v[b:b + 1], True, parts)
        assert torch.equal(_bits(o[b:b + 1]), _bits(ob)) and torch.equal(_bits(lse[b:b + 1]), _bits(lb))
