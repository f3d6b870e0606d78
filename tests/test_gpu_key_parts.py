"""GPU parity of the key-parts instances at the edges of their tiles: key quarters (128-key tiles, each
wave of a 32-row workgroup takes one 32-key quarter) on grids of at most one workgroup per CU, key halves
above, both sides of the switches between them, and the 32-key tiles of the long instance at d = 64.
Every output element against the fp64 oracle at the parity bar (the derived one for sigma > 1)."""

import numpy as np
import pytest

import paper_2609_21264_amd as fa
import workloads as W
from oracle import naive_attention
from parity import compare, rounding_bar, run_gpu, to_f64

pytestmark = pytest.mark.gpu


def _w(name, d, Hq, Hkv, Sq, Sk, causal, **kw):
    return W.small(f"{name} d{d} {Hq}/{Hkv} {Sq}x{Sk} {'causal' if causal else 'full'}", dqk=d, dv=d, Hq=Hq, Hkv=Hkv,
                   Sq=Sq, Sk=Sk, causal=causal, seed=611 + Sq + Sk, **kw)


CASES = [
    # one tile and a key, quarters without a key, whole tiles, one key past them
    *[_w("quarters", 64, 3, 1, sq, sk, c) for sq, sk in ((1, 65), (31, 96), (33, 127), (64, 128), (100, 129), (65, 257))
      for c in (False, True)],
    *[_w("quarters", 128, 2, 2, sq, sk, c) for sq, sk in ((1, 257), (32, 384), (97, 385), (300, 511)) for c in (False, True)],
    _w("rows without keys", 64, 4, 2, 300, 130, True),
    _w("rows without keys", 128, 4, 1, 700, 290, True),
    _w("many tiles", 128, 2, 1, 40, 2900, True, B=2),
    _w("scale 0", 64, 2, 2, 70, 300, False, scale=0.0),
    _w("negative scale", 128, 7, 1, 70, 700, True, scale=-0.07),
    _w("sigma 2", 64, 5, 5, 130, 640, True, sigma=2.0),
    # halves without a mask
    _w("halves", 64, 60, 15, 250, 257, False),
    _w("halves scale 0", 64, 60, 60, 200, 130, False, scale=0.0),
    _w("halves sigma 2", 64, 62, 31, 224, 321, False, sigma=2.0),
    # the last grid of quarters and the first of halves
    *[_w("switch", 64, h, h, 256, 300, False) for h in (32, 33)],
    *[_w("switch", 64, h, h, 200, 200, True) for h in (73, 74)],
    *[_w("switch", 128, h, h, 64, 400, True) for h in (128, 129)],
    *[_w("switch", 128, h, h, 1100, 2100, True) for h in (14, 15)],
    # the long instance's 32-key tiles at d = 64 (more than 1024 blocks)
    *[_w("long", 64, 1026, hkv, sq, sk, c) for hkv, sq, sk in ((1026, 1, 1), (342, 40, 31), (513, 65, 33), (1026, 33, 160))
      for c in (False, True)],
    _w("long rows without keys", 64, 1028, 257, 100, 63, True),
    _w("long sigma 2", 64, 1026, 114, 70, 200, True, sigma=2.0),
]


def _instance(w):
    return fa.fa_fwd_instance(w.B, w.Hq, w.Hkv, w.Sq, w.Sk, w.dqk, w.dv, w.causal)


def expected_instance(w):
    if w.name.startswith("long"):
        return fa.FA_INSTANCE_LONG
    halves = w.name.startswith("halves") or (w.name.startswith("switch") and w.Hq in (33, 74, 129, 15))
    return fa.FA_INSTANCE_HALVES if halves else fa.FA_INSTANCE_QUARTERS


@pytest.mark.parametrize("spiked", [False, True], ids=["plain", "rising"])
@pytest.mark.parametrize("w", CASES, ids=[w.name for w in CASES])
def test_key_parts_match_oracle(w, spiked):
    """"rising": keys scaled x4 .. x16 a third, two thirds and all the way through, so that parts redo a
    tile from its exact maximum and the parts' references differ widely."""
    assert _instance(w) == expected_instance(w)
    q, k, v = W.make_inputs(w)
    if spiked:
        for key, factor in ((w.Sk // 3, 4.0), (2 * w.Sk // 3, 8.0), (w.Sk - 1, 16.0)):
            k[:, :, key] *= factor
    print(f"\n[case] {w}", flush=True)
    o, lse = run_gpu(q, k, v, w)
    vf = to_f64(v)
    o_ref, lse_ref = naive_attention(to_f64(q), to_f64(k), vf, w.scale, w.causal)
    # spiked or sigma = 2: the bar derived from the bf16 rounding of P and O
    compare(to_f64(o), lse.cpu().double().numpy(), o_ref, lse_ref, w.name, max(1.0, w.sigma),
            o_bar=rounding_bar(vf, w.Hq) if spiked or w.sigma > 1.0 else None)


# At least four chunks of key/value heads (long instance): the work order visits every (head, query
# block) once whatever the heads left after the whole chunks, the group size and the batch.
CHUNKED = [
    _w("chunks", 128, 37, 37, 8200, 40, False),
    _w("chunks gqa8", 128, 264, 33, 2100, 120, True),
    _w("chunks gqa7", 128, 231, 33, 2400, 300, True),
    _w("chunks", 64, 67, 67, 8200, 33, False),
    W.small("chunks 192/128", B=3, Hq=23, Hkv=23, Sq=8200, Sk=260, dqk=192, dv=128, causal=True, seed=633),
]


@pytest.mark.parametrize("w", CHUNKED, ids=[w.name for w in CHUNKED])
def test_head_chunks_match_oracle(w):
    assert _instance(w) == fa.FA_INSTANCE_LONG
    q, k, v = W.make_inputs(w)
    print(f"\n[case] {w}", flush=True)
    o, lse = run_gpu(q, k, v, w)
    o_ref, lse_ref = naive_attention(to_f64(q), to_f64(k), to_f64(v), w.scale, w.causal)
    compare(to_f64(o), lse.cpu().double().numpy(), o_ref, lse_ref, w.name)
