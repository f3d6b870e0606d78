"""GPU parity of chunk-of-a-prompt shapes (more than twice as many keys as query rows) on both sides of the
lines at which they leave the instance their grid would otherwise run, each with the instance it runs.
Sampled heads against the fp64 oracle."""

import numpy as np
import pytest
import torch

import paper_2609_21264_amd as fa
import workloads as W
from oracle import attention_head
from parity import compare, to_f64

pytestmark = pytest.mark.gpu

QUARTERS, HALVES, SHORT, SHORT_WIDE, LONG = (fa.FA_INSTANCE_QUARTERS, fa.FA_INSTANCE_HALVES, fa.FA_INSTANCE_SHORT,
                                            fa.FA_INSTANCE_SHORT_WIDE, fa.FA_INSTANCE_LONG)

CASES = [(W.small(f"d{d} {hq}/{hkv} {sq}x{sk} {'causal' if c else 'full'}", dqk=d, dv=d, Hq=hq, Hkv=hkv, Sq=sq, Sk=sk,
                  causal=c, seed=71 + hq + sk), inst)
         for d, hq, hkv, sq, sk, c, inst in (
             (128, 159, 53, 70, 141, True, HALVES), (128, 160, 20, 70, 141, True, HALVES),
             (128, 160, 160, 70, 140, True, HALVES), (128, 128, 32, 300, 777, False, LONG),
             (128, 80, 80, 257, 515, True, HALVES), (128, 256, 64, 33, 257, False, SHORT),
             # both sides of six times as many keys, of the long instance's padding and of a full short grid
             (128, 160, 160, 200, 1200, True, LONG), (128, 160, 160, 200, 1199, True, SHORT),
             (128, 80, 80, 300, 601, False, SHORT), (128, 80, 80, 400, 801, False, LONG),
             (128, 96, 24, 280, 1700, True, HALVES), (128, 160, 160, 128, 770, True, HALVES),
             (64, 200, 50, 90, 300, True, HALVES), (64, 201, 67, 90, 300, True, SHORT),
             (64, 160, 20, 257, 1100, True, HALVES), (64, 201, 201, 150, 300, True, HALVES),
             (64, 201, 201, 200, 401, True, SHORT), (64, 256, 16, 20, 900, True, QUARTERS),
             (64, 256, 64, 40, 300, True, HALVES), (64, 240, 60, 100, 300, True, SHORT),
             (64, 240, 80, 150, 310, True, HALVES), (64, 72, 24, 700, 1500, True, SHORT_WIDE))]


@pytest.mark.parametrize("w,instance", CASES, ids=[w.name for w, _ in CASES])
def test_flat_grids_match_oracle(w, instance):
    assert fa.fa_fwd_instance(w.B, w.Hq, w.Hkv, w.Sq, w.Sk, w.dqk, w.dv, w.causal) == instance
    q, k, v = (x.cuda() for x in W.make_inputs(w))
    o, lse = fa.forward(q, k, v, causal=w.causal, scale=w.scale, return_lse=True)
    torch.cuda.synchronize()
    group = w.Hq // w.Hkv
    heads = sorted({0, 1, w.Hq // 2, w.Hq - 1})
    ref = [attention_head(to_f64(q[0, h]), to_f64(k[0, h // group]), to_f64(v[0, h // group]), w.scale, w.causal)
           for h in heads]
    compare(to_f64(o[0, heads]), lse[0, heads].cpu().double().numpy(), np.stack([r[0] for r in ref]),
            np.stack([r[1] for r in ref]), w.name)
