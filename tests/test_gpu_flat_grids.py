"""GPU parity of chunk-of-a-prompt shapes (more than twice as many keys as query rows) on both sides of the
block counts at which they leave the instance their grid would otherwise run. Sampled heads against the
fp64 oracle."""

import numpy as np
import pytest
import torch

import paper_2609_21264_amd as fa
import workloads as W
from oracle import attention_head
from parity import compare, to_f64

pytestmark = pytest.mark.gpu

CASES = [W.small(f"d{d} {hq}/{hkv} {sq}x{sk} {'causal' if c else 'full'}", dqk=d, dv=d, Hq=hq, Hkv=hkv, Sq=sq, Sk=sk,
                 causal=c, seed=71 + hq + sk)
         for d, hq, hkv, sq, sk, c in (
             (128, 159, 53, 70, 141, True), (128, 160, 20, 70, 141, True), (128, 160, 160, 70, 140, True),
             (128, 128, 32, 300, 777, False), (128, 80, 80, 257, 515, True), (128, 256, 64, 33, 257, False),
             (64, 200, 50, 90, 300, True), (64, 201, 67, 90, 300, True), (64, 160, 20, 257, 1100, True),
             (64, 201, 201, 150, 300, True))]


@pytest.mark.parametrize("w", CASES, ids=[w.name for w in CASES])
def test_flat_grids_match_oracle(w):
    q, k, v = (x.cuda() for x in W.make_inputs(w))
    o, lse = fa.forward(q, k, v, causal=w.causal, scale=w.scale, return_lse=True)
    torch.cuda.synchronize()
    group = w.Hq // w.Hkv
    heads = sorted({0, 1, w.Hq // 2, w.Hq - 1})
    ref = [attention_head(to_f64(q[0, h]), to_f64(k[0, h // group]), to_f64(v[0, h // group]), w.scale, w.causal)
           for h in heads]
    compare(to_f64(o[0, heads]), lse[0, heads].cpu().double().numpy(), np.stack([r[0] for r in ref]),
            np.stack([r[1] for r in ref]), w.name)
