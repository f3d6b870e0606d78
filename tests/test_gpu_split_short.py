"""GPU parity of split mode at the edges of its instances: blocks of 128 row-heads where they pad the query
rows less than blocks of 256 or those leave compute units idle, blocks of 256 otherwise (and always at
d_qk = 192). Every output element against the fp64 oracle at the parity bar."""

import pytest
import torch

import paper_2609_21264_amd as fa
import workloads as W
from oracle import naive_attention
from parity import compare, to_f64

pytestmark = pytest.mark.gpu


SHORT, LONG = fa.FA_INSTANCE_SHORT, fa.FA_INSTANCE_LONG


def _w(d, Hq, Hkv, Sq, Sk, causal, parts, B=1, instance=SHORT):
    w = W.small(f"d{d} {B}x{Hq}/{Hkv} {Sq}x{Sk} {'causal' if causal else 'full'} parts {parts}", dqk=d,
                dv=min(d, 128), B=B, Hq=Hq, Hkv=Hkv, Sq=Sq, Sk=Sk, causal=causal, seed=17 + Sq + Sk)
    return pytest.param(w, parts, instance, id=w.name)


CASES = [
    # one head, two heads and four heads of a group per workgroup, at the edges of a wave's 32 rows and a
    # block's 128, 64 and 32 rows; parts without a key tile
    *[_w(d, hq, 2, sq, 300, c, 3) for d in (64, 128) for hq, sq in ((2, 1), (2, 128), (2, 129), (4, 65), (8, 31), (8, 33))
      for c in (False, True)],
    _w(64, 3, 1, 257, 700, True, 7),
    _w(128, 7, 1, 100, 64, False, 5),
    _w(128, 2, 1, 200, 130, True, 2, B=2),  # rows without keys
    # full grids (256 workgroups and more): the short instance by padding, the long one without it
    _w(64, 64, 16, 32, 520, True, 16),
    _w(64, 64, 16, 64, 520, True, 16, instance=LONG),
    _w(128, 64, 64, 100, 260, False, 4),
    _w(128, 64, 64, 250, 260, True, 4, instance=LONG),
    _w(192, 3, 3, 70, 300, True, 3, instance=LONG),
    # the long instance with two heads of a group per workgroup, with rows and whole parts without keys, and
    # with more parts than key tiles
    _w(64, 64, 32, 100, 700, True, 8, instance=LONG),
    _w(64, 32, 8, 50, 64, False, 40, instance=LONG),
    _w(128, 64, 64, 200, 130, True, 4, instance=LONG),
    _w(128, 28, 4, 130, 333, True, 10, instance=LONG),
]


@pytest.mark.parametrize("w,parts,instance", CASES)
def test_split_matches_oracle(w, parts, instance):
    assert fa.fa_fwd_instance(w.B, w.Hq, w.Hkv, w.Sq, w.Sk, w.dqk, w.dv, w.causal, parts) == instance
    q, k, v = (x.cuda() for x in W.make_inputs(w))
    o, lse = fa.forward(q, k, v, causal=w.causal, scale=w.scale, return_lse=True, n_split=parts)
    torch.cuda.synchronize()
    o64, lse64 = naive_attention(to_f64(q), to_f64(k), to_f64(v), w.scale, w.causal)
    compare(to_f64(o), lse.cpu().double().numpy(), o64, lse64, w.name)
