"""GPU tests: an infinity or a NaN in a key reaches only the rows that see the key.

A causal row that does not see a key must not depend on its value, so with one key of K replaced by
infinities or NaNs the rows above the diagonal at that key keep their finite results (the tolerance is the
parity bar: the values may move the reference maximum of other rows' tiles). The key is placed in each of
the first tiles, whatever the tile width of the instance, and at a tile's edges."""

import pytest
import torch

import paper_2609_21264_amd as fa
import workloads as W

pytestmark = pytest.mark.gpu

QUARTERS, HALVES, SHORT, SHORT_WIDE, LONG = (fa.FA_INSTANCE_QUARTERS, fa.FA_INSTANCE_HALVES, fa.FA_INSTANCE_SHORT,
                                             fa.FA_INSTANCE_SHORT_WIDE, fa.FA_INSTANCE_LONG)

# (d_qk, d_v, Hq, Hkv, S, instance, parts of split mode)
CASES = [(64, 64, 2, 1, 330, QUARTERS, 0), (128, 128, 2, 2, 330, QUARTERS, 0), (64, 64, 80, 40, 330, HALVES, 0),
         (128, 128, 60, 15, 330, HALVES, 0), (64, 64, 330, 110, 200, SHORT, 0), (64, 64, 82, 82, 1030, SHORT_WIDE, 0),
         (128, 128, 200, 50, 250, SHORT, 0), (64, 64, 520, 130, 330, LONG, 0), (128, 128, 132, 33, 330, LONG, 0),
         (192, 128, 4, 4, 330, LONG, 0), (64, 64, 4, 2, 330, SHORT, 2), (128, 128, 4, 2, 330, SHORT, 2),
         (128, 128, 64, 64, 250, LONG, 4)]


@pytest.mark.parametrize("value", [float("nan"), float("inf"), -float("inf")], ids=["nan", "inf", "-inf"])
@pytest.mark.parametrize("dqk,dv,hq,hkv,s,instance,parts", CASES)
def test_rows_that_do_not_see_a_non_finite_key(dqk, dv, hq, hkv, s, instance, parts, value):
    assert fa.fa_fwd_instance(1, hq, hkv, s, s, dqk, dv, True, parts) == instance
    w = W.small("non-finite key", Hq=hq, Hkv=hkv, Sq=s, Sk=s, dqk=dqk, dv=dv, causal=True, seed=77)
    q, k, v = (x.cuda() for x in W.make_inputs(w))
    kw = dict(causal=True, scale=w.scale, return_lse=True, **({"n_split": parts} if parts else {}))
    o_ref, lse_ref = (x.float() for x in fa.forward(q, k, v, **kw))
    assert bool(o_ref.isfinite().all())
    for key in (33, 63, 70, 100, 127, 129, 160, 190, 240, 300):
        if key >= s:
            continue
        bad = k.clone()
        bad[0, 0, key] = value
        o, lse = (x.float() for x in fa.forward(q, bad, v, **kw))
        print(f"\n[case] {instance} key {key}", flush=True)
        assert bool(o[:, :, :key].isfinite().all()) and bool(lse[:, :, :key].isfinite().all())
        assert float((o - o_ref)[:, :, :key].abs().max()) <= 2e-2
        assert float((lse - lse_ref)[:, :, :key].abs().max()) <= 1e-3
        # heads of the other key/value head are the same everywhere
        if hkv > 1:
            assert torch.equal(o[:, hq // hkv:], o_ref[:, hq // hkv:])
