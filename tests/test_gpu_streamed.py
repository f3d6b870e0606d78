"""GPU tests of the instances chosen by the size of the data: the layer-by-layer operators load and store
non-temporally when their data is large, and the softmax kernel has an instance per row length."""

import pytest
import torch

import paper_2609_21264_amd as fa
import test_gpu_lbl as lbl
import workloads as W

pytestmark = pytest.mark.gpu


def _bits(t):
    return t.view(torch.int16 if t.dtype == torch.bfloat16 else torch.int32)


@pytest.mark.parametrize("B,Hq,Hkv,Sq,Sk,dqk,dv,causal", [
    (2, 14, 14, 2100, 2100, 64, 64, False),
    (1, 56, 8, 2050, 2050, 128, 128, True),
    (1, 24, 24, 1000, 4300, 192, 128, True),
])
def test_streamed_spill_equals_cached(B, Hq, Hkv, Sq, Sk, dqk, dv, causal):
    """The whole problem in one chunk (its visible scores exceed 160 MiB: streamed) against chunks of one
    group of heads (below it: cached). The operators do the same arithmetic in the same order, so the
    results are the same bits; the cached path is checked against the oracle in test_gpu_lbl."""
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
