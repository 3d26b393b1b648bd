"""The backward with less workspace than the size query gives: without parts of the heads, and, where workgroups of four waves would
rather have finer slices, with the slices of workgroups of eight, which need the least.  The same gradients come out up to the order of fp32 sums."""
import re

import pytest
import torch

import paper_2506_11498_amd as lrsa
from paper_2506_11498_amd import inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# the last two need less with the slices of eight waves than with their own
@pytest.mark.parametrize("cfg,fewer_slices", [(dict(B=2, Hq=4, Hkv=4, n=1861, L=33, K=16, S=4), False), (dict(B=1, Hq=4, Hkv=2, n=3745, L=59, K=29, S=0), False),
                                              (dict(B=1, Hq=8, Hkv=1, n=2385, L=143, K=27, S=16), True), (dict(B=1, Hq=6, Hkv=1, n=3379, L=196, K=92, S=16), True)])
def test_least_workspace(cfg, fewer_slices):
    w = inputs.small_workload(d=64, dtype="bf16", **cfg)
    x = {k: v.to(DEV) for k, v in inputs.make_inputs(w).items()}
    p = lrsa.params_for(x["Q"], x["K"], sink=w.S, lag=w.L, topk=w.K)
    _, idx = lrsa.lrsa_score_select(p, x["K"], x["V"])
    O, lse = lrsa.lrsa_attn_fwd(p, x["Q"], x["K"], x["V"], idx)
    args = (p, x["Q"], x["K"], x["V"], O, x["dO"], lse, idx)
    with pytest.raises(lrsa.LrsaError) as e:
        lrsa.lrsa_attn_bwd(*args, ws=torch.empty(256, dtype=torch.uint8, device=DEV))
    least, most = int(re.search(r"(\d+) are needed", str(e.value))[1]), lrsa.workspace_bytes(p, 3)
    assert least < most
    small, whole = lrsa.attn_plan(p, bwd_ws_bytes=least), lrsa.attn_plan(p, bwd_ws_bytes=most - 1)
    assert (small.gather_parts, small.window_parts) == (1, 1) and (small.slices < whole.slices) == fewer_slices
    want = lrsa.lrsa_attn_bwd(*args)
    got = [torch.full_like(t, float("nan")) for t in want]
    lrsa.lrsa_attn_bwd(*args, *got, ws=torch.empty(least, dtype=torch.uint8, device=DEV))
    for a, b in zip((t.double() for t in want), (t.double() for t in got)):
        # fp32 sums in another order differ by some 2^-22 of the terms' size: few elements land on the other side of a rounding to bf16, those
        # one step (2^-7 of the element) apart; elements whose terms cancel may differ by more of themselves, by 2^-18 of the largest
        assert ((a - b).abs() <= 2.0 ** -7 * a.abs() + 2.0 ** -18 * a.abs().max()).all()
        assert (a != b).double().mean() <= 0.005
