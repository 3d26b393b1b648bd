"""The backward with the least workspace that it takes, where workgroups of four waves would rather have finer slices: it then takes the
slices of workgroups of eight (two shapes), and the same gradients come out up to the order of fp32 sums."""
import re

import pytest
import torch

import paper_2506_11498_amd as lrsa
from paper_2506_11498_amd import inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("cfg", [dict(B=2, Hq=4, Hkv=4, n=1861, L=33, K=16, S=4), dict(B=1, Hq=4, Hkv=2, n=3745, L=59, K=29, S=0)])
def test_least_workspace(cfg):
    w = inputs.small_workload(d=64, dtype="bf16", **cfg)
    x = {k: v.to(DEV) for k, v in inputs.make_inputs(w).items()}
    p = lrsa.params_for(x["Q"], x["K"], sink=w.S, lag=w.L, topk=w.K)
    _, idx = lrsa.lrsa_score_select(p, x["K"], x["V"])
    O, lse = lrsa.lrsa_attn_fwd(p, x["Q"], x["K"], x["V"], idx)
    args = (p, x["Q"], x["K"], x["V"], O, x["dO"], lse, idx)
    with pytest.raises(lrsa.LrsaError) as e:
        lrsa.lrsa_attn_bwd(*args, ws=torch.empty(256, dtype=torch.uint8, device=DEV))
    least = int(re.search(r"(\d+) are needed", str(e.value))[1])
    assert least < lrsa.workspace_bytes(p, 3)
    want = lrsa.lrsa_attn_bwd(*args)
    got = [torch.full_like(t, float("nan")) for t in want]
    lrsa.lrsa_attn_bwd(*args, *got, ws=torch.empty(least, dtype=torch.uint8, device=DEV))
    for a, b in zip(want, got):
        # sums that differ by fp32 roundings land at most one step of bf16 apart, 2^-7 of an element
        assert (a.double() - b.double()).norm() <= 2.0 ** -7 * a.double().norm()
