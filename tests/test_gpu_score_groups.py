"""Scoring with one workgroup per chunk, and by slices of 64 rows, where the lanes that hold a row (8, 16 or 32 of a wave, by head_dim and
data type) sum its channels among themselves while other rows of the wave are past the end of the chunk; and the cache step with the
same arithmetic.  Against the oracle, with the bars of test_gpu_parity.py; the score buffer is filled with NaN first.
"""
import numpy as np
import pytest
import torch

import paper_2506_11498_amd as lrsa
from paper_2506_11498_amd import inputs
from oracle import lrsa_ref as ref
from test_gpu_parity import check_selection_in_tie_window, to_np

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 128), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("L", [2, 7, 33, 63, 129, 1025])
def test_rows_that_end_inside_a_wave(L, dtype, d):
    w = inputs.small_workload(n=3 + 4 * L + L // 2, L=L, S=3, K=max(1, L // 3), Hq=3, Hkv=3, B=2, d=d, dtype=dtype)
    x = inputs.make_inputs(w)
    K, V = x["K"].to(DEV), x["V"].to(DEV)
    p = lrsa.params_for(x["Q"].to(DEV), K, sink=w.S, lag=w.L, topk=w.K)
    resident = dtype == "bf16" and d == 128 and L >= 64     # those are kept in registers by another kernel, with other sums
    if not resident:
        assert lrsa.score_route(p) == (2 if L >= 1024 else 1)
    score = torch.full((2, 3, lrsa.num_scored_chunks(p), L), float("nan"), device=DEV)
    score, idx = lrsa.lrsa_score_select(p, K, V, score)
    sc_ref = ref.score(x["K"].float().numpy(), x["V"].float().numpy(), w.S, w.L)
    assert np.allclose(to_np(score), sc_ref, rtol=2e-5, atol=1e-9)
    _, outside_rel = check_selection_in_tie_window(w, idx.cpu().numpy(), ref.select(sc_ref, w.S, w.L, w.K), sc_ref)
    assert outside_rel == 0
    assert torch.equal(lrsa.lrsa_score(p, K, V), score)
    if resident:
        return
    # the cache's single step scores its oldest chunk with the same sums: the rows that survive are the first chunk's
    n = w.S + 2 * L
    Kc, Vc = K[:, :, :n].contiguous(), V[:, :, :n].contiguous()
    pos = torch.arange(n, dtype=torch.int32, device=DEV).expand(2, 3, n).contiguous()
    lrsa.lrsa_cache_compress(lrsa.params_for(x["Q"][:, :, :n].contiguous().to(DEV), Kc, sink=w.S, lag=w.L, topk=w.K), Kc, Vc, pos, n, 0)
    assert torch.equal(pos[:, :, w.S:w.S + w.K], idx[:, :, 0].to(pos.dtype))
