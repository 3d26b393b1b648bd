"""Which wave takes which query rows in the forward and dQ kernels (bf16): pieces of 32 rows of one head, neighbouring ones in a
workgroup of four or eight waves, at the edges of chunks, heads and launches, against the fp64 oracle.

With impl = COMPACT the workgroups always have eight waves, without it small launches have four.  A wave's own work does not depend
on its neighbours, so both must give the same bits.  Buffers are filled with NaN first: a row that nobody takes shows.
"""
import numpy as np
import pytest
import torch

import paper_2506_11498_amd as lrsa
from paper_2506_11498_amd import inputs
from oracle import lrsa_ref as ref

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

SHAPES = [
    dict(n=3 + 5 * 33 + 1, L=33, S=3, K=8, Hq=8, Hkv=1),            # two blocks of four heads, eight pieces each
    dict(n=40 + 6 * 32 + 7, L=32, S=40, K=8, Hq=12, Hkv=1),         # blocks of four pieces: a workgroup holds two
    dict(n=5 + 4 * 100 + 33, L=100, S=5, K=25, Hq=20, Hkv=1),       # blocks of sixteen, five of them
    dict(n=33 + 3 * 258 + 2, L=258, S=33, K=64, Hq=6, Hkv=2),       # chunks two rows past a multiple of 32, heads in threes
    dict(n=6 * 65 + 64, L=65, S=0, K=16, Hq=5, Hkv=1, B=2),         # no sink
    dict(n=7 + 3 * 40 + 1, L=40, S=7, K=10, Hq=7, Hkv=1, B=3),      # a tail of one row
    dict(n=16 + 9 * 96 + 50, L=96, S=16, K=24, Hq=24, Hkv=8, B=1),  # 256 and more workgroups of four waves, resident at once
    dict(n=4 + 7 * 64, L=64, S=4, K=16, Hq=64, Hkv=8, B=3),         # more than are resident, short walks: four waves, in turn
]


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("cfg", SHAPES, ids=[f"n{c['n']}_L{c['L']}_G{c['Hq'] // c['Hkv']}" for c in SHAPES])
def test_every_row_once(cfg, d):
    w = inputs.small_workload(d=d, dtype="bf16", **cfg)
    x = inputs.make_inputs(w)
    xf = {k: v.float().numpy() for k, v in x.items()}
    idx = ref.select(ref.score(xf["K"], xf["V"], w.S, w.L), w.S, w.L, w.K)
    O, lse = ref.attn_fwd_dense(xf["Q"], xf["K"], xf["V"], idx, w.S, w.L)
    dQ, dK, dV = ref.attn_bwd_dense(xf["Q"], xf["K"], xf["V"], xf["dO"], idx, w.S, w.L)
    want = dict(O=O, lse=lse, dQ=dQ, dK=dK, dV=dV)
    xd = {k: v.to(DEV) for k, v in x.items()}
    idx = torch.from_numpy(idx).to(DEV)
    got = {}
    for impl in [lrsa.IMPL_AUTO] + [lrsa.IMPL_COMPACT] * (d == 128):
        p = lrsa.params_for(xd["Q"], xd["K"], sink=w.S, lag=w.L, topk=w.K, impl=impl)
        o = dict(O=torch.full_like(xd["Q"], float("nan")), lse=torch.full(xd["Q"].shape[:3], float("nan"), device=DEV),
                 dQ=torch.full_like(xd["Q"], float("nan")), dK=torch.full_like(xd["K"], float("nan")), dV=torch.full_like(xd["K"], float("nan")))
        ws = torch.empty(max(lrsa.workspace_bytes(p, k) for k in (2, 3)), dtype=torch.uint8, device=DEV)
        lrsa.lrsa_attn_fwd(p, xd["Q"], xd["K"], xd["V"], idx, o["O"], o["lse"], ws)
        lrsa.lrsa_attn_bwd(p, xd["Q"], xd["K"], xd["V"], o["O"], xd["dO"], o["lse"], idx, o["dQ"], o["dK"], o["dV"], ws)
        torch.cuda.synchronize()
        for k, r in want.items():   # bf16 results and operands: the bar of the attention tests
            e = np.abs(o[k].double().cpu().numpy() - r).max() / np.abs(r).max()
            assert e < 2e-2, f"{k}: {e:.3e}"
        got[impl] = o
    if d == 128:
        for k in ("O", "lse", "dQ"):
            assert torch.equal(got[lrsa.IMPL_AUTO][k], got[lrsa.IMPL_COMPACT][k]), k


@pytest.mark.parametrize("d,B,Hq,Hkv", [(64, 1, 16, 4), (64, 3, 32, 8), (128, 1, 16, 4), (128, 3, 32, 8)])   # 8, 4, 8 and 4 waves per workgroup
def test_fp32_with_fewer_waves(d, B, Hq, Hkv):
    """Many query tiles: fewer waves share a tile's keys.  The bar of the fp32 kernels: a quarter above the plain kernels' error, plus an ulp."""
    w = inputs.small_workload(d=d, dtype="f32", n=5 + 5 * 50 + 33, L=50, S=5, K=17, Hq=Hq, Hkv=Hkv, B=B)
    x = inputs.make_inputs(w)
    xf = {k: v.numpy() for k, v in x.items()}
    idx = ref.select(ref.score(xf["K"], xf["V"], w.S, w.L), w.S, w.L, w.K)
    O, lse = ref.attn_fwd_dense(xf["Q"], xf["K"], xf["V"], idx, w.S, w.L)
    g = ref.attn_bwd_dense(xf["Q"], xf["K"], xf["V"], xf["dO"], idx, w.S, w.L)
    want = dict(O=O, lse=lse, dQ=g[0], dK=g[1], dV=g[2])
    xd = {k: v.to(DEV) for k, v in x.items()}
    idx = torch.from_numpy(idx).to(DEV)
    errs = []
    for impl in (lrsa.IMPL_AUTO, lrsa.IMPL_GENERIC):
        p = lrsa.params_for(xd["Q"], xd["K"], sink=w.S, lag=w.L, topk=w.K, impl=impl)
        O, lse = lrsa.lrsa_attn_fwd(p, xd["Q"], xd["K"], xd["V"], idx)
        dQ, dK, dV = lrsa.lrsa_attn_bwd(p, xd["Q"], xd["K"], xd["V"], O, xd["dO"], lse, idx)
        got = dict(O=O, lse=lse, dQ=dQ, dK=dK, dV=dV)
        errs.append({k: np.linalg.norm(got[k].double().cpu().numpy() - r) / np.linalg.norm(r) for k, r in want.items()})
    for k in want:
        assert errs[0][k] <= 1.25 * errs[1][k] + 2.0 ** -23, f"{k}: {errs[0][k]:.3e}, the plain kernels {errs[1][k]:.3e}"
