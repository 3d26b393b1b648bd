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
        assert lrsa.attn_plan(p).fwd_waves == lrsa.attn_plan(p).dq_waves == (8 if impl == lrsa.IMPL_COMPACT else 4)
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
        assert impl == lrsa.IMPL_GENERIC or lrsa.attn_plan(p).fwd_waves == (4 if Hq == 32 else 8)
        O, lse = lrsa.lrsa_attn_fwd(p, xd["Q"], xd["K"], xd["V"], idx)
        dQ, dK, dV = lrsa.lrsa_attn_bwd(p, xd["Q"], xd["K"], xd["V"], O, xd["dO"], lse, idx)
        got = dict(O=O, lse=lse, dQ=dQ, dK=dK, dV=dV)
        errs.append({k: np.linalg.norm(got[k].double().cpu().numpy() - r) / np.linalg.norm(r) for k, r in want.items()})
    for k in want:
        assert errs[0][k] <= 1.25 * errs[1][k] + 2.0 ** -23, f"{k}: {errs[0][k]:.3e}, the plain kernels {errs[1][k]:.3e}"


def long_walk(d, n, Hq):
    """fp32 attention of n tokens in two chunks, so that the last rows see all of them: the results and, for the last 256 rows, 64 bits."""
    w = inputs.small_workload(d=d, dtype="f32", n=n, L=n // 2, S=0, K=1, Hq=Hq, Hkv=1)
    x = {k: v.to(DEV) for k, v in inputs.make_inputs(w).items()}

    def run(heads):
        Q, dO = (x[k][:, :heads].contiguous() for k in ("Q", "dO"))
        p = lrsa.params_for(Q, x["K"], sink=0, lag=w.L, topk=1)
        O, lse = lrsa.lrsa_attn_fwd(p, Q, x["K"], x["V"], None)
        return dict(O=O, lse=lse, dQ=lrsa.lrsa_attn_bwd(p, Q, x["K"], x["V"], O, dO, lse, None)[0])

    q, do, k, v = (x[z][0, 0].double() for z in ("Q", "dO", "K", "V"))
    q, do = q[-256:], do[-256:]
    s = (q @ k.T * d ** -0.5).masked_fill(torch.arange(n, device=DEV) > torch.arange(n - 256, n, device=DEV)[:, None], float("-inf"))
    P = torch.softmax(s, -1)
    O = P @ v
    return run, dict(O=O, lse=torch.logsumexp(s, -1), dQ=P * (do @ v.T - (do * O).sum(-1, keepdim=True)) @ k * d ** -0.5)


@pytest.mark.parametrize("d", [64, 128])
def test_fp32_long_walks_do_not_depend_on_the_number_of_heads(d):
    """4096 visible keys: four heads have tiles enough for fewer waves per tile, a single one has not.  Fewer waves would add longer chains,
    whose error is larger (four instead of all, O: 1.08 times at head_dim 64, 1.05 at 128)."""
    run, _ = long_walk(d, 4096, 4)
    four, one = run(4), run(1)
    for k in four:
        assert torch.equal(four[k][:, :1], one[k]), k


@pytest.mark.parametrize("d,bar", [(64, 3.07e-7), (128, 3.54e-7)])
def test_fp32_error_of_long_walks(d, bar):
    """12288 visible keys.  O, 2-norm: all waves 2.7e-7 (head_dim 64) and 3.3e-7 (128), four waves 3.4e-7 and 3.8e-7; the bar lies between.
    lse: one rounding of a value near 10 is 2^-24 of it, the sums add some; dQ: with D a difference of sums, twice the bar of O and more."""
    run, want = long_walk(d, 12288, 1)
    got = run(1)
    e = {k: float((got[k][0, 0, -256:].double() - r).norm() / r.norm()) for k, r in want.items()}
    assert e["O"] <= bar and e["lse"] <= 2.0 ** -23 and e["dQ"] <= 3 * bar, e


@pytest.mark.parametrize("d,n,heads", [(64, 1024, 16), (64, 2048, 5), (128, 512, 20)])   # 4, 8 and 4 waves per tile; a single head has all
def test_fp32_error_of_the_longest_walks_with_fewer_waves(d, n, heads):
    """As long as walks with fewer waves get.  Measured 0.97, 0.99 and 0.99 of the error of O with all waves, 0.98 to 1.0 of dQ's; a tenth is the
    spread of dQ from one set of rows to the next."""
    run, want = long_walk(d, n, heads)
    few, all_waves = run(heads), run(1)
    assert not torch.equal(few["O"][:, :1], all_waves["O"])
    for k, r in want.items():
        e, e_all = (float((x[k][0, 0, -256:].double() - r).norm() / r.norm()) for x in (few, all_waves))
        assert e <= (1.1 if k == "dQ" else 1.03) * e_all, f"{k}: {e:.3e}, with all waves {e_all:.3e}"


def dense64(x, idx, S, L, lp, dev=DEV):
    """O, lse, dQ, dK, dV of every row in 64 bits from the mask of the definitions (ref.visible_mask), on the GPU in plain torch."""
    out = {k: [] for k in ("O", "lse", "dQ", "dK", "dV")}
    B, Hkv, n, d = x["K"].shape
    G = x["Q"].shape[1] // Hkv
    for b in range(B):
        for h in range(Hkv):
            vis = torch.from_numpy(ref.visible_mask(n, S, L, idx[b, h].cpu().numpy(), lp)).to(dev)
            k, v = x["K"][b, h].double(), x["V"][b, h].double()
            dk = dv = 0
            for hq in range(h * G, h * G + G):
                q, do = x["Q"][b, hq].double(), x["dO"][b, hq].double()
                s = (q @ k.T * d ** -0.5).masked_fill(~vis, float("-inf"))
                P = torch.softmax(s, -1)
                O = P @ v
                dS = P * (do @ v.T - (do * O).sum(-1, keepdim=True)) * d ** -0.5
                dk, dv = dk + dS.T @ q, dv + P.T @ do
                for name, t in (("O", O), ("lse", torch.logsumexp(s, -1)), ("dQ", dS @ k)):
                    out[name].append(t)
            out["dK"].append(dk)
            out["dV"].append(dv)
    return {k: torch.stack(v).view(B, -1, *v[0].shape) for k, v in out.items()}


@pytest.mark.parametrize("cfg,lp", [(dict(B=8, Hq=32, Hkv=8, n=5 + 11 * 97 + 13, L=97, S=5, K=24), 1), (dict(B=8, Hq=24, Hkv=4, n=33 + 8 * 130 + 57, L=130, S=33, K=33), 1),
                                    (dict(B=4, Hq=64, Hkv=8, n=7 * 157 - 3, L=157, S=0, K=50), 2)], ids=["G4", "G6", "G8"])
def test_head_dim_64_forward_with_eight_waves_equals_four(cfg, lp):
    """All requests together fill the chip and take eight waves per workgroup, each alone four, which the oracle tests check: the same bits in every
    row, those of keys that hold infinities and NaN among them."""
    w = inputs.small_workload(d=64, dtype="bf16", **cfg)
    x = {k: v.to(DEV) for k, v in inputs.make_inputs(w).items()}
    x["K"][0, 0, w.n - 40], x["V"][0, 0, w.S + 3, 5] = float("nan"), float("inf")
    Ns = lrsa.num_scored_chunks(lrsa.params_for(x["Q"], x["K"], sink=w.S, lag=w.L, topk=w.K, local_prev=lp))
    g = torch.Generator().manual_seed(5)
    idx = torch.rand((w.B, w.Hkv, Ns, w.L), generator=g).argsort(-1)[..., :w.K].sort(-1).values
    idx = (idx + w.S + w.L * torch.arange(Ns)[:, None]).to(torch.int32).to(DEV)

    def run(b):
        Q, K, V, i = (t[b].contiguous() for t in (x["Q"], x["K"], x["V"], idx))
        p = lrsa.params_for(Q, K, sink=w.S, lag=w.L, topk=w.K, local_prev=lp)
        O, lse = torch.full_like(Q, 7.0), torch.full(Q.shape[:3], 7.0, device=DEV)
        lrsa.lrsa_attn_fwd(p, Q, K, V, i, O, lse)
        return lrsa.attn_plan(p).fwd_waves, O.view(torch.int16), lse.view(torch.int32)

    waves, O, lse = run(slice(0, w.B))
    assert waves == 8
    for b in range(w.B):
        waves, o, l = run(slice(b, b + 1))
        assert waves == 4 and torch.equal(o, O[b:b + 1]) and torch.equal(l, lse[b:b + 1]), f"request {b}"


# lags that are no multiple of 32, so that rows and keys at chunk ends inside the sequence leave pieces, steps and waves of keys partly filled
EIGHT = [
    (dict(B=2, Hq=16, Hkv=8, n=2161, L=499, K=235, S=33), 1, (1, 1)),   # G, local_prev, parts of the heads (listed keys, window)
    (dict(B=2, Hq=15, Hkv=3, n=2236, L=422, K=195, S=33), 1, (1, 3)),
    (dict(B=1, Hq=24, Hkv=3, n=2955, L=225, K=111, S=0), 1, (1, 2)),    # two blocks of four heads
    (dict(B=4, Hq=6, Hkv=1, n=2782, L=689, K=296, S=5), 2, (3, 3)),
    (dict(B=4, Hq=8, Hkv=2, n=2669, L=521, K=226, S=16), 2, (1, 2)),
]


@pytest.mark.parametrize("cfg,lp,parts", EIGHT, ids=[f"n{c['n']}_L{c['L']}_G{c['Hq'] // c['Hkv']}" for c, _, _ in EIGHT])
def test_eight_waves_at_odd_lags(cfg, lp, parts):
    """The variants with eight waves of all three kernels that gather by position, in every row.  An element carries its own bf16 rounding
    (2^-9) and that of P and dS, 2^-9 of terms that add up like random ones: a row is off by about 2^-9 to 2^-8 of its norm.  dQ and dK also
    take D = sum(dO * O) from the rounded O: dS of a row whose dA - D nearly cancel is off by more."""
    w = inputs.small_workload(d=128, dtype="bf16", **cfg)
    x = {k: v.to(DEV) for k, v in inputs.make_inputs(w).items()}
    p = lrsa.params_for(x["Q"], x["K"], sink=w.S, lag=w.L, topk=w.K, local_prev=lp)
    plan = lrsa.attn_plan(p)
    assert (plan.fwd_waves, plan.dq_waves, plan.key_waves, (plan.gather_parts, plan.window_parts)) == (8, 8, 8, parts)
    _, idx = lrsa.lrsa_score_select(p, x["K"], x["V"])
    got = dict(O=torch.full_like(x["Q"], float("nan")), lse=torch.full(x["Q"].shape[:3], float("nan"), device=DEV),
               dQ=torch.full_like(x["Q"], float("nan")), dK=torch.full_like(x["K"], float("nan")), dV=torch.full_like(x["K"], float("nan")))
    lrsa.lrsa_attn_fwd(p, x["Q"], x["K"], x["V"], idx, got["O"], got["lse"])
    lrsa.lrsa_attn_bwd(p, x["Q"], x["K"], x["V"], got["O"], x["dO"], got["lse"], idx, got["dQ"], got["dK"], got["dV"])
    for k, r in dense64(x, idx, w.S, w.L, lp).items():
        g = got[k].double()
        assert g.isfinite().all(), k
        if k == "lse":
            assert (g - r).abs().max() <= 1e-5          # sixteen ulps of values near 8
            continue
        bar = 2.0 ** -7
        if k == "dQ":
            late = slice(w.S + 2 * w.L, None)
            e = ((g - r).norm(dim=-1) / r.norm(dim=-1))[:, :, late].max()
            assert e <= bar, f"dQ behind the first two chunks: {float(e):.3e}"
            r_norm, bar = r.norm(dim=-1) + r.norm(dim=-1).mean(), 2.0 ** -4   # the first rows see few keys: P near one, dA near D
        else:
            r_norm = r.norm(dim=-1)
        e = ((g - r).norm(dim=-1) / r_norm).max()
        assert e <= bar, f"{k}: {float(e):.3e}"
