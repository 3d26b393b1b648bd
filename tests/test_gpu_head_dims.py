"""The tiled attention kernels of head_dim 64 (bf16) and of fp32 data at the edges of their tiles, against the fp64 oracle.

bf16, head_dim 64: these kernels hold the fp32 probabilities and dS as three bf16 terms, which is all 24 bits of them, as the
plain fp32-arithmetic kernels (IMPL_GENERIC) do.  The bar is the plain kernels' own error: at most 5 % above it (two independent
roundings of some thousand values differ by less) plus 2^-16 of the result's norm.  That error is the rounding of the bf16 results
(2^-9); test_bf16_head_dim_64_keeps_fp32_weights looks below it.

fp32: both kinds of kernel sum in fp32, in different orders; the tiled ones may be off by a quarter more than the plain
ones, plus one ulp (2^-23) of the result's norm where the plain error is that small.
"""
import numpy as np
import pytest
import torch

import paper_2506_11498_amd as lrsa
from paper_2506_11498_amd import inputs
from oracle import lrsa_ref as ref

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# tiles: 64 keys and four pieces of 32 rows of a head (heads of a group side by side) in the query-outer kernels, 128 keys and steps of 32
# query rows in the key-outer one
BF16_D64 = [
    dict(n=1, L=8, S=0, K=2, Hq=1, Hkv=1),                          # one row
    dict(n=40, L=32, S=64, K=8, Hq=2, Hkv=1),                       # sink only
    dict(n=5 + 7 * 100 + 33, L=100, S=5, K=37, Hq=6, Hkv=2, B=2),   # group of 3: pieces of three heads side by side
    dict(n=16 + 5 * 64 + 63, L=64, S=16, K=16, Hq=64, Hkv=8),       # group of 8, heads spread over the XCDs
    dict(n=33 + 4 * 257 + 1, L=257, S=33, K=64, Hq=2, Hkv=1),       # a chunk one row past a key tile, a tail of one row
    dict(n=7 + 6 * 130 + 129, L=130, S=7, K=130, Hq=4, Hkv=1),      # every token survives
    dict(n=4 + 9 * 64, L=64, S=4, K=1, Hq=3, Hkv=3, B=2),           # one survivor per chunk
    dict(n=16 + 4 * 127 + 31, L=127, S=16, K=37, Hq=1, Hkv=1),      # chunks and the list of chunk 4 (127 entries) one below a tile, a tail of 31 rows
    dict(n=16 + 4 * 128 + 32, L=128, S=16, K=56, Hq=2, Hkv=2),      # chunks, the list of chunk 3 and a tail of 32 rows that just fill theirs
    dict(n=33 + 4 * 129 + 33, L=129, S=33, K=48, Hq=1, Hkv=1, B=2),   # chunks, the list of chunk 3 (129), sink and tail one past theirs
]


def run(w, xd, idx, impl, **kw):
    p = lrsa.params_for(xd["Q"], xd["K"], sink=w.S, lag=w.L, topk=w.K, impl=impl, **kw)
    lrsa.timing_enable(True)
    O, lse = lrsa.lrsa_attn_fwd(p, xd["Q"], xd["K"], xd["V"], idx)
    dQ, dK, dV = lrsa.lrsa_attn_bwd(p, xd["Q"], xd["K"], xd["V"], O, xd["dO"], lse, idx)
    torch.cuda.synchronize()
    names = {n for n, _ in lrsa.timing_records()}
    lrsa.timing_enable(False)
    return dict(O=O, lse=lse, dQ=dQ, dK=dK, dV=dV), names


def reference(w, x, local_prev):
    xf = {k: v.float().numpy() for k, v in x.items()}
    idx = None
    if ref.partition(w.n, w.S, w.L, local_prev)["Ns"]:
        idx = ref.select(ref.score(xf["K"], xf["V"], w.S, w.L, local_prev=local_prev), w.S, w.L, w.K)
    O, lse = ref.attn_fwd_dense(xf["Q"], xf["K"], xf["V"], idx, w.S, w.L, local_prev=local_prev)
    g = ref.attn_bwd_dense(xf["Q"], xf["K"], xf["V"], xf["dO"], idx, w.S, w.L, local_prev=local_prev)
    return idx, dict(O=O, lse=lse, dQ=g[0], dK=g[1], dV=g[2])


def err(x, r):
    x = x.detach().double().cpu().numpy()
    if np.abs(r).max() < 1e-12:
        # one key: dA = D, so dQ and dK vanish but for the rounding of two sums of d products of O(1) inputs, which is
        # at most d * 2^-23 of them: counted in that unit
        return np.abs(x).max() / (x.shape[-1] * 2.0 ** -23) * 2.0 ** -23
    return np.linalg.norm(x - r) / np.linalg.norm(r)


def rows_strided(t):
    """The same values as [B, n, H, d] memory seen as [B, H, n, d]."""
    return t.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)


@pytest.mark.parametrize("layout", ["bhnd", "bnhd"])
@pytest.mark.parametrize("local_prev", [1, 2])
@pytest.mark.parametrize("cfg", BF16_D64, ids=[f"n{c['n']}_L{c['L']}_K{c['K']}_G{c['Hq'] // c['Hkv']}" for c in BF16_D64])
def test_bf16_head_dim_64(cfg, local_prev, layout):
    w = inputs.small_workload(d=64, dtype="bf16", **cfg)
    x = inputs.make_inputs(w)
    idx, want = reference(w, x, local_prev)
    idx_dev = None if idx is None else torch.from_numpy(idx).to(DEV)
    xd = {k: v.to(DEV) if layout == "bhnd" else rows_strided(v.to(DEV)) for k, v in x.items()}
    got, names = run(w, xd, idx_dev, lrsa.IMPL_AUTO, local_prev=local_prev)
    assert {"k_fwd_mfma", "k_bwd_dq", "k_bwd_dkv"} <= names
    plain, names = run(w, xd, idx_dev, lrsa.IMPL_GENERIC, local_prev=local_prev)
    assert not any("mfma" in n for n in names)
    for k in want:
        bar = 1.05 * err(plain[k], want[k]) + 2.0 ** -16
        assert err(got[k], want[k]) <= bar, f"{k}: {err(got[k], want[k]):.3e} (bar {bar:.3e})"


@pytest.mark.parametrize("structure", ["none", "channel_scale"])
def test_bf16_head_dim_64_keeps_fp32_weights(structure):
    """O and dV are sums of weights times bf16 numbers, rounded once to bf16: with fp32 weights an element misses the correctly
    rounded exact value only where that lies within some 2^-24 of a rounding boundary.  Their number grows with the error of the
    weights (two bf16 terms, 2^-17: about eight times as many as the plain fp32-arithmetic kernels miss).  Bar: twice the plain kernels'
    number, and 10 for the spread of the small counts."""
    w = inputs.small_workload(d=64, dtype="bf16", n=16 + 10 * 128 + 100, L=128, S=16, K=32, Hq=8, Hkv=2, structure=structure)
    x = inputs.make_inputs(w)
    idx, want = reference(w, x, 1)
    idx_dev = torch.from_numpy(idx).to(DEV)
    xd = {k: v.to(DEV) for k, v in x.items()}
    got, _ = run(w, xd, idx_dev, lrsa.IMPL_AUTO)
    plain, _ = run(w, xd, idx_dev, lrsa.IMPL_GENERIC)
    for k in ("O", "dV"):
        ideal = torch.from_numpy(want[k]).to(torch.bfloat16)
        missed = [int((o[k].cpu() != ideal).sum()) for o in (got, plain)]
        assert missed[0] <= 2 * missed[1] + 10, f"{k}: {missed[0]} elements off the correct rounding, the plain kernels {missed[1]}"


# tiles: 16 keys, 16 query rows; 16, 8 or 4 waves (head_dim 64; 8 or 4: 128) take the tiles in turn; up to 8 workgroups share the rows
# of a key tile, one where there are more than 512 key tiles
F32 = [
    dict(n=1, L=8, S=0, K=2, Hq=1, Hkv=1),
    dict(n=40, L=32, S=64, K=8, Hq=2, Hkv=1),                       # sink only
    dict(n=6 + 2 * 32, L=32, S=6, K=8, Hq=2, Hkv=1),                # nothing compressed
    dict(n=5 + 7 * 50 + 33, L=50, S=5, K=17, Hq=6, Hkv=2, B=2),     # 33 rows of a chunk do not survive: 2 tiles and a row
    dict(n=17 + 5 * 65 + 1, L=65, S=17, K=16, Hq=4, Hkv=1),         # tail of one row, sink one past a tile
    dict(n=3 + 6 * 33 + 32, L=33, S=3, K=33, Hq=2, Hkv=2),          # every token survives
    dict(n=4 + 9 * 48, L=48, S=4, K=1, Hq=3, Hkv=3, B=2),           # one survivor per chunk
    dict(n=64 + 3 * 300 + 77, L=300, S=64, K=75, Hq=16, Hkv=8, B=1),   # one slice, several workgroups per CU
]


@pytest.mark.parametrize("layout", ["bhnd", "bnhd"])
@pytest.mark.parametrize("local_prev", [1, 2])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("cfg", F32, ids=[f"n{c['n']}_L{c['L']}_K{c['K']}_G{c['Hq'] // c['Hkv']}" for c in F32])
def test_f32(cfg, d, local_prev, layout):
    w = inputs.small_workload(d=d, dtype="f32", **cfg)
    x = inputs.make_inputs(w)
    idx, want = reference(w, x, local_prev)
    idx_dev = None if idx is None else torch.from_numpy(idx).to(DEV)
    xd = {k: v.to(DEV) if layout == "bhnd" else rows_strided(v.to(DEV)) for k, v in x.items()}
    got, names = run(w, xd, idx_dev, lrsa.IMPL_AUTO, local_prev=local_prev)
    assert names - {"k_bwd_dkv_f32_sum"} == {"k_fwd_f32", "k_bwd_dq_f32", "k_bwd_dkv_f32"}
    plain, names = run(w, xd, idx_dev, lrsa.IMPL_GENERIC, local_prev=local_prev)
    assert not any("f32" in n for n in names)
    for k in want:
        bar = 1.25 * err(plain[k], want[k]) + 2.0 ** -23
        assert err(got[k], want[k]) <= bar, f"{k}: {err(got[k], want[k]):.3e} (bar {bar:.3e})"


@pytest.mark.parametrize("dtype,B", [("f32", 64), ("bf16", 65)])
def test_more_heads_than_a_launch_of_the_tiled_kernels_holds(dtype, B):
    """B x 65535 query heads of three rows: two query tiles of fp32 per head, 1024 threads each, are past 2^32 work-items, and bf16 at lag 2
    has few keys per row, so the plain kernels serve the call.  All keys are visible causally (two chunks); some heads against 64 bits, dK and dV over
    all heads."""
    dt = {"f32": torch.float32, "bf16": torch.bfloat16}[dtype]
    Hq, n, d = 65535, 3, 64
    g = torch.Generator(device=DEV).manual_seed(11)
    Q, dO = (torch.randn((B, Hq, n, d), generator=g, device=DEV, dtype=dt) for _ in range(2))
    K, V = (torch.randn((B, 1, n, d), generator=g, device=DEV, dtype=dt) for _ in range(2))
    p = lrsa.params_for(Q, K, sink=0, lag=2, topk=1)
    assert lrsa.attn_route(p) == 0 and lrsa.num_scored_chunks(p) == 0
    O, lse = lrsa.lrsa_attn_fwd(p, Q, K, V, None)
    dQ, dK, dV = lrsa.lrsa_attn_bwd(p, Q, K, V, O, dO, lse, None)
    mask = torch.ones(n, n, dtype=torch.bool, device=DEV).tril()
    # roundings of the results, and of some hundred (dK, dV: 200 K) fp32 additions
    tol, tol_kv = {"f32": (2e-6, 2e-5), "bf16": (1e-2, 1e-2)}[dtype]
    for b in (0, B - 1):
        Kb, Vb = K[b, 0].double(), V[b, 0].double()
        q, o, go = (t[b].double() for t in (Q, dO, O))
        s = (q @ Kb.T * d ** -0.5).masked_fill(~mask, float("-inf"))
        P = torch.softmax(s, -1)
        want_O = P @ Vb
        dS = P * (o @ Vb.T - (o * want_O).sum(-1, keepdim=True)) * d ** -0.5
        for got, want, t in ((go, want_O, tol), (lse[b].double(), torch.logsumexp(s, -1), tol), (dQ[b].double(), dS @ Kb, 2 * tol),
                             (dK[b, 0].double(), (dS.transpose(1, 2) @ q).sum(0), tol_kv), (dV[b, 0].double(), (P.transpose(1, 2) @ o).sum(0), tol_kv)):
            assert (got - want).norm() <= t * want.norm()


@pytest.mark.parametrize("which", ["K", "V", "Q", "dO"])
@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("f32", 64), ("f32", 128)])
def test_non_finite_rows_stay_with_those_that_see_them(dtype, d, which):
    """Infinities and NaN in a row (padding behind the end, say) reach only the queries that see the key and the keys that the query
    sees, although a tile multiplies its masked pairs by zero.  Everything else is as with finite values there: the same bits in
    fp32; in bf16 up to the last bit (a wave refreshes its running maxima for all of its queries at once)."""
    def same(a, b):
        return torch.equal(a, b) if dtype == "f32" else bool(a.isfinite().all()) and bool((a - b).float().norm() <= 2.0 ** -9 * b.float().norm())

    w = inputs.small_workload(d=d, dtype=dtype, n=5 + 6 * 72 + 41, L=72, S=5, K=20, Hq=4, Hkv=2)
    x = inputs.make_inputs(w)
    idx, _ = reference(w, x, 1)
    idx_dev = torch.from_numpy(idx).to(DEV)
    clean, _ = run(w, {k: v.to(DEV) for k, v in x.items()}, idx_dev, lrsa.IMPL_AUTO)
    # rows inside and at the edges of tiles, in a chunk that is compressed, in the last ones, the last row; values in a few channels
    rows = [5 + 2 * 72 + 25, 5 + 4 * 72, 5 + 5 * 72 + 16, w.n - 9, w.n - 1]
    for i, t in enumerate(rows):
        for c, v in ((i, float("nan")), (17 + i, float("-inf")), (40 + i, float("inf")))[:1 if i % 2 else 3]:
            x[which][:, :, t, c] = v
    got, _ = run(w, {k: v.to(DEV) for k, v in x.items()}, idx_dev, lrsa.IMPL_AUTO)
    bad = torch.zeros(w.n, dtype=torch.bool)
    bad[rows] = True
    for hq in range(w.Hq):
        h = hq // (w.Hq // w.Hkv)
        vis = torch.from_numpy(ref.visible_mask(w.n, w.S, w.L, idx[0, h], 1))
        q_bad = (vis & bad).any(1) if which in "KV" else bad
        assert 0 < q_bad.sum() < w.n
        for k in ("O", "lse", "dQ"):
            if which == "dO" and k != "dQ":
                assert torch.equal(got[k], clean[k])
                continue
            a, b = got[k][0, hq].cpu(), clean[k][0, hq].cpu()
            assert same(a[~q_bad], b[~q_bad]), f"{k}: {which} reaches queries that do not see it"
            if k != "lse":
                assert not a[q_bad].isfinite().all(-1).any(), f"{k}: a query that sees {which} does not show it"
        k_bad = (vis & q_bad[:, None]).any(0)                # keys that an affected query sees
        assert 0 < k_bad.sum() < w.n
        for k in ("dK", "dV"):
            if which in ("Q", "dO"):
                assert not got[k][0, h].cpu()[(vis & bad[:, None]).any(0)].isfinite().all(-1).any(), f"{k}: {which} does not show"
            a, b = got[k][0, h].cpu(), clean[k][0, h].cpu()
            assert same(a[~k_bad], b[~k_bad]), f"{k}: {which} reaches keys that no affected query sees"
