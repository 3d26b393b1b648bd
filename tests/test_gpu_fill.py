"""Attention by filling steps (lrsa_attn_fwd_fill / lrsa_attn_bwd_fill / lrsa_attn_bwd_finish; Section 3.2 of the
paper, Attention Filling 1 / 2 / repeat): m query chunks per step against sink + survivors + the previous chunk.

Bars: O, lse and dQ of the steps, put together, equal the one-shot calls bit for bit (same tiles, same walk);
dK, dV equal them within the bf16 tolerance (the fp32 additions come in another order); everything is within
2e-2 relative of the fp64 oracle, which knows nothing of steps.  The workspace of a step is printed beside the
one-shot workspace.
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
    dict(name="gqa", n=16 + 6 * 64 + 40, L=64, S=16, K=16, d=128, Hq=8, Hkv=2, B=2),
    dict(name="odd_sizes_no_tail_chunk", n=5 + 7 * 100, L=100, S=5, K=37, d=128, Hq=2, Hkv=1, B=1),
    dict(name="no_sink_long_chunks", n=0 + 5 * 320 + 100, L=320, S=0, K=80, d=128, Hq=4, Hkv=1, B=1),
    dict(name="heads_in_uneven_parts", n=16 + 9 * 128 + 50, L=128, S=16, K=32, d=128, Hq=10, Hkv=2, B=1),
    dict(name="group_of_six", n=7 + 12 * 96 + 20, L=96, S=7, K=24, d=128, Hq=6, Hkv=1, B=1),
    dict(name="many_chunks", n=64 + 20 * 128 + 9, L=128, S=64, K=32, d=128, Hq=8, Hkv=1, B=1),
]


def windows(w, m):
    """Row windows of the filling steps: the sink with the first m chunks, then m chunks at a time."""
    if w.n <= w.S:
        return [(0, w.n)]
    nq = -(-(w.n - w.S) // w.L)
    cuts = [0] + [w.S + q * w.L for q in range(m, nq, m)] + [w.n]
    return list(zip(cuts[:-1], cuts[1:]))


def rel(x, r):
    x = np.asarray(x, np.float64); r = np.asarray(r, np.float64)
    return max(np.abs(x - r).max() / np.abs(r).max(), np.linalg.norm(x - r) / np.linalg.norm(r))


@pytest.mark.parametrize("m", [1, 2, 3])
@pytest.mark.parametrize("local_prev", [1, 2])
@pytest.mark.parametrize("cfg", SHAPES, ids=[c["name"] for c in SHAPES])
def test_filling_steps_equal_one_shot_and_oracle(cfg, m, local_prev):
    if local_prev == 2 and cfg["name"] != "gqa":
        pytest.skip("local_prev = 2 is exercised on one shape")
    cfg = {k: v for k, v in cfg.items() if k != "name"}
    w = inputs.small_workload(dtype="bf16", **cfg)
    x = inputs.make_inputs(w)
    xf = {k: v.float().numpy() for k, v in x.items()}
    xd = {k: v.to(DEV) for k, v in x.items()}
    p = lrsa.params_for(xd["Q"], xd["K"], sink=w.S, lag=w.L, topk=w.K, local_prev=local_prev)
    Ns = lrsa.num_scored_chunks(p)
    idx_ref = ref.select(ref.score(xf["K"], xf["V"], w.S, w.L, local_prev=local_prev), w.S, w.L, w.K) if Ns else None
    idx = torch.from_numpy(idx_ref).to(DEV) if Ns else None
    O1, lse1 = lrsa.lrsa_attn_fwd(p, xd["Q"], xd["K"], xd["V"], idx)
    dQ1, dK1, dV1 = lrsa.lrsa_attn_bwd(p, xd["Q"], xd["K"], xd["V"], O1, xd["dO"], lse1, idx)

    O = torch.zeros_like(O1); lse = torch.zeros_like(lse1); dQ = torch.zeros_like(dQ1)
    accK = torch.zeros(xd["K"].shape, dtype=torch.float32, device=DEV)
    accV = torch.zeros_like(accK)
    steps = windows(w, m)
    ws_fwd = ws_bwd = 0
    for a, b in steps:
        Qs = xd["Q"][:, :, a:b].contiguous()
        pf = lrsa.params_for(Qs, xd["K"], sink=w.S, lag=w.L, topk=w.K, local_prev=local_prev)
        pf.seq = w.n
        ws_fwd = max(ws_fwd, lrsa.fill_workspace_bytes(pf, a, b, 2))
        Os, ls = lrsa.lrsa_attn_fwd_fill(pf, a, b, Qs, xd["K"], xd["V"], idx)
        O[:, :, a:b] = Os
        lse[:, :, a:b] = ls
    assert torch.equal(O, O1) and torch.equal(lse, lse1)
    for a, b in reversed(steps):
        Qs, Os, dOs = (xd[k][:, :, a:b].contiguous() if k != "O" else O[:, :, a:b].contiguous() for k in ("Q", "O", "dO"))
        pf = lrsa.params_for(Qs, xd["K"], sink=w.S, lag=w.L, topk=w.K, local_prev=local_prev)
        pf.seq = w.n
        ws_bwd = max(ws_bwd, lrsa.fill_workspace_bytes(pf, a, b, 3))
        dQ[:, :, a:b] = lrsa.lrsa_attn_bwd_fill(pf, a, b, Qs, xd["K"], xd["V"], Os, dOs, lse[:, :, a:b].contiguous(), idx, accK, accV)
    dK, dV = torch.empty_like(xd["K"]), torch.empty_like(xd["K"])
    lrsa.lrsa_attn_bwd_finish(p, accK, accV, dK, dV)
    torch.cuda.synchronize()
    print(f"m={m}: workspace per step fwd {ws_fwd} / bwd {ws_bwd} bytes; one-shot fwd {lrsa.workspace_bytes(p, 2)} / "
          f"bwd {lrsa.workspace_bytes(p, 3)} bytes")
    assert torch.equal(dQ, dQ1)
    assert rel(dK.float().cpu().numpy(), dK1.float().cpu().numpy()) < 2e-2
    assert rel(dV.float().cpu().numpy(), dV1.float().cpu().numpy()) < 2e-2
    O_ref, lse_ref = ref.attn_fwd_dense(xf["Q"], xf["K"], xf["V"], idx_ref, w.S, w.L, local_prev=local_prev)
    g = ref.attn_bwd_dense(xf["Q"], xf["K"], xf["V"], xf["dO"], idx_ref, w.S, w.L, local_prev=local_prev)
    assert rel(O.float().cpu().numpy(), O_ref) < 2e-2
    assert np.abs(lse.cpu().numpy() - lse_ref).max() < 1e-3
    assert rel(dQ.float().cpu().numpy(), g[0]) < 2e-2
    assert rel(dK.float().cpu().numpy(), g[1]) < 2e-2
    assert rel(dV.float().cpu().numpy(), g[2]) < 2e-2


def test_filling_steps_at_full_size_C4_equal_the_one_shot_call():
    """The headline workload (32K tokens, 32/8 heads) in steps of 4 chunks, with the library's own selection:
    O, lse and dQ bit for bit, dK and dV within 2e-3 of the one-shot call (which the full-size parity tests hold
    against the oracle); the step-wise schedule's time and workspace are printed beside the one-shot call's."""
    w = inputs.WORKLOADS["C4"]
    xd = {k: v.to(DEV) for k, v in inputs.make_inputs(w).items()}
    p = lrsa.params_for(xd["Q"], xd["K"], sink=w.S, lag=w.L, topk=w.K)
    _, idx = lrsa.lrsa_score_select(p, xd["K"], xd["V"])
    O1, lse1 = lrsa.lrsa_attn_fwd(p, xd["Q"], xd["K"], xd["V"], idx)
    dQ1, dK1, dV1 = lrsa.lrsa_attn_bwd(p, xd["Q"], xd["K"], xd["V"], O1, xd["dO"], lse1, idx)
    torch.cuda.synchronize()
    m = 4
    steps = windows(w, m)
    O = torch.empty_like(O1); lse = torch.empty_like(lse1); dQ = torch.empty_like(dQ1)
    accK = torch.zeros(xd["K"].shape, dtype=torch.float32, device=DEV)
    accV = torch.zeros_like(accK)
    dK, dV = torch.empty_like(xd["K"]), torch.empty_like(xd["K"])
    params = {}
    for a, b in steps:
        pf = lrsa.params_for(xd["Q"][:, :, a:b], xd["K"], sink=w.S, lag=w.L, topk=w.K)   # Q, O, dO, dQ rows as views
        pf.seq = w.n
        params[(a, b)] = pf
    ws = torch.empty(max(max(lrsa.fill_workspace_bytes(params[s_], s_[0], s_[1], k) for s_ in steps) for k in (2, 3)) + 256,
                     dtype=torch.uint8, device=DEV)
    lse_rows = {s_: torch.empty((w.B, w.Hq, s_[1] - s_[0]), dtype=torch.float32, device=DEV) for s_ in steps}   # contiguous per step
    for timed in (False, True):          # the first pass warms the allocator and the code objects up
        accK.zero_(); accV.zero_()
        t0, t1, t2 = (torch.cuda.Event(enable_timing=True) for _ in range(3))
        t0.record()
        for a, b in steps:
            lrsa.lrsa_attn_fwd_fill(params[(a, b)], a, b, xd["Q"][:, :, a:b], xd["K"], xd["V"], idx, O[:, :, a:b], lse_rows[(a, b)], ws)
        t1.record()
        for a, b in reversed(steps):
            lrsa.lrsa_attn_bwd_fill(params[(a, b)], a, b, xd["Q"][:, :, a:b], xd["K"], xd["V"], O[:, :, a:b], xd["dO"][:, :, a:b],
                                    lse_rows[(a, b)], idx, accK, accV, dQ[:, :, a:b], ws)
        lrsa.lrsa_attn_bwd_finish(p, accK, accV, dK, dV)
        t2.record()
        torch.cuda.synchronize()
    for a, b in steps:
        lse[:, :, a:b] = lse_rows[(a, b)]
    print(f"C4 in {len(steps)} steps of {m} chunks: forward {t0.elapsed_time(t1):.2f} ms, backward {t1.elapsed_time(t2):.2f} ms "
          f"(host-driven, includes launch gaps); workspace {ws.numel() / 1e6:.0f} MB + {2 * accK.numel() * 4 / 1e6:.0f} MB of accumulators "
          f"against {lrsa.workspace_bytes(p, 3) / 1e6:.0f} MB one-shot")
    assert torch.equal(O, O1) and torch.equal(lse, lse1) and torch.equal(dQ, dQ1)
    for name, x, r in (("dK", dK, dK1), ("dV", dV, dV1)):
        x = x.float(); r = r.float()
        e = max(((x - r).abs().max() / r.abs().max()).item(), ((x - r).norm() / r.norm()).item())
        assert e < 2e-3, (name, e)


def test_fill_rejects_windows_off_the_chunk_grid():
    w = inputs.small_workload(n=16 + 6 * 64 + 40, L=64, S=16, K=16, d=128, Hq=4, Hkv=2, B=1, dtype="bf16")
    xd = {k: v.to(DEV) for k, v in inputs.make_inputs(w).items()}
    p = lrsa.params_for(xd["Q"], xd["K"], sink=w.S, lag=w.L, topk=w.K)
    for a, b in ((0, 50), (17, 16 + 64), (16 + 64, 16 + 64), (16, w.n + 1)):
        assert lrsa.fill_workspace_bytes(p, a, b, 3) == 0


@pytest.mark.parametrize("Hkv,G", [(1, 4), (3, 2)])
def test_steps_that_see_no_compressed_chunk_need_no_idx(Hkv, G):
    """idx may be missing as long as the step's queries see no compressed chunk (the first two chunks): same bits as with one."""
    w = inputs.small_workload(n=16 + 6 * 64 + 40, L=64, S=16, K=16, d=128, Hq=Hkv * G, Hkv=Hkv, B=2, dtype="bf16")
    xd = {k: v.to(DEV) for k, v in inputs.make_inputs(w).items()}
    kw = dict(sink=w.S, lag=w.L, topk=w.K)
    _, idx = lrsa.lrsa_score_select(lrsa.params_for(xd["Q"], xd["K"], **kw), xd["K"], xd["V"])
    for a, b in ((0, 16 + 64), (16 + 64, 16 + 128), (0, 16 + 128)):
        Qs, dOs = xd["Q"][:, :, a:b].contiguous(), xd["dO"][:, :, a:b].contiguous()
        p = lrsa.params_for(Qs, xd["K"], **kw)
        p.seq = w.n
        res = []
        for list_ in (idx, None):
            O, lse = lrsa.lrsa_attn_fwd_fill(p, a, b, Qs, xd["K"], xd["V"], list_)
            acc = [torch.zeros(xd["K"].shape, dtype=torch.float32, device=DEV) for _ in range(2)]
            dQ = lrsa.lrsa_attn_bwd_fill(p, a, b, Qs, xd["K"], xd["V"], O, dOs, lse, list_, *acc)
            res.append((O, lse, dQ, *acc))
        for x, y in zip(*res):
            assert torch.equal(x, y)
    p = lrsa.params_for(xd["Q"], xd["K"], **kw)
    with pytest.raises(lrsa.LrsaError, match="idx"):
        lrsa.lrsa_attn_fwd_fill(p, 0, w.n, xd["Q"], xd["K"], xd["V"], None)


def test_a_workspace_for_the_last_whole_step_serves_every_step():
    """The split plan of an early step may need more than the last step; with that one's workspace it takes the plan without
    splits: dQ the same bits, dK and dV up to the order of the additions."""
    w = inputs.small_workload(n=4087, L=170, S=0, K=42, d=128, Hq=6, Hkv=1, B=4, dtype="bf16")
    xd = {k: v.to(DEV) for k, v in inputs.make_inputs(w).items()}
    kw = dict(sink=w.S, lag=w.L, topk=w.K)
    p = lrsa.params_for(xd["Q"], xd["K"], **kw)
    _, idx = lrsa.lrsa_score_select(p, xd["K"], xd["V"])
    steps = windows(w, 1)
    last = max(s for s in steps if s[1] - s[0] == w.L)
    pq = lrsa.params_for(xd["Q"][:, :, :w.L], xd["K"], **kw)                   # Q, O, dO, dQ rows as views
    pq.seq = w.n
    small = lrsa.fill_workspace_bytes(pq, *last, 3)
    assert max(lrsa.fill_workspace_bytes(pq, a, b, 3) for a, b in steps) > 1.2 * small
    O, lse = lrsa.lrsa_attn_fwd(p, xd["Q"], xd["K"], xd["V"], idx)
    out = []
    for ws in (None, torch.empty(small, dtype=torch.uint8, device=DEV)):
        acc = [torch.zeros(xd["K"].shape, dtype=torch.float32, device=DEV) for _ in range(2)]
        dQ = torch.empty_like(xd["Q"])
        for a, b in steps:
            lrsa.lrsa_attn_bwd_fill(pq, a, b, xd["Q"][:, :, a:b], xd["K"], xd["V"], O[:, :, a:b], xd["dO"][:, :, a:b], lse[:, :, a:b].contiguous(), idx,
                                    *acc, dQ[:, :, a:b], ws)
        out.append((dQ, *acc))
    assert torch.equal(out[0][0], out[1][0])
    for a, b in zip(out[0][1:], out[1][1:]):
        assert (a - b).norm() <= 1e-6 * a.norm()                              # fp32 sums of some hundred to thousand bf16 products
    with pytest.raises(lrsa.LrsaError, match="workspace"):
        lrsa.lrsa_attn_bwd_fill(pq, *last, xd["Q"][:, :, :w.L], xd["K"], xd["V"], O[:, :, :w.L], xd["dO"][:, :, :w.L], lse[:, :, :w.L].contiguous(),
                                idx, *acc, None, torch.empty(1 << 16, dtype=torch.uint8, device=DEV))


def _steps_and_parts(w, m, **kw):
    p = lrsa.make_params((w.B, w.Hq, w.n, w.d), (w.B, w.Hkv, w.n, w.d), (w.Hq * w.n * w.d, w.n * w.d, w.d, 1), (w.Hkv * w.n * w.d, w.n * w.d, w.d, 1),
                         dtype=torch.bfloat16, sink=w.S, lag=w.L, topk=w.K, **kw)
    return [lrsa.attn_bwd_parts(p, a, b) for a, b in (windows(w, m) if m else [(0, w.n)])]


def test_the_shapes_above_split_the_heads():
    """The filling steps and the one-shot calls that are compared above take the split paths of dK/dV: parts of both kinds of work, even
    and uneven ones and different numbers in the steps of one call."""
    seen = {}
    for cfg in SHAPES:
        w = inputs.small_workload(dtype="bf16", **{k: v for k, v in cfg.items() if k != "name"})
        seen[cfg["name"]] = {m: _steps_and_parts(w, m) for m in (0, 1, 2, 3)}
    assert all(min(g, x) > 1 for by_m in seen.values() for parts in by_m.values() for g, x in parts)
    assert seen["heads_in_uneven_parts"][0] == [(2, 5)] and seen["group_of_six"][0] == [(2, 3)]     # 5 heads in 2 parts
    assert {g for g, _ in seen["many_chunks"][2]} == {4, 8} and len(set(seen["gqa"][3])) == 2
    w = inputs.WORKLOADS["C4"]
    assert _steps_and_parts(w, 0) == [(1, 1)]                                  # a long call stays whole


@pytest.mark.parametrize("cfg", [c for c in SHAPES if c["name"] in ("heads_in_uneven_parts", "group_of_six", "odd_sizes_no_tail_chunk")],
                         ids=lambda c: c["name"])
def test_condensed_cache_with_split_heads_equals_gathering(cfg):
    w = inputs.small_workload(dtype="bf16", **{k: v for k, v in cfg.items() if k != "name"})
    xd = {k: v.to(DEV) for k, v in inputs.make_inputs(w).items()}
    res = []
    for impl in (lrsa.IMPL_AUTO, lrsa.IMPL_COMPACT):
        assert min(_steps_and_parts(w, 0, impl=impl)[0]) > 1
        p = lrsa.params_for(xd["Q"], xd["K"], sink=w.S, lag=w.L, topk=w.K, impl=impl)
        _, idx = lrsa.lrsa_score_select(p, xd["K"], xd["V"])
        O, lse = lrsa.lrsa_attn_fwd(p, xd["Q"], xd["K"], xd["V"], idx)
        lrsa.timing_enable(True)
        grads = lrsa.lrsa_attn_bwd(p, xd["Q"], xd["K"], xd["V"], O, xd["dO"], lse, idx)
        torch.cuda.synchronize()
        names = {n for n, _ in lrsa.timing_records()}
        lrsa.timing_enable(False)
        assert ("k_bwd_scatter_dkv" in names) == (impl == lrsa.IMPL_COMPACT)
        res.append((O, lse, *grads))
    for a, b in zip(*res):
        assert torch.equal(a, b)


@pytest.mark.parametrize("m", [1, 2])
@pytest.mark.parametrize("cfg,lp", [(dict(B=2, Hq=16, Hkv=8, n=2161, L=499, K=235, S=33), 1), (dict(B=4, Hq=6, Hkv=1, n=2782, L=689, K=296, S=5), 2)],
                         ids=["n2161_L499", "n2782_L689"])
def test_filling_steps_with_eight_waves_equal_the_one_shot_call(cfg, lp, m):
    """Steps whose dK/dV kernel has eight waves, at lags that leave rows and keys of a step partly filled, with their forward and dQ in four waves where
    the one-shot call has eight: the same bits in O, lse and dQ, and dK, dV up to one rounding to bf16 of fp32 sums in another order."""
    w = inputs.small_workload(d=128, dtype="bf16", **cfg)
    x = {k: v.to(DEV) for k, v in inputs.make_inputs(w).items()}
    kw = dict(sink=w.S, lag=w.L, topk=w.K, local_prev=lp)
    p = lrsa.params_for(x["Q"], x["K"], **kw)
    _, idx = lrsa.lrsa_score_select(p, x["K"], x["V"])
    O, lse = lrsa.lrsa_attn_fwd(p, x["Q"], x["K"], x["V"], idx)
    want = lrsa.lrsa_attn_bwd(p, x["Q"], x["K"], x["V"], O, x["dO"], lse, idx)
    acc = [torch.zeros(x["K"].shape, dtype=torch.float32, device=DEV) for _ in range(2)]
    waves = set()
    for a, b in windows(w, m):
        q, do = (x[k][:, :, a:b].contiguous() for k in ("Q", "dO"))
        pf = lrsa.params_for(q, x["K"], **kw)
        pf.seq = w.n
        waves.add((lrsa.attn_plan(pf, a, b).dq_waves, lrsa.attn_plan(pf, a, b).key_waves))
        o, ls = lrsa.lrsa_attn_fwd_fill(pf, a, b, q, x["K"], x["V"], idx)
        dq = lrsa.lrsa_attn_bwd_fill(pf, a, b, q, x["K"], x["V"], o, do, ls, idx, *acc)
        for got, whole in ((o, O), (ls, lse), (dq, want[0])):
            assert torch.equal(got, whole[:, :, a:b])
    assert lrsa.attn_plan(p).dq_waves == 8 and (4, 8) in waves
    for a, b in zip(acc, want[1:]):
        b = b.double()
        assert ((a.double() - b).abs() <= 2.0 ** -8 * b.abs() + 2.0 ** -18 * b.abs().max()).all()
