"""Inference-time LagKV cache on the GPU (lrsa_cache_compress, lrsa_decode_attn) against the CPU oracle.

Bars: the compressed cache and its position array are copies of input rows, so they must equal the oracle's
bit for bit whenever the selection does (it is checked against the oracle's tie window otherwise, as for the
training-time selection); the attention output within 1e-4 (fp32) / 2e-2 (bf16) relative, lse within 1e-3.
"""
import numpy as np
import pytest
import torch

import paper_2506_11498_amd as lrsa
from paper_2506_11498_amd import inputs
from oracle import lrsa_decode as dec
from oracle import lrsa_ref as ref

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    dict(n=3 + 5 * 16 + 7, L=16, S=3, K=4, d=64, Hq=2, Hkv=1, B=2, dtype="f32"),
    dict(n=0 + 4 * 24 + 1, L=24, S=0, K=24, d=128, Hq=2, Hkv=2, B=1, dtype="f32"),          # keep everything
    dict(n=8 + 5 * 32 + 11, L=32, S=8, K=8, d=64, Hq=4, Hkv=2, B=1, dtype="bf16"),
    dict(n=16 + 4 * 256 + 100, L=256, S=16, K=64, d=128, Hq=8, Hkv=2, B=2, dtype="bf16"),
    dict(n=64 + 3 * 1024 + 500, L=1024, S=64, K=256, d=128, Hq=12, Hkv=1, B=1, dtype="bf16"),  # group of 12: two passes
    dict(n=5, L=8, S=16, K=2, d=64, Hq=1, Hkv=1, B=1, dtype="f32"),                          # shorter than the sink
]


def feed_cache(w, x, feed):
    """Appends the rows of K, V to a device cache `feed` tokens at a time (never past a tail of 2L), compressing
    before each append as the header asks.  Returns (Kc, Vc, pos, length, done) as the last token sees them."""
    cap = w.S + 2 * w.L + w.n            # generous
    Kc = torch.zeros((w.B, w.Hkv, cap, w.d), dtype=x["K"].dtype, device=DEV)
    Vc = torch.zeros_like(Kc)
    p = lrsa.make_params((w.B, w.Hq, cap, w.d), tuple(Kc.shape), (w.Hq * cap * w.d, cap * w.d, w.d, 1), Kc.stride(),
                         dtype=Kc.dtype, sink=w.S, lag=w.L, topk=w.K)
    pos = torch.full((w.B, w.Hkv, cap), -1, dtype=torch.int32, device=DEV)
    Kd, Vd = x["K"].to(DEV), x["V"].to(DEV)
    length = done = t = 0
    while t < w.n:
        length, done = lrsa.lrsa_cache_compress(p, Kc, Vc, pos, length, done)
        room = (w.S + w.K * done + 2 * w.L) - length     # rows until the tail holds 2L
        m = max(1, min(feed, w.n - t, room))
        Kc[:, :, length:length + m] = Kd[:, :, t:t + m]
        Vc[:, :, length:length + m] = Vd[:, :, t:t + m]
        pos[:, :, length:length + m] = torch.arange(t, t + m, dtype=torch.int32, device=DEV)
        length += m
        t += m
    return p, Kc, Vc, pos, length, done


@pytest.mark.parametrize("feed", [1, 7, 4096])
@pytest.mark.parametrize("cfg", CASES, ids=[f"n{c['n']}_L{c['L']}_{c['dtype']}" for c in CASES])
def test_cache_and_decode_attention_against_oracle(cfg, feed):
    if feed == 1 and cfg["n"] > 600:
        pytest.skip("token-by-token feeding is exercised on the short cases")
    w = inputs.small_workload(**cfg)
    x = inputs.make_inputs(w)
    p, Kc, Vc, pos, length, done = feed_cache(w, x, feed)
    Kf, Vf = x["K"].float().numpy(), x["V"].float().numpy()
    t = 1e-4 if w.dtype == "f32" else 2e-2
    q = x["Q"][:, :, w.n - 1].contiguous().to(DEV)           # the last token's queries
    O, lse = lrsa.lrsa_decode_attn(p, q, Kc, Vc, length)
    O, lse = O.float().cpu().numpy(), lse.cpu().numpy()
    for b in range(w.B):
        for h in range(w.Hkv):
            Ko, Vo, po, do = dec.cache_incremental(Kf[b, h], Vf[b, h], w.S, w.L, w.K)
            assert (length, done) == (len(po), do)
            got = pos[b, h, :length].cpu().numpy()
            if not np.array_equal(got, po):
                # the two selections may differ only inside the oracle's fp32 tie window
                sc = ref.score(Kf[b:b + 1, h:h + 1], Vf[b:b + 1, h:h + 1], w.S, w.L)[0, 0]
                for c in range(do):
                    a, o = got[w.S + c * w.K: w.S + (c + 1) * w.K], po[w.S + c * w.K: w.S + (c + 1) * w.K]
                    s = sc[c]
                    diff = np.setxor1d(a, o) - (w.S + c * w.L)
                    assert np.all(np.abs(s[diff] - np.sort(s)[-w.K]) <= 1e-6)
                Ko, Vo = Kf[b, h][got], Vf[b, h][got]
            assert np.array_equal(Kc[b, h, :length].float().cpu().numpy(), Ko)
            assert np.array_equal(Vc[b, h, :length].float().cpu().numpy(), Vo)
            sl = slice(h * w.G, (h + 1) * w.G)
            O_ref, lse_ref = dec.decode_attn(x["Q"][b, sl, w.n - 1].float().numpy(), Ko, Vo)
            top = max(np.abs(O_ref).max(), 1e-2)
            assert np.abs(O[b, sl] - O_ref).max() / top < t
            assert np.abs(lse[b, sl] - lse_ref).max() < 1e-3


def test_compress_is_a_no_op_below_two_chunks_and_rejects_bad_lengths():
    w = inputs.small_workload(n=100, L=16, S=4, K=4, d=64, Hq=1, Hkv=1, B=1, dtype="f32")
    Kc = torch.randn((1, 1, 128, 64), device=DEV)
    p = lrsa.make_params((1, 1, 128, 64), (1, 1, 128, 64), Kc.stride(), Kc.stride(), dtype=torch.float32, sink=4, lag=16, topk=4)
    Vc = torch.randn_like(Kc)
    K0 = Kc.clone()
    assert lrsa.lrsa_cache_compress(p, Kc, Vc, None, 4 + 31, 0) == (35, 0)
    assert torch.equal(Kc, K0)
    assert lrsa.lrsa_cache_compress(p, Kc, Vc, None, 4 + 32, 0) == (4 + 4 + 16, 1)
    with pytest.raises(lrsa.LrsaError):
        lrsa.lrsa_cache_compress(p, Kc, Vc, None, 200, 0)       # beyond the capacity
    with pytest.raises(lrsa.LrsaError):
        lrsa.lrsa_decode_attn(p, torch.randn((1, 1, 64), device=DEV), Kc, Vc, 0)


@pytest.mark.parametrize("G", [1, 3, 16, 17])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("length", [1, 31, 33, 127, 129, 1000])
def test_decode_attention_at_tile_edges(d, G, length):
    """bf16 on the matrix cores: lengths around the 32-row tiles and the slices, groups around the 16 columns of a tile, rows
    behind the end that hold infinities (never to be used).  K grows along the cache, so that the running maximum moves."""
    B, Hkv, cap = 2, 2, length + 40
    g = torch.Generator().manual_seed(length * 100 + G)
    Kc = (torch.randn((B, Hkv, cap, d), generator=g) * torch.linspace(0.2, 3.0, cap)[:, None]).to(torch.bfloat16)
    Vc = torch.randn((B, Hkv, cap, d), generator=g).to(torch.bfloat16)
    q = torch.randn((B, Hkv * G, d), generator=g).to(torch.bfloat16)
    Kc[:, :, length:] = float("inf")
    Vc[:, :, length:] = float("inf")
    Kd, Vd = Kc.to(DEV), Vc.to(DEV)
    p = lrsa.make_params((B, Hkv * G, cap, d), tuple(Kc.shape), (Hkv * G * cap * d, cap * d, d, 1), Kd.stride(),
                         dtype=torch.bfloat16, sink=4, lag=16, topk=4)
    O, lse = lrsa.lrsa_decode_attn(p, q.to(DEV), Kd, Vd, length)
    O, lse = O.double().cpu().numpy(), lse.cpu().numpy()
    for b in range(B):
        for h in range(Hkv):
            sl = slice(h * G, (h + 1) * G)
            O_ref, lse_ref = dec.decode_attn(q[b, sl].float().numpy(), Kc[b, h, :length].float().numpy(), Vc[b, h, :length].float().numpy())
            # the rounding of the output (8 significant bits: half a unit is up to 2^-8 of the value) and fp32 logits of magnitude
            # up to |lse| (weights off by 2^-20 of that each)
            bound = 2.0 ** -8 * np.abs(O_ref) + 2.0 ** -20 * max(np.abs(lse_ref).max(), 8.0) * np.abs(Vc[b, h, :length].float().numpy()).max()
            assert np.all(np.abs(O[b, sl] - O_ref) <= bound)
            assert np.all(np.abs(lse[b, sl] - lse_ref) <= 2.0 ** -20 * np.maximum(np.abs(lse_ref), 8.0))


# Slices per (batch, KV head): up to 256, four per lane of the merge; few heads and long caches take them all.  fp32: both rules for
# the number of slices (84 units of four heads and more keep fewer).
@pytest.mark.parametrize("dtype,B,Hkv,G,d,length,slices", [
    ("bf16", 1, 1, 1, 128, 128 * 256 + 5, 256), ("bf16", 1, 1, 4, 64, 128 * 200 + 77, 201), ("bf16", 1, 4, 3, 128, 128 * 128 + 1, 128),
    ("bf16", 1, 2, 2, 64, 128 * 65, 65), ("bf16", 1, 1, 2, 128, 40000, 256), ("f32", 1, 1, 1, 64, 128 * 256 + 5, 256),
    ("f32", 1, 1, 9, 128, 128 * 190 + 3, 191), ("f32", 1, 2, 2, 128, 128 * 66 + 100, 67), ("f32", 2, 2, 4, 64, 3000, 24),
    ("f32", 11, 8, 4, 64, 1500, 6), ("f32", 10, 8, 4, 64, 1500, 6), ("f32", 33, 4, 3, 64, 1100, 4), ("f32", 3, 4, 8, 128, 129, 2),
])
def test_decode_attention_over_many_slices(dtype, B, Hkv, G, d, length, slices):
    cap = length + 3
    g = torch.Generator(device=DEV).manual_seed(length + G)
    T = {"bf16": torch.bfloat16, "f32": torch.float32}[dtype]
    # K grows along the cache: the slices' maxima differ, and the last ones do not hold all of the weight
    Kc = (torch.randn((B, Hkv, cap, d), generator=g, device=DEV) * torch.linspace(0.5, 1.5, cap, device=DEV)[:, None]).to(T)
    Vc = torch.randn((B, Hkv, cap, d), generator=g, device=DEV).to(T)
    q = torch.randn((B, Hkv * G, d), generator=g, device=DEV).to(T)
    p = lrsa.make_params((B, Hkv * G, cap, d), tuple(Kc.shape), (Hkv * G * cap * d, cap * d, d, 1), Kc.stride(), dtype=T, sink=4, lag=16, topk=4)
    ws = torch.full((lrsa.workspace_bytes(p, lrsa.binding.WS_DECODE_ATTN) // 4,), float("nan"), device=DEV)
    O, lse = lrsa.lrsa_decode_attn(p, q, Kc, Vc, length, ws=ws)
    torch.cuda.synchronize()
    # the records of the slices, as many as the case is meant for, fill the front of the workspace
    assert int((~ws.isnan()).sum()) == B * Hkv * G * slices * (d + 2)
    K64, V64 = (t[:, :, :length].double().cpu().numpy() for t in (Kc, Vc))
    for b in sorted({0, B - 1}):
        for h in sorted({0, Hkv - 1}):
            sl = slice(h * G, (h + 1) * G)
            O_ref, lse_ref = dec.decode_attn(q[b, sl].double().cpu().numpy(), K64[b, h], V64[b, h])
            # fp32 logits of magnitude up to |lse| (weights off by 2^-20 of that each), and the rounding of a bf16 output
            bound = 2.0 ** -20 * max(np.abs(lse_ref).max(), 8.0) * np.abs(V64[b, h]).max() + (2.0 ** -8 * np.abs(O_ref) if dtype == "bf16" else 0.0)
            assert np.all(np.abs(O[b, sl].double().cpu().numpy() - O_ref) <= bound)
            assert np.all(np.abs(lse[b, sl].cpu().numpy() - lse_ref) <= 2.0 ** -20 * np.maximum(np.abs(lse_ref), 8.0))
