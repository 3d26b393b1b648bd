"""lrsa_cache_compress with a workspace (what the binding calls: all steps of a call at once, over many workgroups)
against the one-workgroup-per-head steps of the call without one, and against the oracle's token-by-token procedure.

Bar: bit-identical cache, positions and counts -- rows are chosen by the same scores (the same additions in the same
order) and moved, never computed; bytes outside the rows of the new cache that the old call leaves alone stay alone.
"""
import ctypes

import numpy as np
import pytest
import torch

import paper_2506_11498_amd as lrsa
from oracle import lrsa_decode as dec

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _vp(t):
    return None if t is None else ctypes.c_void_p(t.data_ptr())


def _without_ws(p, Kc, Vc, pos, length, done):
    a, b = ctypes.c_int32(0), ctypes.c_int32(0)
    rc = lrsa.lib().lrsa_cache_compress(ctypes.byref(p), _vp(Kc), _vp(Vc), _vp(pos), length, done, ctypes.byref(a), ctypes.byref(b),
                                        ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0, lrsa.lib().lrsa_last_error()
    return a.value, b.value


# steps > 1 with a rest longer and shorter than the shift (through the workspace or straight), ragged lags, keep one and
# keep all, lags below a slice and the largest, several chunks compressed before, both types and head dimensions
@pytest.mark.parametrize("B,Hkv,d,L,K,S,done,chunks,rest,dtype,pos", [
    (1, 2, 128, 64, 16, 4, 0, 2, 0, "bf16", True),
    (2, 2, 128, 64, 60, 0, 0, 6, 63, "bf16", True),
    (1, 1, 128, 100, 37, 5, 3, 2, 17, "bf16", False),
    (1, 3, 128, 1024, 256, 64, 2, 2, 0, "bf16", False),
    (1, 2, 128, 1024, 512, 64, 0, 9, 777, "bf16", True),
    (1, 1, 128, 4096, 1, 0, 0, 3, 5, "bf16", True),
    (1, 1, 128, 300, 299, 7, 1, 4, 299, "bf16", True),
    (1, 2, 64, 16, 4, 3, 0, 5, 7, "f32", True),
    (2, 1, 128, 24, 24, 0, 0, 4, 1, "f32", True),
    (1, 2, 128, 200, 199, 1, 0, 3, 199, "f32", True),
    (1, 2, 64, 333, 100, 8, 0, 7, 11, "bf16", True),
])
def test_all_steps_at_once_equal_the_steps_one_by_one(B, Hkv, d, L, K, S, done, chunks, rest, dtype, pos):
    dt = {"bf16": torch.bfloat16, "f32": torch.float32}[dtype]
    length = S + K * done + chunks * L + rest
    cap = length + 9
    g = torch.Generator(device=DEV).manual_seed(L * 7 + K)
    Kc, Vc = (torch.randn((B, cap, Hkv, d), generator=g, device=DEV).to(dt).permute(0, 2, 1, 3) for _ in range(2))  # strided rows
    P = torch.arange(B * Hkv * cap, dtype=torch.int32, device=DEV).reshape(B, Hkv, cap) if pos else None
    p = lrsa.make_params((B, Hkv, cap, d), (B, Hkv, cap, d), Kc.stride(), Kc.stride(), dtype=dt, sink=S, lag=L, topk=K)
    want = [t.clone(memory_format=torch.preserve_format) if t is not None else None for t in (Kc, Vc, P)]
    counts = _without_ws(p, *want, length, done)
    assert lrsa.lrsa_cache_compress(p, Kc, Vc, P, length, done) == counts
    torch.cuda.synchronize()
    new = counts[0]
    assert counts[1] == done + chunks - 1
    for got, ref in zip((Kc, Vc, P), want):
        if ref is not None:
            assert torch.equal(got[:, :, :new], ref[:, :, :new])
            assert torch.equal(got[:, :, length:], ref[:, :, length:])


# one step on both sides of the line that its route is chosen by: chunks of 64 KB (32 heads of K, bf16), 256 KB (64 heads), 128
# KB per 256 workgroups (fp32), never more than 64 heads; ragged lags, a rest longer and shorter than the shift
@pytest.mark.parametrize("B,Hkv,d,L,K,S,done,rest,dtype,long", [
    (2, 16, 128, 256, 100, 5, 1, 255, "bf16", True),
    (2, 16, 128, 255, 100, 5, 1, 3, "bf16", False),
    (3, 1, 64, 513, 512, 0, 2, 511, "bf16", True),
    (11, 3, 128, 1023, 17, 3, 0, 0, "bf16", False),
    (11, 3, 128, 1024, 17, 3, 0, 9, "bf16", True),
    (5, 13, 64, 2048, 1000, 1, 0, 1, "bf16", False),
    (1, 1, 128, 4096, 4095, 64, 1, 4000, "bf16", True),
    (2, 8, 128, 257, 1, 7, 3, 250, "f32", True),
    (2, 8, 128, 255, 1, 7, 3, 250, "f32", False),
    (1, 17, 128, 511, 200, 0, 0, 33, "f32", False),
    (1, 17, 128, 515, 200, 0, 0, 33, "f32", True),
    (1, 3, 64, 600, 599, 2, 1, 0, "f32", True),
])
def test_one_step_by_either_route(B, Hkv, d, L, K, S, done, rest, dtype, long):
    dt = {"bf16": torch.bfloat16, "f32": torch.float32}[dtype]
    length = S + K * done + 2 * L + rest
    cap = length + 3
    g = torch.Generator(device=DEV).manual_seed(L * 5 + K)
    Kc, Vc = (torch.randn((B, cap, Hkv, d), generator=g, device=DEV).to(dt).permute(0, 2, 1, 3) for _ in range(2))
    P = torch.arange(B * Hkv * cap, dtype=torch.int32, device=DEV).reshape(B, Hkv, cap)
    p = lrsa.make_params((B, Hkv, cap, d), (B, Hkv, cap, d), Kc.stride(), Kc.stride(), dtype=dt, sink=S, lag=L, topk=K)
    assert (lrsa.cache_compress_ws_bytes(p, length, done) > 0) == long
    want = [t.clone(memory_format=torch.preserve_format) for t in (Kc, Vc, P)]
    counts = _without_ws(p, *want, length, done)
    assert lrsa.lrsa_cache_compress(p, Kc, Vc, P, length, done) == counts == (length - (L - K), done + 1)
    torch.cuda.synchronize()
    for got, ref in zip((Kc, Vc, P), want):
        assert torch.equal(got[:, :, :counts[0]], ref[:, :, :counts[0]])
        assert torch.equal(got[:, :, length:], ref[:, :, length:])


def test_a_whole_prompt_equals_the_token_by_token_procedure():
    B, Hkv, d, L, K, S, n = 1, 2, 128, 64, 16, 8, 8 + 9 * 64 + 30
    g = torch.Generator().manual_seed(3)
    K0, V0 = (torch.randn((B, Hkv, n, d), generator=g).to(torch.bfloat16) for _ in range(2))
    Kc, Vc = K0.to(DEV), V0.to(DEV)
    pos = torch.arange(n, dtype=torch.int32, device=DEV).expand(B, Hkv, n).contiguous()
    p = lrsa.make_params((B, Hkv, n, d), (B, Hkv, n, d), Kc.stride(), Kc.stride(), dtype=torch.bfloat16, sink=S, lag=L, topk=K)
    length, done = lrsa.lrsa_cache_compress(p, Kc, Vc, pos, n, 0)
    for h in range(Hkv):
        Ko, Vo, po, do = dec.cache_incremental(K0[0, h].float().numpy(), V0[0, h].float().numpy(), S, L, K)
        # the procedure compresses only when a further token arrives: n leaves a tail of L + 30 rows either way
        assert (length, done) == (len(po), do)
        assert np.array_equal(pos[0, h, :length].cpu().numpy(), po)
        assert np.array_equal(Kc[0, h, :length].float().cpu().numpy(), Ko)
        assert np.array_equal(Vc[0, h, :length].float().cpu().numpy(), Vo)


def _prompt():
    B, Hkv, d, L, K, S, n = 1, 2, 128, 64, 16, 8, 8 + 5 * 64 + 7
    g = torch.Generator().manual_seed(4)
    Kc, Vc = (torch.randn((B, Hkv, n, d), generator=g).to(torch.bfloat16).to(DEV) for _ in range(2))
    pos = torch.arange(n, dtype=torch.int32, device=DEV).expand(B, Hkv, n).contiguous()
    p = lrsa.make_params((B, Hkv, n, d), (B, Hkv, n, d), Kc.stride(), Kc.stride(), dtype=torch.bfloat16, sink=S, lag=L, topk=K)
    return p, (Kc, Vc, pos), n


def test_under_graph_capture_nothing_is_allocated():
    """A workspace from torch's allocator would not be held until the replays: without one of the caller's, the steps are
    recorded that need none.  Every replay, with eager work in between, equals the eager call."""
    p, start, n = _prompt()
    want = [t.clone() for t in start]
    counts = lrsa.lrsa_cache_compress(p, *want, n, 0)
    for own_ws in (False, True):
        ws = torch.empty(lrsa.cache_compress_ws_bytes(p, n, 0), dtype=torch.uint8, device=DEV) if own_ws else None
        bufs = [t.clone() for t in start]
        lrsa.lrsa_cache_compress(p, *bufs, n, 0, ws)                  # everything is loaded before the capture
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            before = torch.cuda.memory_stats()["allocation.all.allocated"]
            assert lrsa.lrsa_cache_compress(p, *bufs, n, 0, ws) == counts
            assert torch.cuda.memory_stats()["allocation.all.allocated"] == before
        for _ in range(3):
            for b, t in zip(bufs, start):
                b.copy_(t)
            torch.empty(1 << 20, device=DEV).normal_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            for b, r in zip(bufs, want):
                assert torch.equal(b[:, :, :counts[0]], r[:, :, :counts[0]])


def test_without_memory_for_a_workspace_the_call_still_runs(monkeypatch):
    p, start, n = _prompt()
    want = [t.clone() for t in start]
    counts = lrsa.lrsa_cache_compress(p, *want, n, 0)

    def no_memory(*a, **k):
        raise torch.OutOfMemoryError("out of memory")
    monkeypatch.setattr(torch, "empty", no_memory)
    assert lrsa.lrsa_cache_compress(p, *start, n, 0) == counts
    monkeypatch.undo()
    for b, r in zip(start, want):
        assert torch.equal(b[:, :, :counts[0]], r[:, :, :counts[0]])


def test_missing_buffers_and_short_workspaces_are_reported_by_the_library():
    p, (Kc, Vc, pos), n = _prompt()
    for K, V in ((None, Vc), (Kc, None), (None, None)):
        with pytest.raises(lrsa.LrsaError, match="NULL"):
            lrsa.lrsa_cache_compress(p, K, V, pos, n, 0)
    with pytest.raises(lrsa.LrsaError, match="workspace"):
        lrsa.lrsa_cache_compress(p, Kc, Vc, pos, n, 0, torch.empty(256, dtype=torch.uint8, device=DEV))
