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
