"""Finite scores far beyond what an exponent holds, in the forms of the estimate that normalise without a second sweep (short contexts in
one launch, short steps): one key of 1e12 and more gives a query all of its mass or none of it, by the sign of its channel, and
no rounding of a product that size may make it, or its stride, drop out."""
import pytest
import torch

import gpu_util as gu

pytestmark = pytest.mark.gpu

B = 128


# R = 128 / S; one to four tiles to a wavefront of the first form, unprotected steps that take it, and steps beyond 1024 strides
@pytest.mark.parametrize("L,Lq,Hq,Hkv,S", [(2048, 2048, 8, 2, 16), (16000, 16000, 4, 1, 16), (4000, 4000, 4, 2, 8), (20000, 20000, 2, 1, 32),
                                           (2500, 2500, 4, 2, 4), (16000, 40, 8, 2, 16), (64512, 40, 8, 2, 16), (40000, 8, 8, 2, 8),
                                           (65536, 64, 8, 2, 32), (128 * 140 + 2, 9, 8, 2, 4)])
@pytest.mark.parametrize("value", [1e7, 1e12, 1e30, -1e36])
def test_one_key_beyond_all_others(L, Lq, Hq, Hkv, S, value):
    import paper_2602_05853_amd as rr
    q0, m0 = L - Lq, (L - Lq) // B
    g = torch.Generator(device="cuda:0").manual_seed(L)
    Q = (2 * torch.randn(1, Hq, Lq, 128, generator=g, device="cuda:0")).bfloat16()
    K = torch.randn(1, Hkv, L, 128, generator=g, device="cuda:0").bfloat16()
    for kv in range(Hkv):
        K[0, kv, L // 3 + 211 * kv, 19 + kv] = value
    print(f"[far] {Lq} of {L}, {Hq}/{Hkv} heads, S {S}, a key of {value}", flush=True)
    mask = rr.rr_estimate(Q, K, S, B, 0.9, flags=0, block_mass=True)
    torch.cuda.synchronize()
    for h in range(Hq):
        ref = gu.stride_masses(Q[0, h], K[0, h // (Hq // Hkv)], S, B, q0, h)
        assert (mask.block_mass[0, h].double() - ref).abs().max() <= 1e-5, h
        # blocks left out of a row hold less than a tenth of it
        assert not ((ref > 0.1 + 1e-5) & (mask.dense[0, h] == 0)).any(), h
