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


# The same call with one query far: what every other row holds is what it holds without it, bit for bit.
@pytest.mark.parametrize("L,Lq,Hq,Hkv,S", [(2048, 2048, 8, 2, 16), (16000, 16000, 4, 1, 16), (2500, 2500, 4, 2, 4), (64512, 40, 8, 2, 16), (65536, 64, 8, 2, 32)])
@pytest.mark.parametrize("value", [1e12, float("inf")])
def test_other_rows_stay_as_they_are(L, Lq, Hq, Hkv, S, value):
    import paper_2602_05853_amd as rr
    g = torch.Generator(device="cuda:0").manual_seed(L)
    Q = (2 * torch.randn(1, Hq, Lq, 128, generator=g, device="cuda:0")).bfloat16()
    K = torch.randn(1, Hkv, L, 128, generator=g, device="cuda:0").bfloat16()
    clean = rr.rr_estimate(Q, K, S, B, 0.9, flags=0, block_mass=True)
    h, i = 1, L // S - 1
    p = i * S + S - 1 - h % S
    Q[0, h, p - (L - Lq), 3] = value
    print(f"[far] {Lq} of {L}, {Hq}/{Hkv} heads, S {S}, a query of {value}", flush=True)
    mask = rr.rr_estimate(Q, K, S, B, 0.9, flags=0, block_mass=True)
    torch.cuda.synchronize()
    others = torch.ones(mask.row_count.shape, dtype=torch.bool, device="cuda:0")
    others[0, h, p // B - (L - Lq) // B] = False
    for a, b in ((mask.dense, clean.dense), (mask.row_count, clean.row_count), (mask.block_mass, clean.block_mass)):
        assert torch.equal(a[others], b[others])
