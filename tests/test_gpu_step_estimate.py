"""Estimate of short steps deep in a context (one sweep over the key strides, softmax and selection in a second launch): block masses
against the method in 64 bits, the selection against those masses, the row order against the one made from the finished mask.
Masses are sums of at most some thousand fp32 terms of exact products: 2^-24 times the logits' spread (below 64) and the
additions' depth, within 1e-5 of the row."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


def _masses(Q, K, S, B, q0):
    """[Hq, rows, Nb] in 64 bits: fractions of a row; rows without a sampled query are 0"""
    _, Hq, Lq, d = Q.shape
    Hkv, L = K.shape[1], K.shape[2]
    Ls, R, Nb = L // S, B // S, -(-L // B)
    m0 = q0 // B
    sums = K[0, :, :Ls * S].double().reshape(Hkv, Ls, S, d).sum(2)
    out = torch.zeros(Hq, Nb - m0, Nb, dtype=torch.float64, device=Q.device)
    for h in range(Hq):
        for i in range(q0 // S, Ls):
            p = i * S + S - 1 - h % S - q0
            if p < 0:
                continue
            w = torch.softmax(sums[h // (Hq // Hkv), :i + 1] @ Q[0, h, p].double() / (S * math.sqrt(d)), 0)
            out[h, i // R - m0].index_add_(0, torch.arange(i + 1, device=Q.device) // R, w)
    return out / out.sum(2, keepdim=True).clamp_min(1e-300)


@pytest.mark.parametrize("Hq,Hkv,L,Lq,S", [(8, 2, 128 * 300, 8, 16), (4, 4, 128 * 257 - 19, 1, 16), (8, 1, 128 * 1024, 3, 16),
                                           (14, 2, 128 * 600 + 3, 30, 16), (8, 2, 128 * 130 + 40, 50, 8), (32, 8, 128 * 66 + 1, 5, 4),
                                           (8, 2, 128 * 512, 100, 32), (4, 1, 128 * 400 + 20, 16, 16), (4, 1, 128 * 400 + 20, 4, 16)])
@pytest.mark.parametrize("tau", [0.9])
def test_step_estimate(Hq, Hkv, L, Lq, S, tau):
    import paper_2602_05853_amd as rr
    B, dev = 128, "cuda:0"
    g = torch.Generator(device=dev).manual_seed(L + Lq)
    K = torch.randn(1, Hkv, L, 128, generator=g, device=dev)
    K = (K + 2.0 * torch.randn(1, Hkv, -(-L // 512), 128, generator=g, device=dev).repeat_interleave(512, 2)[:, :, :L]).bfloat16()
    Q = (2.0 * torch.randn(1, Hq, Lq, 128, generator=g, device=dev)).bfloat16()
    print(f"[step] {Hq}/{Hkv} heads, {Lq} of {L}, S {S}", flush=True)
    mask = rr.rr_estimate(Q, K, S, B, tau, flags=0, block_mass=True)
    torch.cuda.synchronize()
    ref, q0 = _masses(Q, K, S, B, L - Lq), L - Lq
    got = mask.block_mass[0].double()
    assert (got - ref).abs().max() <= 1e-5
    sampled = ref.sum(2) > 0.5
    rows = ref.shape[1]
    causal = torch.arange(ref.shape[2], device=dev)[None] <= (q0 // B + torch.arange(rows, device=dev))[:, None]
    kept = mask.dense[0].bool()
    assert not (kept & ~causal).any()
    assert torch.equal(kept[~sampled], causal.expand(Hq, -1, -1)[~sampled])
    for h, r in sampled.nonzero().tolist():
        a, b = got[h, r][kept[h, r]], got[h, r][~kept[h, r]]
        assert a.sum() >= tau - 1e-5 and (a.sum() - a.min() < tau + 1e-5) and (b.numel() == 0 or b.max() <= a.min())
        n = int(mask.row_count[0, h, r])
        assert torch.equal(mask.row_list[0, h, r, :n].long(), kept[h, r].nonzero().flatten())
    again = rr.rr_mask_from_dense(Q, K, mask.dense, B)
    assert torch.equal(again.row_order, mask.row_order) and not mask.queue.any()
