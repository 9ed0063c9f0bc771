"""Estimate of short steps deep in a context (one sweep over the key strides, softmax and selection in a second launch): block masses
against the method in 64 bits, the selection against those masses, the row order against the one made from the finished mask.
Masses are sums of at most some thousand fp32 terms of exact products: 2^-24 times the logits' spread (below 64) and the
additions' depth, within 1e-5 of the row."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

B = 128


def _context(batch, Hq, Hkv, L, Lq, seed):
    g = torch.Generator(device="cuda:0").manual_seed(seed)
    K = torch.randn(batch, Hkv, L, 128, generator=g, device="cuda:0")
    K = (K + 2.0 * torch.randn(batch, Hkv, -(-L // 512), 128, generator=g, device="cuda:0").repeat_interleave(512, 2)[:, :, :L]).bfloat16()
    return (2.0 * torch.randn(batch, Hq, Lq, 128, generator=g, device="cuda:0")).bfloat16(), K


def _dirty(Q, K, S, batch, Hq, Hkv, L, Lq):
    """a workspace of set bytes and a mask whose every array holds garbage"""
    import paper_2602_05853_amd as rr
    ws = torch.full((rr.rr_workspace_bytes(Q, K, S, B),), 0xFF, dtype=torch.uint8, device=Q.device)
    Nb = -(-L // B)
    out = rr.BlockMask.allocate(batch, Hq, Nb, B, Q.device, block_mass=True, Hkv=Hkv, rows=Nb - (L - Lq) // B)
    for t in (out.row_count, out.row_list, out.row_order, out.queue):
        t.fill_(0x7A7A7A7A)
    out.dense.fill_(0x7A)
    out.block_mass.fill_(float("nan"))
    return ws, out


def _one_sweep(ws):
    """two sweeps leave the softmax states of their last key chunk in the last 2 KB, the forms of short steps and contexts nothing"""
    return bool((ws[-2048:] == 0xFF).all())


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


# A block that holds several sampled queries of a head, one of them not finite: the row's mass is unknown, so it keeps every block, in
# every form of the estimate (`sweeps`: False for the short steps of this file and for a short context in one launch); rows of
# other heads and blocks are what they are without it.
@pytest.mark.parametrize("Hq,Hkv,L,Lq,S,sweeps", [(8, 2, 128 * 1024, 12, 4, False), (16, 8, 128 * 700 + 64, 80, 16, False),
                                                  (8, 2, 128 * 300 + 24, 24, 8, False), (8, 2, 128 * 513, 64, 32, False),
                                                  (8, 2, 128 * 60, 130, 16, False), (8, 2, 128 * 140, 300, 16, True)])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_row_with_a_query_that_is_not_finite_keeps_every_block(Hq, Hkv, L, Lq, S, sweeps, value):
    import paper_2602_05853_amd as rr
    Q, K = _context(1, Hq, Hkv, L, Lq, L + Lq)
    q0, m0, h = L - Lq, (L - Lq) // B, Hq - 2
    clean = rr.rr_estimate(Q, K, S, B, 0.9, flags=0, block_mass=True)
    position = lambda i: i * S + S - 1 - h % S - q0                                 # of the sampled query of stride i, in the step
    held = [i for i in range(q0 // S, L // S) if position(i) >= 0]
    row = lambda i: i * S // B - m0
    r = row(held[-1])
    assert sum(row(i) == r for i in held) >= 2 and int(clean.row_count[0, h, r]) < m0 + r + 1
    Q[0, h, position(held[-1]), 17] = value
    ws, mask = _dirty(Q, K, S, 1, Hq, Hkv, L, Lq)
    print(f"[step] {Hq}/{Hkv} heads, {Lq} of {L}, S {S}: query {value} in row {r} of head {h}", flush=True)
    rr.rr_estimate(Q, K, S, B, 0.9, flags=0, out=mask, workspace=ws)
    torch.cuda.synchronize()
    assert _one_sweep(ws) != sweeps
    n = torch.arange(mask.Nb, device="cuda:0")
    assert torch.equal(mask.dense[0, h, r].bool(), n <= m0 + r) and int(mask.row_count[0, h, r]) == m0 + r + 1
    others = torch.ones(mask.row_count.shape, dtype=torch.bool, device="cuda:0")
    others[0, h, r] = False
    for a, b in ((mask.dense, clean.dense), (mask.row_count, clean.row_count), (mask.block_mass, clean.block_mass)):
        assert torch.equal(a[others], b[others])
