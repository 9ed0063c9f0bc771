"""The two forms of a row in the bf16 d = 128 attention kernel, four waves or eight, on both sides of the rule that chooses
by rows and context length (eight waves up to 15 rows per key block and 64; the last two calls have more).  Rows of
every small count, the diagonal block alone, without it, empty rows, lengths that end inside a block and steps that
start inside one, dense and under lists, with and without the queue, against attention in fp32 with P unrounded.

Bound: P is rounded by at most 2^-8 and so is O, a convex combination of the values: 2^-7 max|V|, plus fp32 sums; the
log-sum-exp is that of a sum of rounded terms, log(1 + 2^-8) at most."""
import dataclasses

import pytest
import torch

pytestmark = pytest.mark.gpu


def _attention(Q, K, V, keep):
    s = (Q.float() @ K.float().T / 128 ** 0.5).masked_fill(~keep, float("-inf"))
    lse = torch.logsumexp(s, 1)
    p = torch.exp(s - lse.nan_to_num(neginf=0.0)[:, None])
    return p @ V.float(), lse


@pytest.mark.parametrize("Hq,Hkv,L,Lq", [(2, 1, 128 * 9, 128 * 9), (6, 3, 128 * 37 - 41, 128 * 37 - 41), (12, 2, 128 * 24, 128 * 24),
                                         (8, 8, 128 * 33 + 1, 700), (4, 2, 128 * 40 - 3, 1), (8, 2, 128 * 70, 128 * 70),
                                         (32, 8, 128 * 40, 128 * 40), (64, 8, 128 * 16 - 5, 128 * 16 - 5)])
def test_rows_of_four_and_of_eight_waves(Hq, Hkv, L, Lq):
    import paper_2602_05853_amd as rr
    dev, B = "cuda:0", 128
    g = torch.Generator(device=dev).manual_seed(L + Hq)
    Q, K, V = (torch.randn(1, h, n, 128, generator=g, device=dev).bfloat16() for h, n in ((Hq, Lq), (Hkv, L), (Hkv, L)))
    Q, K = Q * 1.5, K                                       # (a few large weights)
    Nb, q0 = -(-L // B), L - Lq
    rows = Nb - q0 // B
    m = torch.arange(Nb - rows, Nb, device=dev)[:, None]
    n = torch.arange(Nb, device=dev)[None]
    dense = (torch.rand(1, Hq, rows, Nb, generator=g, device=dev) < 0.3)
    dense[0, 0] |= n == m
    dense[0, 1] &= n != m                                   # never the diagonal block
    if Hq > 2:
        dense[0, 2] = n == m
        dense[0, 2, ::2] = False                            # empty rows
    dense[0, Hq - 1, rows - 1] = True                       # a row of every block
    dense = (dense & (n <= m)).to(torch.uint8)
    mask = rr.rr_mask_from_dense(Q, K, dense, B)
    qpos, kpos = torch.arange(q0, L, device=dev), torch.arange(L, device=dev)
    causal = kpos[None] <= qpos[:, None]
    bound = 2.0 ** -7 * V.abs().max().item() + 1e-5
    print(f"[wide] {Hq}/{Hkv} heads, {Lq} of {L}: {Hq * rows} rows of up to {Nb} blocks", flush=True)
    for what in ("queue", "no queue", "dense"):
        O = torch.full_like(Q, float("nan"))
        lse = torch.full(Q.shape[:3], float("nan"), dtype=torch.float32, device=dev)
        if what == "dense":
            rr.rr_dense_attn(Q, K, V, B, O=O, lse=lse)
        else:
            rr.rr_sparse_attn(Q, K, V, mask if what == "queue" else dataclasses.replace(mask, queue=None), O=O, lse=lse)
        torch.cuda.synchronize()
        assert int(mask.queue.abs().sum().item()) == 0
        for h in sorted({0, 1, 2 % Hq, Hq // 2, Hq - 1}):
            keep = causal
            if what != "dense":
                keep = causal & dense[0, h].bool()[qpos // B - q0 // B][:, kpos // B]
            want, want_lse = _attention(Q[0, h], K[0, h // (Hq // Hkv)], V[0, h // (Hq // Hkv)], keep)
            assert (O[0, h].float() - want).abs().max().item() <= bound, (what, h)
            empty = torch.isinf(want_lse)
            assert torch.equal(torch.isneginf(lse[0, h]), empty) and not O[0, h][empty].any()
            off = (lse[0, h] - want_lse)[~empty].abs()
            assert off.numel() == 0 or off.max().item() <= 2.0 ** -8 + 1e-5, (what, h)


@pytest.mark.parametrize("Hq,Hkv,L,Lq", [(8, 2, 128 * 34 - 20, 60), (8, 8, 128 * 300, 100), (9, 9, 128 * 300 - 7, 100),
                                         (2, 1, 128 * 17, 128), (3, 1, 128 * 60 - 50, 40)])
def test_equal_parts_of_four_and_of_eight_waves(Hq, Hkv, L, Lq):
    """Split launches of up to 256 parts (eight waves) and of more (288, four): rows of no entry, of the diagonal block
    alone, of fewer entries than parts, without the diagonal block, and of every block.  The parts are merged in fp32 from
    sums that round P as above; the log-sum-exp of each is off by log(1 + 2^-8) at most."""
    import paper_2602_05853_amd as rr
    dev, B = "cuda:0", 128
    g = torch.Generator(device=dev).manual_seed(L + Hq)
    Q, K, V = (torch.randn(1, h, n, 128, generator=g, device=dev).bfloat16() for h, n in ((Hq, Lq), (Hkv, L), (Hkv, L)))
    Q = Q * 1.5
    Nb, q0 = -(-L // B), L - Lq
    rows = Nb - q0 // B
    assert rows == 1 and Hq // Hkv * Lq > 32                # neither a planned launch nor the decode kernel
    m = Nb - 1
    dense = (torch.rand(1, Hq, rows, Nb, generator=g, device=dev) < 0.3).to(torch.uint8)
    for h, cols in enumerate(([], [m], [0, m], [1, 5], range(Nb), [m - 1], range(0, Nb - 1), [0])[:Hq]):
        dense[0, h] = 0
        dense[0, h, 0, list(cols)] = 1
    mask = rr.rr_mask_from_dense(Q, K, dense, B)
    ws = torch.full((rr.rr_attn_workspace_bytes(Q, K, B),), 0xFF, dtype=torch.uint8, device=dev)
    assert ws.numel() > 0
    kpos = torch.arange(L, device=dev)
    causal = kpos[None] <= torch.arange(q0, L, device=dev)[:, None]
    bound = 2.0 ** -7 * V.abs().max().item() + 1e-5
    print(f"[parts] {Hq}/{Hkv} heads, {Lq} of {L}", flush=True)
    for what in ("sparse", "dense"):
        O = torch.full_like(Q, float("nan"))
        lse = torch.full(Q.shape[:3], float("nan"), dtype=torch.float32, device=dev)
        if what == "dense":
            rr.rr_dense_attn(Q, K, V, B, O=O, lse=lse, workspace=ws)
        else:
            rr.rr_sparse_attn(Q, K, V, mask, O=O, lse=lse, workspace=ws)
        torch.cuda.synchronize()
        for h in range(Hq):
            keep = causal
            if what == "sparse":
                keep = causal & dense[0, h, 0].bool().repeat_interleave(B)[:L][None]
            want, want_lse = _attention(Q[0, h], K[0, h // (Hq // Hkv)], V[0, h // (Hq // Hkv)], keep)
            empty = torch.isinf(want_lse)
            assert torch.equal(torch.isinf(lse[0, h]), empty), (what, h)
            assert not empty.any() or O[0, h][empty].abs().max() == 0
            if (~empty).any():
                assert (O[0, h].float() - want)[~empty].abs().max() <= bound, (what, h)
                assert (lse[0, h] - want_lse)[~empty].abs().max() <= 2.0 ** -8, (what, h)
