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
