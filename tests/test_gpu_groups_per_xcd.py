"""Launches whose XCDs take the rows of KV groups of their own: rows drawn from one queue per group or per eight (sparse calls of eight
rows and more to a workgroup, four where a queue has several groups), and dense calls.  The same per-row arithmetic as a workgroup
per row in another order, so results are equal bit for bit and every row is computed."""
import dataclasses

import pytest
import torch

pytestmark = pytest.mark.gpu


def _tensors(batch, L, Hq, Hkv):
    dev, d = "cuda:0", 128
    g = torch.Generator(device=dev).manual_seed(L + 10 * Hq + batch)
    Q = torch.randn(batch, Hq, L, d, generator=g, device=dev).bfloat16()
    K, V = (torch.randn(batch, Hkv, L, d, generator=g, device=dev).bfloat16() for _ in range(2))
    # groups whose rows keep very different numbers of blocks: the queues run empty one after the other
    u = torch.randn(d, generator=g, device=dev)
    scale = torch.linspace(0.0, 1.0, batch * Hkv, device=dev).view(batch, Hkv, 1, 1)
    K[:, :, : L // 8] += (scale * u).bfloat16()
    Q += (scale.repeat_interleave(Hq // Hkv, 1) * u).bfloat16()
    return Q, K, V


# one group to all XCDs, two, three (XCDs 0 and 1 have three each), seven, eight, nine (queue 0 has two groups), sixteen; rows of
# eight waves beyond 256 blocks; lengths that end inside a block; fewer rows than the rule asks for
@pytest.mark.parametrize("batch,L,Hq,Hkv", [(1, 16384, 32, 1), (1, 16300, 34, 2), (1, 16384, 33, 3), (1, 16000, 35, 7), (1, 16384, 32, 8),
                                            (3, 16384, 6, 3), (2, 8100, 32, 8), (1, 33000, 8, 2), (1, 16256, 32, 8)])
def test_rows_by_group_equal_rows_one_by_one(batch, L, Hq, Hkv):
    import paper_2602_05853_amd as rr
    Q, K, V = _tensors(batch, L, Hq, Hkv)
    mask = rr.rr_estimate(Q, K, 16, 128, 0.7)
    print(f"[groups] {batch} x {Hq}/{Hkv} heads, {L} tokens, blocks to a group {mask.row_count.view(batch * Hkv, -1).sum(1).tolist()}", flush=True)
    ref = rr.rr_sparse_attn(Q, K, V, dataclasses.replace(mask, queue=None))
    for rep in range(3):
        O = torch.full_like(Q, float("nan"))
        rr.rr_sparse_attn(Q, K, V, mask, O=O)
        torch.cuda.synchronize()
        assert int(mask.queue.abs().max()) == 0, rep
        assert torch.equal(O, ref), rep


@pytest.mark.parametrize("batch,L,Hq,Hkv", [(1, 2048, 8, 1), (1, 2048, 6, 2), (1, 1500, 12, 4), (1, 2048, 16, 8), (2, 1000, 8, 8), (1, 1024, 6, 3), (3, 1024, 4, 4)])
def test_dense_rows_by_group_are_all_computed(batch, L, Hq, Hkv):
    """Against a list of every block in a launch order of its own."""
    import paper_2602_05853_amd as rr
    Q, K, V = _tensors(batch, L, Hq, Hkv)
    Nb = -(-L // 128)
    mask = rr.rr_mask_from_dense(Q, K, torch.ones(batch, Hq, Nb, Nb, dtype=torch.uint8, device=Q.device).tril(), 128)
    ref = rr.rr_sparse_attn(Q, K, V, mask)
    O = torch.full_like(Q, float("nan"))
    rr.rr_dense_attn(Q, K, V, 128, O=O)
    torch.cuda.synchronize()
    assert torch.equal(O, ref)
