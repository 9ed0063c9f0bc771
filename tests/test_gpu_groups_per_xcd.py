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


def _by_group(batch, L, Hq, Hkv):
    """Whether a sparse call with a row order and a queue draws its rows by KV group: enough rows to a workgroup, keys and values of the
    groups in flight within 256 MB.  (Seventeen groups, a prime number, are one to a set otherwise.)"""
    Nb, NG = -(-L // 128), batch * Hkv
    rows = batch * Hq * Nb
    units = torch.cuda.get_device_properties(0).multi_processor_count // 8 * 8
    resident = (1 if rows <= min(15 * Nb + 64, 5000) else 2) * units
    return rows >= (4 if NG > 8 and (NG % 8 == 0 or NG == 17) else 8) * resident and min(NG, 8) * 4 * Nb * 128 * 128 < 256 << 20


# one group to all XCDs, two, three (XCDs 0 and 1 have three each), seven, eight, nine and seventeen (queue 0 has one more), sixteen; rows of
# eight waves beyond 256 blocks; lengths that end inside a block; fewer rows than the rule asks for
@pytest.mark.parametrize("batch,L,Hq,Hkv", [(1, 16384, 32, 1), (1, 16300, 34, 2), (1, 16384, 33, 3), (1, 16000, 35, 7), (1, 16384, 32, 8),
                                            (3, 16384, 12, 3), (1, 16000, 17, 17), (2, 8100, 32, 8), (1, 33000, 8, 2), (1, 16256, 32, 8)])
def test_rows_by_group_equal_rows_one_by_one(batch, L, Hq, Hkv):
    import paper_2602_05853_amd as rr
    assert _by_group(batch, L, Hq, Hkv) == (L != 16256)
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


# groups that keep very little beside one that keeps half of its blocks, so that its rows are left for the workgroups of the others: two queues
# of one group each, three, eight of one and of two groups, a length that ends inside a block
@pytest.mark.parametrize("batch,L,Hq,Hkv", [(1, 16384, 32, 2), (1, 16300, 33, 3), (1, 16384, 32, 8), (2, 8192, 32, 8)])
def test_rows_that_are_missing_or_empty_in_a_launch_that_goes_on_with_other_queues(batch, L, Hq, Hkv):
    """Order entries that name no row, at the start of a group, in runs and at its end, and rows without a block, in the heavy group and
    in others: every named row is what a workgroup per row makes of it, the others stay untouched."""
    import paper_2602_05853_amd as rr
    assert _by_group(batch, L, Hq, Hkv)
    B, Nb, G = 128, -(-L // 128), Hq // Hkv
    g = torch.Generator(device="cuda:0").manual_seed(L + Hkv)
    Q, K, V = (torch.randn(batch, h, L, 128, generator=g, device="cuda:0").bfloat16() for h in (Hq, Hkv, Hkv))
    dense = torch.zeros(batch, Hq, Nb, Nb, dtype=torch.uint8, device="cuda:0")
    n = torch.arange(Nb, device="cuda:0")
    dense[:, :, n, n] = 1
    heavy = 1 if Hkv > 1 else 0                              # of the last prompt
    rows = slice(heavy * G, (heavy + 1) * G)
    dense[batch - 1, rows] |= (torch.rand(G, Nb, Nb, generator=g, device="cuda:0") < 0.5).to(torch.uint8).tril()
    dense[:, :, 5::7] = 0                                    # rows without a block
    mask = rr.rr_mask_from_dense(Q, K, dense, B)
    order, N = mask.row_order, G * Nb
    for grp in range(batch * Hkv):
        o = order[grp // Hkv, grp % Hkv]
        o[N // 2 + 8 * grp: N // 2 + 8 * grp + 40] = -1      # behind the rows that the workgroups start with
        o[N // 2 + 90: N // 2 + 130: 2] = N + grp
    order[batch - 1, heavy, :3] = -7
    order[batch - 1, heavy, N - 60:] = 2 ** 31 - 1
    order[0, Hkv - 1] = -1 if Hkv > 2 else order[0, Hkv - 1]   # a group without a row
    named = torch.zeros(batch * Hkv, N, dtype=torch.bool, device="cuda:0")
    for grp in range(batch * Hkv):
        o = order[grp // Hkv, grp % Hkv]
        named[grp, o[(o >= 0) & (o < N)].long()] = True
    named = named.view(batch, Hq, Nb).repeat_interleave(B, 2)[:, :, :L, None]
    print(f"[groups] {batch} x {Hq}/{Hkv} heads, {L} tokens, {int(named.sum())} of {named.numel()} positions named", flush=True)
    ref = rr.rr_sparse_attn(Q, K, V, dataclasses.replace(mask, queue=None, row_order=None))
    for rep in range(5):
        O = torch.full_like(Q, 7.0)
        rr.rr_sparse_attn(Q, K, V, mask, O=O)
        torch.cuda.synchronize()
        assert int(mask.queue.abs().max()) == 0, rep
        assert torch.equal(O, torch.where(named, ref, torch.full_like(ref, 7.0))), rep


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
