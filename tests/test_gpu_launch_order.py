"""The launch order of sparse calls changes no result: sets of KV groups with the heaviest rows of all groups in front (more
groups than one set holds), against the order without a row order, bit for bit, and every row of the mask is computed.
Row order with and without a queue, whole blocks and lengths that end inside one, a number of groups that is no power of two."""
import dataclasses

import pytest
import torch

pytestmark = pytest.mark.gpu


# batch, L, Hq, Hkv: 16 groups of 2.6 MB of K and V (sets of 8), 15 groups (sets of 5 and 5 and 5), 4 groups of 10 MB, groups
# of 7 heads, and 30 groups whose first run is half of their rows; 64 heads, the most whose first runs go in front of short prompts, 84, 80
# and 65 without, 66 heads of 128 blocks with them and of 127 without
@pytest.mark.parametrize("batch,L,Hq,Hkv", [(2, 5120, 16, 8), (5, 5100, 6, 3), (4, 20480, 2, 1), (3, 9000, 28, 4), (40, 2048, 2, 1),
                                            (2, 9000, 28, 4), (30, 2048, 2, 1), (1, 5000, 64, 16), (13, 3000, 5, 1), (33, 16300, 2, 1),
                                            (33, 16250, 2, 1)])
@pytest.mark.parametrize("queue", [True, False])
def test_sets_of_groups_compute_every_row(batch, L, Hq, Hkv, queue):
    import paper_2602_05853_amd as rr
    dev, d = "cuda:0", 128
    g = torch.Generator(device=dev).manual_seed(L + Hq)
    Q = torch.randn(batch, Hq, L, d, generator=g, device=dev).bfloat16()
    K, V = (torch.randn(batch, Hkv, L, d, generator=g, device=dev).bfloat16() for _ in range(2))
    # structure, so that rows of very different length meet: a part of the keys that only some queries look for
    u = torch.randn(d, generator=g, device=dev)
    K[:, :, : L // 8] += 0.7 * u.bfloat16()
    Q[:, :, ::3] += 0.7 * u.bfloat16()
    mask = rr.rr_estimate(Q, K, 16, 128, 0.7)
    if not queue:
        mask = dataclasses.replace(mask, queue=None)
    print(f"[order] {batch} x {Hq}/{Hkv} heads, {L} tokens, queue {queue}, counts {int(mask.row_count.min())}..{int(mask.row_count.max())}", flush=True)
    O = torch.full_like(Q, float("nan"))
    rr.rr_sparse_attn(Q, K, V, mask, O=O)
    ref = rr.rr_sparse_attn(Q, K, V, dataclasses.replace(mask, row_order=None, queue=None))
    torch.cuda.synchronize()
    assert torch.isfinite(O.float()).all()
    assert torch.equal(O, ref)
    if queue:
        assert int(mask.queue.abs().max()) == 0
