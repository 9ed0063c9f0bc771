"""The launch-order hint against its rule, applied on the host: rows of a KV head by count class (counts that differ by
less than 8 blocks), heaviest first, inside a class by descending query block and then head, launch ranks transposed in
runs of 8 G rows.  Row counts at the edges of a wavefront and of the workgroup, with equal and with spread counts."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("equal", [False, True])
@pytest.mark.parametrize("G,Nb", [(1, 1), (1, 63), (1, 64), (1, 65), (3, 21), (4, 256), (4, 257), (7, 311), (5, 205), (2, 1500)])
def test_row_order_follows_its_rule(G, Nb, equal):
    import paper_2602_05853_amd as rr
    B, Hkv, d = 8, 2, 8
    Hq = G * Hkv
    dev = "cuda:0"
    Q = torch.zeros(1, Hq, Nb * B, d, device=dev)
    K = torch.zeros(1, Hkv, Nb * B, d, device=dev)
    rng = np.random.default_rng(G * 1000 + Nb)
    dense = np.zeros((Hq, Nb, Nb), dtype=np.uint8)
    for h in range(Hq):
        for m in range(Nb):
            dense[h, m, : 1 if equal else rng.integers(0, m + 2)] = 1
    mask = rr.rr_mask_from_dense(Q, K, torch.from_numpy(dense)[None].to(dev), B)
    torch.cuda.synchronize()
    count = dense.sum(-1).astype(int)
    assert np.array_equal(mask.row_count.cpu().numpy()[0], count)
    got = mask.row_order.cpu().numpy()[0]
    print(f"[row order] G={G} Nb={Nb} equal={equal}", flush=True)
    N = G * Nb
    for kv in range(Hkv):
        rows = [(m, hl) for m in range(Nb - 1, -1, -1) for hl in range(G)]
        rows.sort(key=lambda r: (Nb - count[kv * G + r[1], r[0]]) >> 3)          # stable
        want = np.empty(N, dtype=np.int32)
        full = N // (8 * G) * (8 * G)
        for i, (m, hl) in enumerate(rows):
            rank = i
            if G > 1 and i < full:
                base, w = i // (8 * G) * (8 * G), i % (8 * G)
                rank = base + 8 * (w % G) + w // G
            want[rank] = hl * Nb + m
        assert np.array_equal(got[kv], want)


@pytest.mark.parametrize("equal", [False, True])
@pytest.mark.parametrize("G,Nb", [(1, 255), (1, 256), (1, 257), (8, 64), (1, 513), (2, 512)])
def test_row_order_at_the_largest_sizes_of_its_workgroups(G, Nb, equal):
    """256, 512 and 1024 threads."""
    test_row_order_follows_its_rule(G, Nb, equal)
