"""Generic sparse attention whose last query block is taken on smaller query tiles than the others: a list of every block against
the dense call, which takes all blocks alike.  Each query's keys meet the same waves in the same order, so the results are
equal to the bit; the dense call is checked against the oracle elsewhere."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# (B, d, dtype): 64-, 32- and 16-query tiles for the other blocks; blocks that are no multiple of either tile
@pytest.mark.parametrize("B,d,dtype", [(64, 64, "bf16"), (128, 40, "bf16"), (48, 64, "bf16"), (34, 72, "bf16"), (24, 128, "bf16"),
                                       (64, 128, "f32"), (33, 64, "f32"), (17, 16, "f32"), (16, 64, "f32")])
@pytest.mark.parametrize("blocks,cut,Lq_off", [(20, 0, 0), (33, 15, 0), (36, 7, 5), (90, 1, 0)])   # cut: of the last block; a step inside a block
def test_list_of_every_block_equals_the_dense_call(B, d, dtype, blocks, cut, Lq_off):
    import paper_2602_05853_amd as rr
    dev, Hq, Hkv = "cuda:0", 16, 4
    L = B * blocks - min(cut, B - 1)
    Lq = L - Lq_off
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device=dev).manual_seed(B * d + blocks)
    Q = torch.randn(1, Hq, Lq, d, generator=g, device=dev).to(t)
    K = torch.randn(1, Hkv, L, d, generator=g, device=dev).to(t)
    V = torch.randn(1, Hkv, L, d, generator=g, device=dev).to(t)
    Nb, m0 = -(-L // B), (L - Lq) // B
    dense = torch.ones(Nb, Nb, dtype=torch.uint8, device=dev).tril()[m0:].expand(1, Hq, Nb - m0, Nb).contiguous()
    print(f"[last] B {B} d {d} {dtype}: {Lq} of {L}", flush=True)
    mask = rr.rr_mask_from_dense(Q, K, dense, B)
    out = []
    for call in (lambda **k: rr.rr_dense_attn(Q, K, V, B, **k), lambda **k: rr.rr_sparse_attn(Q, K, V, mask, **k)):
        O = torch.full_like(Q, float("nan"))
        lse = torch.full((1, Hq, Lq), float("nan"), dtype=torch.float32, device=dev)
        call(O=O, lse=lse)
        torch.cuda.synchronize()
        out.append((O, lse))
    (a, la), (b, lb) = out
    assert torch.equal(a, b) and torch.equal(la, lb)
