"""The merge of a decode step's parts, which takes eight parts per wavefront at once, for numbers of parts around its trips of 32, against
attention in 64 bits; with one block far above the others, so that parts of weight zero are among them, and without."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# blocks of the context -> parts of at least two blocks; the last ones on 256 parts of three blocks and fewer
@pytest.mark.parametrize("blocks", [1, 2, 3, 15, 17, 62, 64, 66, 130, 700])
@pytest.mark.parametrize("far", [False, True])
def test_parts_are_merged(blocks, far):
    import paper_2602_05853_amd as rr
    dev, d, Hq = "cuda:0", 128, 3
    L = 128 * blocks - (5 if blocks % 2 else 0)
    g = torch.Generator(device=dev).manual_seed(blocks)
    Q = torch.randn(1, Hq, 1, d, generator=g, device=dev).bfloat16()
    K, V = (torch.randn(1, 1, L, d, generator=g, device=dev).bfloat16() for _ in range(2))
    if far:
        at = L // 3
        K[0, 0, at] = (40.0 * Q[0, 0, 0].float()).bfloat16()      # a score of some 400 for the first head
    need = rr.rr_attn_workspace_bytes(Q, K, 128)
    ws = torch.full((max(need, 1),), 0xFF, dtype=torch.uint8, device=dev)
    print(f"[merge] {blocks} blocks, {need // (Hq * 129 * 4)} parts", flush=True)
    lse = torch.empty(1, Hq, 1, device=dev)
    O = rr.rr_dense_attn(Q, K, V, 128, lse=lse, workspace=ws)
    torch.cuda.synchronize()
    s = Q[0, :, 0].double() @ K[0, 0].double().T / d ** 0.5
    ref = torch.softmax(s, 1) @ V[0, 0].double()
    # products and sums in 32 bits, weights of at most one: 2^-15 of the largest value, and the output's own rounding to bf16
    assert ((O[0, :, 0].double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 2.0 ** -15 * V.abs().max()).all()
    assert ((lse[0, :, 0].double() - torch.logsumexp(s, 1)).abs() <= 2.0 ** -18 * s.abs().max() + 1e-5).all()
