"""The merge of a split launch (steps of more than 32 query rows to a KV head), which requests one, four or eight parts at once by how many are
left, for numbers of parts around those trips, against attention in 64 bits; dense, and sparse with parts that hold none of a row's blocks."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# an eighth of the blocks of the context is the number of parts
@pytest.mark.parametrize("parts", [2, 3, 4, 5, 8, 9, 12, 13, 17, 32])
@pytest.mark.parametrize("sparse", [False, True])
def test_parts_of_a_split_launch_are_merged(parts, sparse):
    import paper_2602_05853_amd as rr
    dev, d, Hq, Hkv, T = "cuda:0", 128, 4, 1, 40
    L = 128 * 8 * parts - 7
    g = torch.Generator(device=dev).manual_seed(parts)
    Q = torch.randn(1, Hq, T, d, generator=g, device=dev).bfloat16()
    K, V = (torch.randn(1, Hkv, L, d, generator=g, device=dev).bfloat16() for _ in range(2))
    need = rr.rr_attn_workspace_bytes(Q, K, 128)
    assert need // (Hq * T * (d + 1) * 4) == parts          # (whole 256 bytes)
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device=dev)
    print(f"[split merge] {parts} parts of {L}, {'sparse' if sparse else 'dense'}", flush=True)
    lse = torch.empty(1, Hq, T, device=dev)
    sees = (torch.arange(L, device=dev)[None] <= torch.arange(L - T, L, device=dev)[:, None]).expand(Hq, T, L)
    if sparse:
        Nb = 8 * parts
        blocks = torch.zeros(1, Hq, 1, Nb, dtype=torch.uint8, device=dev)
        blocks[0, 0, 0, [0, Nb - 1]] = 1                      # nothing in between
        blocks[0, 1, 0, 3:9] = 1                              # the diagonal block is not among them
        blocks[0, 2] = (torch.rand(1, Nb, generator=g, device=dev) < 0.5).to(torch.uint8)
        blocks[0, 2, 0, 1] = 1
        mask = rr.rr_mask_from_dense(Q, K, blocks, 128)       # head 3: no block at all
        O = rr.rr_sparse_attn(Q, K, V, mask, lse=lse, workspace=ws)
        sees = sees & blocks[0, :, 0].bool().repeat_interleave(128, 1)[:, None, :L]
    else:
        O = rr.rr_dense_attn(Q, K, V, 128, lse=lse, workspace=ws)
    torch.cuda.synchronize()
    s = (Q[0].double() @ K[0, 0].double().T / d ** 0.5).masked_fill(~sees, float("-inf"))
    ref = torch.softmax(s, 2).nan_to_num(0.0) @ V[0, 0].double()
    # weights rounded to bf16 and the output's own rounding: 2^-8 of the largest value each; the log-sum-exp's terms as rounded
    assert ((O[0].double() - ref).abs() <= 2.0 ** -8 * (V.abs().max().double() + ref.abs())).all()
    want = torch.logsumexp(s, 2)
    assert torch.equal(lse[0].isinf(), want.isinf())
    assert ((lse[0].double() - want)[~want.isinf()].abs() <= 2.0 ** -8 + 1e-5).all()
