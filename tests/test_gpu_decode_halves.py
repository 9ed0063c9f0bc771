"""Steps of 17 to 32 query rows per KV head on fewer workgroups than compute units: two workgroups to a part, 16 rows each, up to 128 parts in
all, and one of eight waves beyond (the last two cases), against attention in 64 bits.  Heads of which both workgroups have rows, steps that lie in two query blocks, numbers of (part, KV head) pairs that are no multiple of
eight, parts of eight waves and of four, lists that differ from head to head and rows without a block; dense calls."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,Hq,Hkv,T,L", [(1, 4, 1, 5, 128 * 40), (1, 7, 1, 3, 128 * 33 + 2), (1, 3, 1, 10, 128 * 17 + 100), (2, 32, 1, 1, 128 * 150 - 7),
                                              (1, 6, 3, 16, 128 * 50 + 9), (3, 8, 2, 5, 128 * 21), (1, 17, 1, 1, 128 * 16), (1, 10, 2, 6, 128 * 90 + 3),
                                              (12, 3, 1, 8, 128 * 129 - 77), (5, 16, 4, 8, 128 * 60 + 20)])
@pytest.mark.parametrize("sparse", [True, False])
def test_rows_in_two_workgroups(batch, Hq, Hkv, T, L, sparse):
    import paper_2602_05853_amd as rr
    dev, d, G, Nb = "cuda:0", 128, Hq // Hkv, -(-L // 128)
    assert 16 < G * T <= 32
    g = torch.Generator(device=dev).manual_seed(L + T)
    Q = torch.randn(batch, Hq, T, d, generator=g, device=dev).bfloat16()
    K, V = (torch.randn(batch, Hkv, L, d, generator=g, device=dev).bfloat16() for _ in range(2))
    ws = torch.full((rr.rr_attn_workspace_bytes(Q, K, 128),), 0xFF, dtype=torch.uint8, device=dev)
    print(f"[halves] {batch} x {Hq}/{Hkv} heads, {T} of {L}, {ws.numel() // (batch * Hq * T * 129 * 4)} parts", flush=True)
    parts = ws.numel() // (batch * Hq * T * 129 * 4) * batch * Hkv
    assert parts <= 128 if batch < 5 else 128 < parts < 256
    pos = torch.arange(L, device=dev)
    sees = pos[None] <= torch.arange(L - T, L, device=dev)[:, None]                   # [T, L]
    sees = sees.expand(batch, Hq, T, L)
    m0 = (L - T) // 128
    if sparse:
        dense = (torch.rand(batch, Hq, Nb - m0, Nb, generator=g, device=dev) < 0.3).to(torch.uint8)
        dense[:, Hq // 2] = 0                                                          # a head without a block
        dense[:, 0] = 1
        mask = rr.rr_mask_from_dense(Q, K, dense, 128)
        O = rr.rr_sparse_attn(Q, K, V, mask, workspace=ws)
        row = torch.arange(L - T, L, device=dev) // 128 - m0
        sees = sees & dense.bool()[:, :, row][..., pos // 128]
    else:
        O = rr.rr_dense_attn(Q, K, V, 128, workspace=ws)
    torch.cuda.synchronize()
    s = Q.double() @ K.double().repeat_interleave(G, 1).transpose(2, 3).contiguous() / d ** 0.5
    p = torch.softmax(s.masked_fill(~sees, float("-inf")), 3).nan_to_num(0.0)
    ref = p @ V.double().repeat_interleave(G, 1)
    # products and sums in 32 bits, weights of at most one: 2^-15 of the largest value, and the output's own rounding to bf16
    assert ((O.double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 2.0 ** -15 * V.abs().max()).all()
