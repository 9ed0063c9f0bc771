"""Attention of steps with 5 to 32 query rows per KV head (bf16, d = 128, B = 128, with the workspace): row counts at the
edges of the 16-column tiles, steps inside one block and across two, lengths that end inside a block, batches, dense and
under random block lists (one of them with a single block, one empty), against attention in 64 bits under the same mask."""
import math

import numpy as np
import pytest
import torch

import gpu_util as gu

pytestmark = pytest.mark.gpu

CASES = [  # batch, Hq, Hkv, T, L
    (1, 5, 1, 1, 640), (1, 8, 1, 1, 129), (2, 16, 2, 1, 2700), (1, 14, 2, 1, 5000), (1, 6, 1, 1, 1),   # one token
    (1, 8, 2, 2, 3001), (1, 8, 2, 2, 2049), (1, 4, 1, 4, 2690), (2, 8, 2, 4, 2691), (1, 17, 1, 1, 2561),
    (1, 8, 2, 8, 4000), (1, 8, 2, 8, 4099), (1, 7, 1, 4, 2700), (1, 2, 1, 16, 2817), (1, 1, 1, 31, 2700),
    (1, 32, 1, 1, 2688), (1, 16, 1, 2, 2689), (1, 4, 4, 32, 2720),
]


@pytest.mark.parametrize("sparse", [False, True])
@pytest.mark.parametrize("batch,Hq,Hkv,T,L", CASES)
def test_step_attention(batch, Hq, Hkv, T, L, sparse):
    import paper_2602_05853_amd as rr
    B, d = 128, 128
    g = torch.Generator(device="cuda:0").manual_seed(L + T)
    Q = (torch.randn(batch, Hq, T, d, generator=g, device="cuda:0") * 1.5).bfloat16()
    K = torch.randn(batch, Hkv, L, d, generator=g, device="cuda:0").bfloat16()
    V = torch.randn(batch, Hkv, L, d, generator=g, device="cuda:0").bfloat16()
    if T > 1 or batch > 1:                                  # heads inside positions: other strides than the default
        Q, K, V = (t.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3) for t in (Q, K, V))
    Nb, m0 = -(-L // B), (L - T) // B
    rows = Nb - m0
    mask = torch.ones(batch, Hq, rows, Nb, dtype=torch.uint8, device="cuda:0")
    if sparse:
        mask = (torch.rand(mask.shape, generator=g, device="cuda:0") < 0.3).to(torch.uint8)
        mask[:, 0, 0] = 0                                   # nothing selected
        mask[:, Hq - 1, rows - 1] = 0
        mask[:, Hq - 1, rows - 1, Nb // 2] = 1              # one block
    for r in range(rows):
        mask[:, :, r, m0 + r + 1:] = 0
    need = rr.rr_attn_workspace_bytes(Q, K, B)
    assert need > 0
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda:0")
    O = torch.full_like(Q, float("nan"))
    lse = torch.full((batch, Hq, T), float("nan"), dtype=torch.float32, device="cuda:0")
    print(f"[step] {batch} x {Hq}/{Hkv} heads, {T} of {L} {'sparse' if sparse else 'dense'}", flush=True)
    if sparse:
        bm = rr.rr_mask_from_dense(Q, K, mask.contiguous(), B)
        rr.rr_sparse_attn(Q, K, V, bm, O=O, lse=lse, workspace=ws)
    else:
        rr.rr_dense_attn(Q, K, V, B, O=O, lse=lse, workspace=ws)
    torch.cuda.synchronize()
    G = Hq // Hkv
    q, k, v = (t.double().cpu() for t in (Q, K, V))
    k, v = k.repeat_interleave(G, 1), v.repeat_interleave(G, 1)
    pos = torch.arange(L - T, L)
    seen = mask.cpu().bool()[:, :, pos // B - m0].repeat_interleave(B, 3)[..., :L] & (torch.arange(L) <= pos[:, None])
    s = ((q[:, :, :, None, :] * k[:, :, None]).sum(-1) / math.sqrt(d)).masked_fill(~seen, float("-inf"))
    want_lse = torch.logsumexp(s, -1)
    p = torch.exp(s - want_lse.clamp_min(-1e300)[..., None])
    want = (p[..., None] * v[:, :, None]).sum(-2)
    err = (O.double().cpu() - want).abs()
    assert err.max() <= gu.BF16_MAX_ABS and err.mean() <= gu.BF16_MEAN_ABS, (err.max(), err.mean())
    got = lse.double().cpu()
    assert torch.equal(torch.isinf(got), torch.isinf(want_lse))
    finite = ~torch.isinf(want_lse)
    if finite.any():
        # scores and sums are held in 32 bits: a few 2^-24 of logits of magnitude 20
        assert (got - want_lse)[finite].abs().max() <= 1e-4


@pytest.mark.parametrize("T,L", [(1, 2700), (4, 2700), (4, 2690)])
def test_blocks_a_row_did_not_select_do_not_reach_it(T, L):
    """Infinite and NaN keys and values in blocks that one head alone selected (and, across two query blocks, in the
    second one): the rows without them are what they are with ordinary values there, bit for bit."""
    import paper_2602_05853_amd as rr
    B, dev = 128, "cuda:0"
    g = torch.Generator(device=dev).manual_seed(L + T)
    Q = torch.randn(1, 6, T, 128, generator=g, device=dev).bfloat16()
    K = torch.randn(1, 1, L, 128, generator=g, device=dev).bfloat16()
    V = torch.randn(1, 1, L, 128, generator=g, device=dev).bfloat16()
    Nb, m0 = -(-L // B), (L - T) // B
    rows = Nb - m0
    mask = torch.ones(1, 6, rows, Nb, dtype=torch.uint8, device=dev)
    mask[:, 1:, :, 3] = 0
    mask[:, 1:, :, 7] = 0
    for r in range(rows):
        mask[:, :, r, m0 + r + 1:] = 0
    bm = rr.rr_mask_from_dense(Q, K, mask.contiguous(), B)
    ws = torch.empty(rr.rr_attn_workspace_bytes(Q, K, B), dtype=torch.uint8, device=dev)
    clean = rr.rr_sparse_attn(Q, K, V, bm, workspace=ws).clone()
    dense_clean = rr.rr_dense_attn(Q, K, V, B, workspace=ws).clone()
    K2, V2 = K.clone(), V.clone()
    K2[:, :, 3 * B:4 * B] = float("nan")
    V2[:, :, 3 * B:4 * B] = float("nan")
    V2[:, :, 7 * B + 5] = float("inf")
    got = rr.rr_sparse_attn(Q, K2, V2, bm, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(got[:, 1:], clean[:, 1:])
    if rows == 2:                                           # dense: the second query block's keys are past the first one's rows
        V3 = V.clone()
        V3[:, :, (m0 + 1) * B:] = float("nan")
        first = (m0 + 1) * B - (L - T)
        got = rr.rr_dense_attn(Q, K, V3, B, workspace=ws)
        torch.cuda.synchronize()
        assert torch.equal(got[:, :, :first], dense_clean[:, :, :first])


@pytest.mark.parametrize("Hq,Hkv,longest", [(32, 8, 16), (28, 4, 8), (16, 1, 4), (64, 8, 6)])
def test_a_workspace_sized_for_the_longest_step_serves_the_shorter_ones(Hq, Hkv, longest):
    """Steps of 1 .. longest positions on one workspace, on one of the size they ask for themselves (fewer parts) and on a
    large one (as many parts as pay).  bf16 outputs of fp32 sums in another order: neighbouring numbers at most, 2^-7."""
    import paper_2602_05853_amd as rr
    from paper_2602_05853_amd import binding as bd
    dev, B, L = "cuda:0", 128, 128 * 80
    g = torch.Generator(device=dev).manual_seed(Hq)
    Qall = torch.randn(1, Hq, longest, 128, generator=g, device=dev).bfloat16()
    K, V = (torch.randn(1, Hkv, L, 128, generator=g, device=dev).bfloat16() for _ in range(2))
    steps = {T: Qall[:, :, longest - T:].contiguous() for T in range(1, longest + 1)}
    need = {T: rr.rr_attn_workspace_bytes(Q, K, B) for T, Q in steps.items()}
    small = [T for T in (1, 2) if Hq // Hkv * T <= 8]       # these need what they ask for
    assert all(need[T] <= need[T + 1] for T in range(1, longest) if T not in small)
    one = torch.empty(max(need[T] for T in small + [longest]), dtype=torch.uint8, device=dev)
    large = torch.empty(16 << 20, dtype=torch.uint8, device=dev)
    for T, Q in steps.items():
        mask = rr.rr_mask_from_dense(Q, K, (torch.rand(1, Hq, 1, L // B, generator=g, device=dev) < 0.4).to(torch.uint8), B)
        for call in (lambda **kw: rr.rr_dense_attn(Q, K, V, B, **kw), lambda **kw: rr.rr_sparse_attn(Q, K, V, mask, **kw)):
            out = []
            for ws in (one, torch.empty(need[T], dtype=torch.uint8, device=dev), large):
                lse = torch.empty(1, Hq, T, dtype=torch.float32, device=dev)
                out.append((call(workspace=ws, lse=lse).float(), lse))
            torch.cuda.synchronize()
            for got, lse in out[:2]:
                assert ((got - out[2][0]).abs() <= 2.0 ** -7 * out[2][0].abs() + 1e-5).all(), T
                assert (lse - out[2][1]).abs().max() <= 1e-4, T
    # what no form of the step can do with is refused as before
    with pytest.raises(bd.RRError) as err:
        rr.rr_dense_attn(Qall, K, V, B, workspace=one[:256])
    assert err.value.status == bd.RR_ERR_WORKSPACE
