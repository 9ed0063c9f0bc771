"""Planned chunk launches whose rows take every number of parts (runs of eight parts are dealt to the XCDs, what is left over is
not) and start at any slot.  Every output row against the same call without a workspace.

The values tell which blocks a row attended: block n adds 1 to channel n mod 61 and 1 to channel 61 + n mod 67, so a block lost, taken
twice or taken for its neighbour moves a channel by one of its at most 13 blocks, or moves it away from 0.  Nothing cancels in
these sums, so both sides hold every channel to a share of itself: the probabilities are rounded to bf16 relative to references of
their own (2^-9 each, in numerator and denominator) and so is the result, 3 times 2^-9 a side, and the log-sum-exp to 2^-8."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("listed", [True, False])
@pytest.mark.parametrize("Hq,Hkv,L,Lq", [(2, 1, 128 * 300, 128 * 20), (8, 2, 128 * 700 - 5, 128 * 12 - 77)])
def test_rows_of_every_number_of_parts(Hq, Hkv, L, Lq, listed):
    import paper_2602_05853_amd as rr
    B, dev = 128, "cuda:0"
    g = torch.Generator(device=dev).manual_seed(Lq)
    Q = torch.randn(1, Hq, Lq, 128, generator=g, device=dev).bfloat16()
    K = torch.randn(1, Hkv, L, 128, generator=g, device=dev).bfloat16()
    Nb, m0 = -(-L // B), (L - Lq) // B
    V = torch.zeros(1, Hkv, L, 128, dtype=torch.bfloat16, device=dev)
    key = torch.arange(L, device=dev)
    V[:, :, key, key // B % 61] = 1
    V[:, :, key, 61 + key // B % 67] = 1
    rows = Nb - m0
    print(f"[parts] {Hq}/{Hkv} heads, {Lq} of {L}, listed {listed}", flush=True)
    call = lambda **k: rr.rr_dense_attn(Q, K, V, B, **k)
    if listed:
        dense = np.zeros((Hq, rows, Nb), dtype=np.uint8)
        for i in range(Hq * rows):              # 17 i + 3 entries: 1 part, 1, 1, 2, .. and the diagonal block in every other row
            h, r = i % Hq, i // Hq
            n = m0 + r + 1
            kept = np.arange(n)[-min(n, (17 * i + 3) % n + 1):]
            dense[h, r, kept if i % 2 else kept - kept[0]] = 1
        mask = rr.rr_mask_from_dense(Q, K, torch.from_numpy(dense)[None].to(dev), B)
        call = lambda **k: rr.rr_sparse_attn(Q, K, V, mask, **k)
    need = rr.rr_attn_workspace_bytes(Q, K, B)
    assert need > 0
    out = []
    for ws in (None, torch.full((need,), 0xFF, dtype=torch.uint8, device=dev)):
        O = torch.full_like(Q, float("nan"))
        lse = torch.full((1, Hq, Lq), float("nan"), dtype=torch.float32, device=dev)
        call(O=O, lse=lse, workspace=ws)
        torch.cuda.synchronize()
        out.append((O.float(), lse))
    (a, la), (b, lb) = out
    assert torch.isfinite(la).all() and torch.isfinite(lb).all()
    assert (la - lb).abs().max() <= 2.0 ** -8
    assert ((a - b).abs() <= 6 * 2.0 ** -9 * torch.maximum(a, b)).all()
