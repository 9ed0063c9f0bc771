"""Planned chunk launches whose rows need parts of different lengths: all rows long (the slots hold them only with longer
parts, or no row is cut), a few long among short ones, none long.  Every output row against the same call without a
workspace, which walks every row in one piece.  Both round the probabilities to bf16, relative to references that differ
between them: each by at most 2^-8, and by half of that and less where hundreds of terms are rounded either way, so a
result moves by at most 2^-8 sum(p |v|) <= 2^-8 max|v| (max|v| taken from the inputs, about 5.3) plus its own last rounding,
2^-8 of the value.  The log-sum-exp is the logarithm of the sum of the rounded probabilities (unrounded where a step moved
the reference), so likewise 2^-8 between the two forms, and far less in the mean."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows_kept", ["all", "none_long", "some", "half"])
@pytest.mark.parametrize("Hq,Hkv,L,Lq", [(4, 1, 128 * 200, 600), (16, 4, 128 * 700 - 41, 512), (32, 8, 128 * 170, 2048),
                                          (32, 8, 128 * 160, 5000)])   # more rows than the plan takes at once
def test_parts_fit_the_slots(Hq, Hkv, L, Lq, rows_kept):
    import paper_2602_05853_amd as rr
    B, dev = 128, "cuda:0"
    g = torch.Generator(device=dev).manual_seed(L)
    Q = torch.randn(1, Hq, Lq, 128, generator=g, device=dev).bfloat16()
    K = torch.randn(1, Hkv, L, 128, generator=g, device=dev).bfloat16()
    V = torch.randn(1, Hkv, L, 128, generator=g, device=dev).bfloat16()
    Nb, m0 = -(-L // B), (L - Lq) // B
    rows = Nb - m0
    rng = np.random.default_rng(Nb)
    dense = np.zeros((Hq, rows, Nb), dtype=np.uint8)
    for h in range(Hq):
        for r in range(rows):
            long = {"all": True, "none_long": False, "some": r == rows - 1, "half": rng.random() < 0.5}[rows_kept]
            n = m0 + r + 1
            dense[h, r, :n] = 1 if long else rng.random(n) < 30.0 / n
    print(f"[plan] {Hq}/{Hkv} heads, {Lq} of {L}, {rows_kept}: {int(dense.sum())} entries, {Hq * rows} rows", flush=True)
    mask = rr.rr_mask_from_dense(Q, K, torch.from_numpy(dense)[None].to(dev), B)
    need = rr.rr_attn_workspace_bytes(Q, K, B)
    assert need > 0
    out = []
    for ws in (None, torch.full((need,), 0xFF, dtype=torch.uint8, device=dev)):
        O = torch.full_like(Q, float("nan"))
        lse = torch.full((1, Hq, Lq), float("nan"), dtype=torch.float32, device=dev)
        rr.rr_sparse_attn(Q, K, V, mask, O=O, lse=lse, workspace=ws)
        torch.cuda.synchronize()
        out.append((O.float(), lse))
    (a, la), (b, lb) = out
    assert torch.equal(torch.isinf(la), torch.isinf(lb))
    fin = torch.isfinite(la)
    assert fin.any() and (la - lb)[fin].abs().max() <= 2.0 ** -8 and (la - lb)[fin].abs().mean() <= 2.0 ** -12
    top = V.abs().max().float()
    assert ((a - b).abs() <= 2.0 ** -8 * torch.maximum(a.abs(), b.abs()) + 2.0 ** -8 * top).all()
