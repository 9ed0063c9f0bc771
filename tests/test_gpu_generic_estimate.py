"""The estimate for shapes other than bf16, d = 128: every way a score tile of 16 queries is filled (4 to 32 queries a block,
one to four heads of a KV head side by side, other numbers through LDS), head widths that end inside a chunk of 16
channels, strides that do not fill a tile, softmax state in LDS and in the workspace, both against the oracle."""
import numpy as np
import pytest
import torch

import gpu_util as gu

pytestmark = pytest.mark.gpu

CASES = [  # B, S, d, Hq, Hkv, L, dtype
    (64, 16, 64, 4, 1, 64 * 9, "bf16"),        # 4 queries a block, four heads a tile
    (64, 16, 24, 4, 2, 64 * 9 - 5, "f32"),     # ... two heads
    (64, 8, 40, 4, 2, 64 * 11 - 30, "bf16"),   # 8 queries, two heads
    (32, 4, 8, 3, 3, 32 * 13 - 7, "f32"),      # ... heads that share no KV head
    (64, 4, 136, 4, 2, 64 * 7, "f32"),         # 16 queries
    (128, 4, 72, 2, 1, 128 * 5 - 100, "bf16"), # 32 queries
    (48, 4, 56, 4, 2, 48 * 9 - 11, "bf16"),    # 12 queries: through LDS
    (20, 4, 64, 2, 1, 20 * 12 - 3, "f32"),     # 5 queries
    (128, 1, 16, 1, 1, 128 * 3, "f32"),        # every query
    (32, 4, 64, 2, 1, 32 * 2200, "bf16"),      # rows of thousands of blocks: state in the workspace
]


@pytest.mark.parametrize("B,S,d,Hq,Hkv,L,dtype", CASES)
def test_generic_estimate_matches_the_oracle(B, S, d, Hq, Hkv, L, dtype):
    import paper_2602_05853_amd as rr
    from oracle import rr_oracle as oracle
    rng = np.random.default_rng(B * 7 + d)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x = {"Q": 2.0 * rng.standard_normal((Hq, L, d)), "K": rng.standard_normal((Hkv, L, d)),
         "V": np.zeros((Hkv, 1, d))}
    x = {k: torch.from_numpy(v.astype(np.float32)).to(tdt).float().numpy() for k, v in x.items()}
    t = gu.to_device(x, dtype)
    print(f"[generic estimate] B={B} S={S} d={d} {Hq}/{Hkv} L={L} {dtype}", flush=True)
    long = L > 10000                                        # the oracle row by row there
    Nb = -(-L // B)
    mask = rr.rr_estimate(t["Q"], t["K"], S, B, 0.9, block_mass=True)
    torch.cuda.synchronize()
    mass = mask.block_mass.cpu().numpy()[0]
    if long:
        dense = mask.dense.cpu().numpy()[0]
        for h, m in [(0, 0), (1, 63), (0, 64), (1, 1000), (0, Nb - 2)]:
            row_mask, row_frac, row_margin = oracle.estimate_row(x["Q"][h], x["K"][h // (Hq // Hkv)], h, m, S, B, 0.9)[:3]
            n = m + 1
            assert np.abs(mass[h, m, :n] - row_frac[:n]).max() <= 1e-6
            differ = dense[h, m, :n] != row_mask[:n]
            assert not (differ & (np.abs(row_margin[:n]) > gu.MARGIN_TOL)).any(), (h, m)
        return
    gu.check_mask_structures(mask)
    ref_mask, ref_frac, ref_margin = gu.oracle_estimate(x, S, B, 0.9)
    rep = gu.compare_estimate(mask, ref_mask, ref_frac, ref_margin, 0.9)
    # fractions of a row are at most 1 and come from 32-bit logits of magnitude below 4: a few 2^-24 each
    assert rep["failed"] == 0 and rep["mass_max_abs_err"] <= 1e-6, rep


# Blocks of 32 keys and 4 to 32 sampled queries: a batch of more than 512 workgroups (four waves each) and its prompts alone, of up to 512
# (eight, up to 256 blocks: the last case has 257 and stays on four).  As many heads as KV heads, one to a workgroup.
@pytest.mark.parametrize("S,batch,Nb,H", [(8, 130, 5, 4), (4, 40, 16, 4), (2, 9, 64, 4), (1, 3, 200, 2), (4, 3, 255, 2), (8, 5, 256, 2), (1, 3, 256, 2),
                                          (4, 5, 257, 1)])
def test_workgroups_of_four_and_of_eight_waves(S, batch, Nb, H):
    import paper_2602_05853_amd as rr
    B, d, L = 32, 40, 32 * Nb - 3
    assert batch * H * Nb > 512 and H * Nb <= 512
    g = torch.Generator(device="cuda:0").manual_seed(Nb)
    Q, K = (2.0 * torch.randn(batch, H, L, d, generator=g, device="cuda:0") for _ in range(2))
    print(f"[waves] S {S}: {batch} prompts of {Nb} blocks, {H} heads", flush=True)
    whole = rr.rr_estimate(Q, K, S, B, 0.8, block_mass=True)
    for b in (0, batch - 1):
        one = rr.rr_estimate(Q[b:b + 1], K[b:b + 1], S, B, 0.8, block_mass=True)
        torch.cuda.synchronize()
        for name in ("row_count", "dense", "block_mass", "row_order"):
            assert torch.equal(getattr(one, name)[0], getattr(whole, name)[b]), (name, b)
