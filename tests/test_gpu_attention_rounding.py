"""Rounding of the probabilities in the bf16 d = 128 attention kernel: one key outweighs the others by a factor that bf16
holds worst (2^k (1 + 0.9 / 256), rounded down by delta = 0.35 %), all rows alike, so that the error of a result does not
average out over the rows.  The key comes after a step of keys that set the softmax reference: inside the diagonal block,
where a row is that block alone, and, in a chunk of a longer context with the workspace, in a block of the pipeline.

Bound.  The denominator sums the rounded probabilities, so the error of the large weight w leaves delta (1 - w): in the
first case 1 - w <= 1/17, 2.1e-4.  In the chunk a weight more than 2^6 above the reference becomes the reference and is
exact; of the other 255 keys the 58 at most that come after it are rounded, by 2^-9: 3.6e-4 of the sum.  A channel's last
rounding is at most 2^-8, 0.58 of that in the mean square, and the mean of 128 channels of random mantissas is off by 4 x 0.58 x 2^-8 / sqrt(128) = 8e-4 at most.  A weight that is
rounded in the numerator alone is off by 3e-3, one that stays as far above the reference by 2.3e-3."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


def _factors(bits):
    """two bf16 numbers whose product is a score of log2 = bits after the scale by 1 / sqrt(128)"""
    want = bits * math.log(2.0) * math.sqrt(128.0)
    best = None
    for i in range(128, 256):
        for e in (1, 2, 4, 8):
            x = i / 128.0 * e
            y = float(torch.tensor(want / x).bfloat16())
            if best is None or abs(x * y - want) < best[0]:
                best = (abs(x * y - want), x, y)
    assert best[0] / math.sqrt(128.0) * 1.4427 < 4e-4, best
    return best[1], best[2]


CASES = ([("diagonal", k, f) for k in (4, 7) for f in ("plain", "queue", "ragged")] +
         [("pipeline", k, "parts") for k in (6, 7)])


@pytest.mark.parametrize("case,k,form", CASES)
def test_large_weights_are_not_rounded_alone(case, k, form):
    import paper_2602_05853_amd as rr
    dev, heads = "cuda:0", 32 if form == "queue" else 2
    Nb = 130 if form == "parts" else 32
    L = 128 * Nb - (5 if form == "ragged" else 0)
    Lq = 600 if form == "parts" else L
    qx, ky = _factors(k + math.log2(1 + 0.9 / 256))
    g = torch.Generator(device=dev).manual_seed(k)
    Q = torch.zeros(1, heads, Lq, 128, device=dev)
    K, V = (torch.zeros(1, heads, L, 128, device=dev) for _ in range(2))
    Q[..., 0] = qx
    v = 1 + torch.rand(128, generator=g, device=dev).bfloat16().float()
    rows = Nb - (L - Lq) // 128
    dense = torch.zeros(1, heads, rows, Nb, dtype=torch.uint8, device=dev)
    if case == "diagonal":
        n = torch.arange(Nb, device=dev)
        dense[0, :, n, n] = 1
        K[..., 0] = -1e4
        first = torch.arange(0, L, 128, device=dev)
        K[:, :, first, 0] = 0.                              # the block's first key sets the reference
        at = first + 40                                     # its second step brings the large one
        seen = torch.arange(L, device=dev) % 128 >= 64
    else:
        dense[..., 0] = 1                                   # 128 keys of weight 1, then the block of the large one
        dense[..., 1] = 1
        at = torch.tensor([128 + 70], device=dev)
        seen = torch.ones(Lq, dtype=torch.bool, device=dev)
    K[:, :, at, 0] = ky
    V[:, :, at] = v
    Q, K, V = Q.bfloat16(), K.bfloat16(), V.bfloat16()
    mask = rr.rr_mask_from_dense(Q, K, dense, 128)
    if form != "queue":
        mask.queue = None
    ws = None
    if form == "parts":
        need = rr.rr_attn_workspace_bytes(Q, K, 128)
        assert need > 0
        ws = torch.empty(need, dtype=torch.uint8, device=dev)
    lse = torch.empty(1, heads, Lq, dtype=torch.float32, device=dev)
    O = rr.rr_sparse_attn(Q, K, V, mask, lse=lse, workspace=ws)
    torch.cuda.synchronize()
    score = float(Q[0, 0, 0, 0]) * float(K[0, 0, int(at[0]), 0]) / math.sqrt(128.0)
    total = math.exp(score) + (1 if case == "diagonal" else 255)
    off = (O[0][:, seen].double() / (math.exp(score) / total * V[0, 0, int(at[0])].double())).mean(-1) - 1
    lse_off = (lse[0][:, seen].double() - math.log(total)).abs().max().item()
    print(f"[rounding] {case} 2^{k} {form}: mean error {off.abs().max().item():.2e}, lse {lse_off:.1e}", flush=True)
    assert off.abs().max().item() <= (2.1e-4 if case == "diagonal" else 3.6e-4) + 8e-4
    # the diagonal block's terms are known unrounded: fp32 sums and exponentials of scores of magnitude 5
    assert lse_off <= (1e-5 if case == "diagonal" else 3.6e-4)
