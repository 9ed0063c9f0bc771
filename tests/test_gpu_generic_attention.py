"""Attention on the path for every shape that is not bf16, d = 128, B = 128: block sizes and head widths at the edges
of its tiles (16 queries or 32, 16 keys, channels in chunks of 16 and 32), both types, lengths that end inside a
block and inside a tile, rows with no block, one block, a block other than the diagonal one only, against the
oracle's attention under the same mask."""
import numpy as np
import pytest
import torch

import gpu_util as gu
from oracle import rr_oracle as oracle

pytestmark = pytest.mark.gpu

# B, d: blocks shorter than a tile, one past a tile, three tiles, the largest; widths of half a chunk, of every piece of
# a row a lane may load (16, 32, 64, 128 channels), the widest
SHAPES = [(1, 8), (7, 8), (15, 40), (16, 24), (17, 16), (31, 56), (32, 256), (33, 136), (48, 80), (64, 64), (64, 128),
          (128, 48), (100, 72), (24, 232), (36, 200), (40, 112)]


def _inputs(L, Hq, Hkv, d, dtype, seed):
    rng = np.random.default_rng(seed)
    x = {"Q": 2.0 * rng.standard_normal((Hq, L, d)), "K": rng.standard_normal((Hkv, L, d)),
         "V": rng.standard_normal((Hkv, L, d))}
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    return {k: torch.from_numpy(v.astype(np.float32)).to(tdt).float().numpy() for k, v in x.items()}


# launches of 512 workgroups and more: more queries to a workgroup (64 for narrow bf16 heads, 32 for fp32)
LARGE = [(40, 64, "bf16"), (64, 40, "bf16"), (128, 16, "bf16"), (48, 72, "bf16"), (33, 128, "f32"), (64, 24, "f32")]


@pytest.mark.parametrize("B,d,dtype,Hq,Nb", [(B, d, t, 4, 9) for B, d in SHAPES for t in ("bf16", "f32")] +
                         [(B, d, t, 16, 33) for B, d, t in LARGE])
def test_generic_attention_matches_the_oracle(B, d, dtype, Hq, Nb):
    import paper_2602_05853_amd as rr
    L = Nb * B - B // 3
    x = _inputs(L, Hq, Hq // 2, d, dtype, seed=1000 * B + d)
    rng = np.random.default_rng(B + d)
    mask = np.tril(rng.random((Hq, Nb, Nb)) < 0.5).astype(np.uint8)
    mask[:, Nb - 1] = 1                                     # the protected last row
    mask[1, 4] = 0                                          # a row with nothing selected
    mask[2, 5], mask[2, 5, 5] = 0, 1                        # the diagonal block alone
    mask[3, 6], mask[3, 6, 2] = 0, 1                        # one block, not the diagonal one
    t = gu.to_device(x, dtype, layout="blhd" if B % 3 == 0 else "bhld")     # two sets of strides
    print(f"[generic] B={B} d={d} {dtype} L={L}", flush=True)
    O = torch.full_like(t["Q"], float("nan"))
    lse = torch.full(t["Q"].shape[:3], float("nan"), dtype=torch.float32, device="cuda:0")
    rr.rr_sparse_attn(t["Q"], t["K"], t["V"], gu.blockmask_from_dense(mask, B), O=O, lse=lse)
    torch.cuda.synchronize()
    want, want_lse = oracle.sparse_attention(x["Q"], x["K"], x["V"], mask, B)
    worst, mean = gu.attention_errors(O[0], want)
    got_lse = lse[0].cpu().numpy()
    empty = np.isinf(want_lse)
    assert np.array_equal(empty, np.isneginf(got_lse))
    lse_err = np.abs(got_lse[~empty] - want_lse[~empty]).max()
    if dtype == "bf16":
        assert worst <= gu.BF16_MAX_ABS and mean <= gu.BF16_MEAN_ABS
    else:
        assert worst <= gu.F32_MAX_ABS
    # the scores and their sum are formed in 32 bits for both types
    assert lse_err <= gu.F32_MAX_ABS


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_more_query_blocks_than_a_grid_axis_holds(dtype):
    """Blocks of one position, 66 000 of them, dense: rows around the 65 535th from either end and a sample of others
    against attention in 64 bits (weights of thousands of keys: the output is a mean, of magnitude 0.01 and more)."""
    import paper_2602_05853_amd as rr
    dev, L, d = "cuda:0", 66000, 8
    g = torch.Generator(device=dev).manual_seed(3)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    Q, K, V = (torch.randn(1, 1, L, d, generator=g, device=dev).to(tdt) for _ in range(3))
    print(f"[generic] {L} blocks of one position, {dtype}", flush=True)
    O = torch.full_like(Q, float("nan"))
    lse = torch.full((1, 1, L), float("nan"), device=dev)
    rr.rr_dense_attn(Q, K, V, 1, O=O, lse=lse)
    torch.cuda.synchronize()
    assert torch.isfinite(O.float()).all() and torch.isfinite(lse).all()
    rows = sorted({0, 1, 463, 464, 465, 466, 65534, 65535, 65536, L - 1} | set(range(777, L, 4999)))
    for r in rows:
        s = K[0, 0, :r + 1].double() @ Q[0, 0, r].double() / d ** 0.5
        want = torch.softmax(s, 0) @ V[0, 0, :r + 1].double()
        off = (O[0, 0, r].double() - want).abs()
        assert (off <= (2.0 ** -8 if dtype == "bf16" else 0.0) * want.abs() + gu.F32_MAX_ABS).all(), r
        assert (lse[0, 0, r].double() - torch.logsumexp(s, 0)).abs() <= gu.F32_MAX_ABS, r
