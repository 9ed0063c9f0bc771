"""Estimate of short steps deep in a context (one sweep over the key strides, softmax and selection in a second launch): block masses
against the method in 64 bits, the selection against those masses, the row order against the one made from the finished mask.
Masses are sums of at most some thousand fp32 terms of exact products: 2^-24 times the logits' spread (below 64) and the
additions' depth, within 1e-5 of the row.

Which form a call takes is a rule on its shape.  The two sweeps leave the softmax states of their key chunks at the end of the
workspace, and the last chunk of the last KV head writes its 2 KB whatever it holds; the sums of the one sweep end before
them in every shape here.  So bytes set beforehand tell the two apart, and each test says which one it is about."""
import pytest
import torch

import gpu_util as gu

pytestmark = pytest.mark.gpu

B = 128


def _context(batch, Hq, Hkv, L, Lq, seed):
    g = torch.Generator(device="cuda:0").manual_seed(seed)
    K = torch.randn(batch, Hkv, L, 128, generator=g, device="cuda:0")
    K = (K + 2.0 * torch.randn(batch, Hkv, -(-L // 512), 128, generator=g, device="cuda:0").repeat_interleave(512, 2)[:, :, :L]).bfloat16()
    return (2.0 * torch.randn(batch, Hq, Lq, 128, generator=g, device="cuda:0")).bfloat16(), K


def _dirty(Q, K, S, batch, Hq, Hkv, L, Lq):
    """a workspace of set bytes and a mask whose every array holds garbage"""
    import paper_2602_05853_amd as rr
    ws = torch.full((rr.rr_workspace_bytes(Q, K, S, B),), 0xFF, dtype=torch.uint8, device=Q.device)
    Nb = -(-L // B)
    out = rr.BlockMask.allocate(batch, Hq, Nb, B, Q.device, block_mass=True, Hkv=Hkv, rows=Nb - (L - Lq) // B)
    for t in (out.row_count, out.row_list, out.row_order, out.queue):
        t.fill_(0x7A7A7A7A)
    out.dense.fill_(0x7A)
    out.block_mass.fill_(float("nan"))
    return ws, out


def _one_sweep(ws):
    return bool((ws[-2048:] == 0xFF).all())


PLAIN, HYBRID = {}, dict(offset_mode="hybrid", layer=5, sink_blocks=2, recent_blocks=3)


# batch, Hq, Hkv, L, Lq, S: every R = 128 / S; one row and two, up to 64 tiles of key strides to 1024 blocks; the last two hold no
# sampled query at all
@pytest.mark.parametrize("batch,Hq,Hkv,L,Lq,S,more",
                         [(1, 8, 2, 128 * 300, 8, 16, PLAIN), (1, 8, 1, 128 * 1024, 3, 16, PLAIN), (1, 14, 2, 128 * 600 + 3, 30, 16, PLAIN),
                          (2, 4, 2, 128 * 300 + 16, 16, 16, HYBRID), (1, 8, 2, 128 * 700 + 30, 60, 16, PLAIN),
                          (1, 16, 8, 128 * 700 + 64, 80, 16, HYBRID),
                          (1, 8, 2, 128 * 130 + 40, 9, 8, PLAIN), (1, 8, 2, 128 * 300 + 8, 24, 8, HYBRID), (2, 8, 2, 128 * 600 + 5, 17, 8, PLAIN),
                          (1, 8, 2, 128 * 512, 32, 32, PLAIN), (1, 8, 2, 128 * 512 + 32, 64, 32, HYBRID), (2, 8, 2, 128 * 260, 33, 32, PLAIN),
                          (1, 32, 8, 128 * 66 + 1, 5, 4, PLAIN), (2, 8, 2, 128 * 140 + 2, 9, 4, HYBRID), (1, 8, 2, 128 * 1024, 12, 4, PLAIN),
                          (1, 4, 1, 128 * 400 + 20, 16, 16, PLAIN), (1, 4, 4, 128 * 257 - 19, 1, 16, PLAIN), (1, 4, 1, 128 * 400 + 20, 4, 16, PLAIN)])
@pytest.mark.parametrize("tau", [0.9, 1.0])
def test_step_estimate(batch, Hq, Hkv, L, Lq, S, more, tau):
    import paper_2602_05853_amd as rr
    q0, G, Nb = L - Lq, Hq // Hkv, -(-L // B)
    m0 = q0 // B
    rows = Nb - m0
    Q, K = _context(batch, Hq, Hkv, L, Lq, L + Lq)
    ws, mask = _dirty(Q, K, S, batch, Hq, Hkv, L, Lq)
    print(f"[step] {batch} x {Hq}/{Hkv} heads, {Lq} of {L}, S {S}, tau {tau}, {more}", flush=True)
    rr.rr_estimate(Q, K, S, B, tau, flags=0, out=mask, workspace=ws, **more)
    torch.cuda.synchronize()
    assert _one_sweep(ws)
    ref = torch.stack([torch.stack([gu.stride_masses(Q[b, h], K[b, h // G], S, B, q0,
                                                     (h + 5 if more else h)) for h in range(Hq)]) for b in range(batch)])
    got = mask.block_mass.double()
    assert (got - ref).abs().max() <= 1e-5
    sampled = ref.sum(-1) > 0.5
    n = torch.arange(Nb, device="cuda:0")
    m = m0 + torch.arange(rows, device="cuda:0")[:, None]
    causal = n[None] <= m
    forced = causal & ((n[None] < more.get("sink_blocks", 0)) | (n[None] > m - more.get("recent_blocks", 0)))
    assert int(mask.dense.max()) <= 1
    kept = mask.dense.bool()
    assert not (kept & ~causal).any()
    all_rows = causal.expand(batch, Hq, -1, -1)
    if tau == 1.0:
        assert torch.equal(kept, all_rows)
    assert torch.equal(kept[~sampled], all_rows[~sampled])
    assert (kept | ~forced).all()
    for b, h, r in (sampled.nonzero().tolist() if tau < 1.0 else []):
        mass, k = got[b, h, r], kept[b, h, r]
        if not more:
            a, rest = mass[k], mass[~k]
            assert a.sum() >= tau - 1e-5 and (a.sum() - a.min() < tau + 1e-5) and (rest.numel() == 0 or rest.max() <= a.min())
        else:
            # the shortest prefix by mass reaches tau, and the forced blocks come on top
            top, at = mass.sort(descending=True, stable=True)
            cum = top.cumsum(0)
            size = int((cum < tau).sum()) + 1
            base = torch.zeros_like(k)
            base[at[:size]] = True
            off = (k != (base | forced[r])).nonzero().flatten()
            assert off.numel() == 0 or (cum - tau).abs().min() < 1e-5, (b, h, r, off.tolist())
    count = mask.row_count
    assert torch.equal(count, mask.dense.sum(-1).int())
    for b, h, r in (count >= 0).nonzero().tolist():
        assert torch.equal(mask.row_list[b, h, r, :int(count[b, h, r])].long(), kept[b, h, r].nonzero().flatten())
    again = rr.rr_mask_from_dense(Q, K, mask.dense, B)
    assert torch.equal(again.row_order, mask.row_order) and not mask.queue.any()


# A block that holds several sampled queries of a head, one of them not finite: the row's mass is unknown, so it keeps every block, in
# every form of the estimate (`sweeps`: False for the short steps of this file and for a short context in one launch); rows of
# other heads and blocks are what they are without it.
@pytest.mark.parametrize("Hq,Hkv,L,Lq,S,sweeps", [(8, 2, 128 * 1024, 12, 4, False), (16, 8, 128 * 700 + 64, 80, 16, False),
                                                  (8, 2, 128 * 300 + 24, 24, 8, False), (8, 2, 128 * 513, 64, 32, False),
                                                  (8, 2, 128 * 60, 130, 16, False), (8, 2, 128 * 140, 300, 16, True)])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_row_with_a_query_that_is_not_finite_keeps_every_block(Hq, Hkv, L, Lq, S, sweeps, value):
    import paper_2602_05853_amd as rr
    Q, K = _context(1, Hq, Hkv, L, Lq, L + Lq)
    q0, m0, h = L - Lq, (L - Lq) // B, Hq - 2
    clean = rr.rr_estimate(Q, K, S, B, 0.9, flags=0, block_mass=True)
    position = lambda i: i * S + S - 1 - h % S - q0                                 # of the sampled query of stride i, in the step
    held = [i for i in range(q0 // S, L // S) if position(i) >= 0]
    row = lambda i: i * S // B - m0
    r = row(held[-1])
    assert sum(row(i) == r for i in held) >= 2 and int(clean.row_count[0, h, r]) < m0 + r + 1
    Q[0, h, position(held[-1]), 17] = value
    ws, mask = _dirty(Q, K, S, 1, Hq, Hkv, L, Lq)
    print(f"[step] {Hq}/{Hkv} heads, {Lq} of {L}, S {S}: query {value} in row {r} of head {h}", flush=True)
    rr.rr_estimate(Q, K, S, B, 0.9, flags=0, out=mask, workspace=ws)
    torch.cuda.synchronize()
    assert _one_sweep(ws) != sweeps
    n = torch.arange(mask.Nb, device="cuda:0")
    assert torch.equal(mask.dense[0, h, r].bool(), n <= m0 + r) and int(mask.row_count[0, h, r]) == m0 + r + 1
    others = torch.ones(mask.row_count.shape, dtype=torch.bool, device="cuda:0")
    others[0, h, r] = False
    for a, b in ((mask.dense, clean.dense), (mask.row_count, clean.row_count), (mask.block_mass, clean.block_mass)):
        assert torch.equal(a[others], b[others])


def _new_strides(S, known, L, Lq):
    """The stride sums of the first `known` positions are in the workspace, the step's last query is position L - 1.  As the call that forms
    all sums itself, and what it left is what the next call takes."""
    import paper_2602_05853_amd as rr
    Hq, Hkv = 4, 2
    cap = -(-(L + B) // 4096) * 4096
    g = torch.Generator(device="cuda:0").manual_seed(known + L)
    Q = torch.randn(1, Hq, Lq, 128, generator=g, device="cuda:0").bfloat16()
    K = torch.randn(1, Hkv, L + 1, 128, generator=g, device="cuda:0").bfloat16()
    room = K.new_empty((1, Hkv, cap, 128), device="meta")
    ws = torch.full((rr.rr_workspace_bytes(Q.new_empty((1, Hq, L, 128), device="meta"), room, S, B),), 0xFF, dtype=torch.uint8, device="cuda:0")
    print(f"[new strides] S {S}: {L // S - known // S} behind {known // S}, {Lq} of {L}", flush=True)
    rr.rr_estimate(Q[:, :, :1], K[:, :, :known], S, B, 0.9, flags=0, workspace=ws, ksum_capacity=cap)
    one_sweep = []
    for end in (L, L + 1):
        queries, keys = Q if end == L else Q[:, :, :1], K[:, :, :end]
        kept = rr.rr_estimate(queries, keys, S, B, 0.9, flags=0, workspace=ws, block_mass=True, ksum_capacity=cap, ksum_valid=known if end == L else L)
        own, plain = _dirty(queries, keys, S, 1, Hq, Hkv, end, queries.shape[2])
        rr.rr_estimate(queries, keys, S, B, 0.9, flags=0, out=plain, workspace=own)
        torch.cuda.synchronize()
        one_sweep.append(_one_sweep(own))
        for name in ("row_count", "dense", "block_mass", "row_order"):
            assert torch.equal(getattr(kept, name), getattr(plain, name)), (name, end)
    sums = ws[:3 * Hkv * (cap // S) * 128 * 2].view(torch.bfloat16).view(3, Hkv, cap // S, 128)[:, :, :L // S].double().sum(0)
    ref = K[0, :, :L // S * S].double().view(Hkv, L // S, S, 128).sum(2)
    # three terms of 8 bits hold the 32-bit sum of up to 32 values exactly: its rounding
    assert ((sums - ref).abs() <= 2.0 ** -20 * K[0].double().abs().max() * S).all()
    return one_sweep


# new strides of a step, wherever they lie in a tile of 32 strides and in their block; a context that ends inside a stride.  (Most of
# them have more than 32 strides to the end of their block and are summed by a launch of their own.)
@pytest.mark.parametrize("S", [4, 8, 16, 32])
@pytest.mark.parametrize("first,new,more", [(0, 1, 0), (31, 1, 2), (31, 2, 0), (17, 31, 1), (1, 32, 0), (0, 32, 3), (20, 33, 0)])
def test_new_strides_of_a_step(S, first, new, more):
    """The stride sums are known up to stride `first` of a tile; the step brings `new` more and `more` tokens of the next one."""
    known = (34 * 32 + first) * S
    L = known + new * S + min(more, S - 1)
    _new_strides(S, known, L, min(L - known, 2 * S + 1))


# New strides that are formed where they are scored: `to_end` strides without sums up to the end of the last block, at most 32, of which
# `new` are complete; and one more than 32, which a launch of its own sums.  `blocks` puts that end at a tile's end or inside one, so that the
# strides lie in one tile or two (`tiles`: how many of them in each); up to eight turns of four strides to a wavefront, whole and not.
@pytest.mark.parametrize("S,blocks,to_end,new,more,tiles",
                         [(4, 36, 32, 32, 0, (32,)), (4, 36, 32, 31, 3, (32,)), (4, 36, 32, 17, 1, (32,)), (4, 36, 27, 22, 0, (27,)), (4, 36, 5, 5, 0, (5,)),
                          (4, 36, 33, 33, 0, (1, 32)), (4, 36, 33, 2, 1, (1, 32)),
                          (8, 71, 32, 32, 0, (16, 16)), (8, 71, 32, 17, 5, (16, 16)), (8, 71, 20, 5, 1, (4, 16)), (8, 70, 32, 31, 7, (32,)),
                          (8, 71, 33, 33, 0, (17, 16)), (8, 71, 33, 18, 1, (17, 16)),
                          (16, 139, 32, 32, 0, (8, 24)), (16, 139, 32, 31, 15, (8, 24)), (16, 137, 12, 5, 1, (4, 8)), (16, 139, 22, 17, 3, (22,)),
                          (16, 139, 33, 33, 0, (9, 24)),
                          (32, 275, 32, 32, 0, (20, 12)), (32, 275, 32, 31, 9, (20, 12)), (32, 275, 17, 17, 0, (5, 12)), (32, 275, 7, 5, 31, (7,)),
                          (32, 275, 33, 31, 1, (21, 12))])
def test_new_strides_formed_where_they_are_scored(S, blocks, to_end, new, more, tiles):
    Ls = blocks * B // S
    first = Ls - to_end
    L = (first + new) * S + more
    # the path goes by the strides to the end of the padded last block
    assert -(-L // B) == blocks and more < S and new + (more > 0) <= to_end and Ls > 1024
    assert tuple(min(t + 32, Ls) - max(t, first) for t in range(first // 32 * 32, Ls, 32)) == tiles
    assert _new_strides(S, first * S, L, min(L - first * S, 2 * S + 1))[0]
