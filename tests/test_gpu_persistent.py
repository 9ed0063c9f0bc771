"""rr_sparse_attn with a row queue (persistent workgroups that draw rows from per-XCD counters) against the
same launch without one (a workgroup per row): the same per-row arithmetic, so every result is equal bit for
bit.  The oracle comparison of both is in the parity tests; here the scheduling is what is tested: more rows
than workgroups, rows left out of the order, lengths that end inside a block, steps, repeated launches."""
import dataclasses

import numpy as np
import pytest
import torch

import rr_inputs as ri
import gpu_util as gu

pytestmark = pytest.mark.gpu


def rr():
    import paper_2602_05853_amd as p
    return p


def _draws(rows, Nb, several=1):
    """The call's rows are drawn from the queue: more rows than workgroups, which are one per compute unit where eight waves
    take a row (up to 15 rows per key block and 64, as the launch decides), two otherwise."""
    per_unit = 1 if rows <= min(15 * Nb + 64, 5000) else 2
    assert rows >= several * per_unit * torch.cuda.get_device_properties(0).multi_processor_count, (rows, Nb)


def _both(p, t, mask, L=None, Lq=None):
    """O and lse with the queue and without it."""
    Q = t["Q"]
    out = []
    for m in (mask, dataclasses.replace(mask, queue=None)):
        O = torch.full_like(Q, float("nan"))
        lse = torch.full((Q.shape[0], Q.shape[1], Q.shape[2]), float("nan"), dtype=torch.float32, device=Q.device)
        p.rr_sparse_attn(Q, t["K"], t["V"], m, O=O, lse=lse)
        torch.cuda.synchronize()
        out.append((O, lse))
    return out


# rows of four waves and of eight, lengths that end inside a block, and (the last) a call of so few rows that none is drawn
@pytest.mark.parametrize("L,Hq,Hkv,tau", [(16384, 8, 2, 0.85), (16384 - 37, 8, 2, 0.9), (8192, 32, 8, 0.95),
                                          (6000, 28, 4, 0.9), (3000, 16, 4, 0.9), (2048, 4, 4, 0.9)])
def test_queue_launch_equals_row_per_workgroup_launch(L, Hq, Hkv, tau):
    p = rr()
    w = ri.custom(L=L, Hq=Hq, Hkv=Hkv, d=128, dtype="bf16", B=128, S=16, seed=77, logit_gain=3.0)
    t = gu.to_device(ri.generate(w), w.dtype)
    mask = p.rr_estimate(t["Q"], t["K"], w.S, w.B, tau)
    torch.cuda.synchronize()
    assert mask.queue is not None and mask.queue.numel() == p.binding.RR_QUEUE_WORDS
    assert int(mask.queue.abs().sum().item()) == 0
    print(f"[persistent] L={L} {Hq}/{Hkv} heads: {Hq * ((L + 127) // 128)} rows", flush=True)
    if L != 2048:
        _draws(Hq * w.Nb, w.Nb)
    for rep in range(3):                                    # the launch leaves the queue ready for the next one
        (O1, l1), (O2, l2) = _both(p, t, mask)
        assert int(mask.queue.abs().sum().item()) == 0, rep
        assert not torch.isnan(O1).any() and not torch.isnan(l1).any()
        assert torch.equal(O1, O2) and torch.equal(l1, l2), rep


@pytest.mark.parametrize("Hq,Hkv", [(8, 2), (32, 2)])
def test_queue_launch_skips_rows_left_out_of_the_order(Hq, Hkv):
    """Rows of eight waves and of four; the runs of entries that name no row lie behind the rows that the workgroups start
    with, so that each is drawn from the queue and live rows are drawn after it."""
    p = rr()
    w = ri.custom(L=8192, Hq=Hq, Hkv=Hkv, d=128, dtype="bf16", B=128, S=16, seed=78, logit_gain=3.0)
    t = gu.to_device(ri.generate(w), w.dtype)
    mask = p.rr_estimate(t["Q"], t["K"], w.S, w.B, 0.9)
    torch.cuda.synchronize()
    _draws(Hq * w.Nb, w.Nb, several=2)
    order = mask.row_order.cpu().numpy()[0]
    N = w.G * w.Nb
    runs = [(0, 3, 40), (0, N // 2 + 20, N // 2 + 70), (1, N // 2 + 5, N // 2 + 60), (1, N - 30, N - 2)]
    bad = mask.row_order.clone()
    for kv, lo, hi in runs:
        bad[0, kv, lo:hi] = -1 if lo % 2 else N
    O = torch.zeros_like(t["Q"])
    p.rr_sparse_attn(t["Q"], t["K"], t["V"], dataclasses.replace(mask, row_order=bad), O=O)
    torch.cuda.synchronize()
    assert int(mask.queue.abs().sum().item()) == 0
    ref = p.rr_sparse_attn(t["Q"], t["K"], t["V"], dataclasses.replace(mask, queue=None))
    torch.cuda.synchronize()
    skipped = {(kv * w.G + int(v) // w.Nb, int(v) % w.Nb) for kv, lo, hi in runs for v in order[kv][lo:hi]}
    for h in range(w.Hq):
        for m in range(w.Nb):
            blk = O[0, h, m * w.B:(m + 1) * w.B]
            if (h, m) in skipped:
                assert bool((blk == 0).all()), (h, m)
            else:
                assert torch.equal(blk, ref[0, h, m * w.B:(m + 1) * w.B]), (h, m)


@pytest.mark.parametrize("Hq,Hkv,Lq", [(16, 4, 3045), (32, 2, 6045)])
def test_queue_launch_on_a_step_that_starts_inside_a_block(Hq, Hkv, Lq):
    p = rr()
    w = ri.custom(L=8192, Hq=Hq, Hkv=Hkv, d=128, dtype="bf16", B=128, S=16, seed=79, logit_gain=3.0)
    t = gu.to_device(ri.generate(w), w.dtype)
    q0 = 8192 - Lq
    ts = {"Q": t["Q"][:, :, q0:].contiguous(), "K": t["K"], "V": t["V"]}
    mask = p.rr_estimate(ts["Q"], ts["K"], w.S, w.B, 0.9, flags=0)
    torch.cuda.synchronize()
    _draws(Hq * (w.Nb - q0 // w.B), w.Nb)
    (O1, l1), (O2, l2) = _both(p, ts, mask)
    assert int(mask.queue.abs().sum().item()) == 0
    assert not torch.isnan(O1).any() and not torch.isnan(l1).any()
    assert torch.equal(O1, O2) and torch.equal(l1, l2)


@pytest.mark.parametrize("L,Lq", [(128 * 18, 128 * 18), (128 * 64 + 1, 128 * 16 + 2), (128 * 40 - 3, 128 * 15 + 7)])
def test_two_tiles_per_block_at_the_edges_of_rows_and_launches(L, Lq):
    """Rows whose only block is the diagonal one, rows of every small count, lengths that end one position into a
    block and steps that start inside one: 32 heads make at least 512 rows, which the queue form takes.  Checked
    against attention in fp32 with P and O rounded to bf16 nowhere: an output is off by at most the rounding of P
    and of O, each at most 2^-8 and 0.58 of that in the mean square of terms rounded either way, of a convex
    combination of values below 6: 2.4e-2, plus fp32 sums.  The log-sum-exp is that of a sum of rounded terms,
    log(1 + 2^-8) at most."""
    p = rr()
    g = torch.Generator(device="cuda:0").manual_seed(L)
    Q, K, V = (torch.randn(1, h, n, 128, generator=g, device="cuda:0").bfloat16() for h, n in ((32, Lq), (8, L), (8, L)))
    Nb, q0 = -(-L // 128), L - Lq
    rows = Nb - q0 // 128
    m = torch.arange(Nb - rows, Nb, device="cuda:0")[:, None]
    n = torch.arange(Nb, device="cuda:0")[None]
    dense = (torch.rand(1, 32, rows, Nb, generator=g, device="cuda:0") < 0.3).to(torch.uint8)
    dense |= (n == m).to(torch.uint8)                                  # every query sees itself
    dense[0, ::3] = (n == m).to(torch.uint8)                           # rows of the diagonal block alone
    dense[0, 1::3, :, :] |= ((n == m - 1) | (n == 0)).to(torch.uint8)
    _draws(32 * rows, Nb)
    mask = p.rr_mask_from_dense(Q, K, dense, 128)
    (O1, l1), (O2, l2) = _both(p, {"Q": Q, "K": K, "V": V}, mask)
    assert int(mask.queue.abs().sum().item()) == 0
    assert torch.equal(O1, O2) and torch.equal(l1, l2)
    qpos = torch.arange(q0, L, device="cuda:0")
    kpos = torch.arange(L, device="cuda:0")
    for h in range(0, 32, 5):
        keep = dense[0, h].bool()[qpos // 128 - q0 // 128][:, kpos // 128] & (kpos[None] <= qpos[:, None])
        s = (Q[0, h].float() @ K[0, h // 4].float().T / 128 ** 0.5).masked_fill(~keep, float("-inf"))
        ref = torch.softmax(s, 1) @ V[0, h // 4].float()
        assert (O1[0, h].float() - ref).abs().max().item() <= 2.5e-2, h
        assert (l1[0, h] - torch.logsumexp(s, 1)).abs().max().item() <= 2.0 ** -8 + 1e-5, h


def test_queue_launch_over_long_runs_of_ranks_without_work():
    """Behind the first row of every workgroup come long runs of ranks that name no row, some followed by rows
    that selected nothing: a workgroup then draws one ticket after the other with little in between, and all its waves
    must follow each of them.  2048 rows against at most two workgroups per compute unit."""
    p = rr()
    L, Hq, Hkv, B = 8192, 32, 8, 128
    Nb, G = L // B, Hq // Hkv
    resident = 2 * torch.cuda.get_device_properties(0).multi_processor_count
    _draws(Hq * Nb, Nb, several=2)
    g = torch.Generator(device="cuda:0").manual_seed(80)
    Q, K, V = (torch.randn(1, h, L, 128, generator=g, device="cuda:0").bfloat16() for h in (Hq, Hkv, Hkv))
    dense = torch.zeros(1, Hq, Nb, Nb, dtype=torch.uint8, device="cuda:0")
    n = torch.arange(Nb, device="cuda:0")
    dense[0, :, n, n] = 1
    dense[0, 1::4, n, 0] = 1
    dense[0, 2::4] = 0                                      # rows without a block
    mask = p.rr_mask_from_dense(Q, K, dense, B)
    first = resident // Hkv                                 # order entries that the workgroups start with
    order = torch.arange(G * Nb, dtype=torch.int32, device="cuda:0").repeat(Hkv, 1)
    order = order.reshape(Hkv, G, Nb).transpose(1, 2).reshape(Hkv, G * Nb).contiguous()     # empty rows between others
    order[:, first:first + 40] = -1
    order[:, first + 41:first + 60] = G * Nb
    order[:, first + 70:first + 100:2] = -7
    mask.row_order.copy_(order[None])
    named = torch.zeros(Hkv, G * Nb, dtype=torch.bool, device="cuda:0")
    for kv in range(Hkv):
        ok = order[kv][(order[kv] >= 0) & (order[kv] < G * Nb)]
        named[kv, ok.long()] = True
    named = named.reshape(Hq, Nb).repeat_interleave(B, 1)[None, :, :, None]
    ref = p.rr_sparse_attn(Q, K, V, dataclasses.replace(mask, queue=None, row_order=None))
    for rep in range(5):
        O = torch.full_like(Q, 7.0)
        p.rr_sparse_attn(Q, K, V, mask, O=O)
        torch.cuda.synchronize()
        assert int(mask.queue.abs().sum().item()) == 0, rep
        assert torch.equal(O, torch.where(named, ref, torch.full_like(ref, 7.0))), rep
