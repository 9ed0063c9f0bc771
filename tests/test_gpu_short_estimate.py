"""The estimate of short contexts in one launch (scores of all key strides in registers, selection in the same kernel) against
the general path, two sweeps over the key tiles and a selection kernel, which serves the same call when it names its
sequences (one sequence of all blocks).  Every number of sampled queries to a block, tiles a wave holds (1, 2, 4), groups of
heads that do not divide a workgroup's rows, lengths that end inside a block and inside a stride, offsets and protections."""
import pytest
import torch

import gpu_util as gu

pytestmark = pytest.mark.gpu

# R = 128 / S, L, Hq, Hkv, batch: one tile, eight tiles and one more, sixteen and one more, the most; a block and less
CASES = [(4, 100, 4, 2, 1), (4, 8192, 6, 2, 1), (4, 8193, 3, 3, 2), (4, 16500, 2, 1, 1), (4, 32768, 4, 2, 1),
         (8, 128, 8, 2, 3), (8, 4096, 8, 2, 1), (8, 4100, 7, 1, 2), (8, 8300, 5, 1, 1), (8, 16384, 4, 4, 1), (8, 15001, 14, 2, 1),
         (16, 1000, 6, 3, 1), (16, 2049, 12, 4, 1), (16, 4097, 9, 3, 1), (16, 8192, 4, 1, 1),
         (32, 130, 2, 2, 1), (32, 1025, 7, 1, 1), (32, 2050, 6, 2, 1), (32, 4096, 3, 1, 2)]


@pytest.mark.parametrize("R,L,Hq,Hkv,batch", CASES)
def test_one_launch_agrees_with_two_sweeps(R, L, Hq, Hkv, batch):
    import paper_2602_05853_amd as rr
    dev, B, tau = "cuda:0", 128, 0.9
    S, Nb = B // R, -(-L // B)
    g = torch.Generator(device=dev).manual_seed(100 * R + L)
    Q = torch.randn(batch, Hq, L, 128, generator=g, device=dev)
    K = torch.randn(batch, Hkv, L, 128, generator=g, device=dev)
    u = torch.randn(128, generator=g, device=dev)
    K[:, :, : max(1, L // 5)] += 1.5 * u                    # some blocks draw far more mass than others
    Q = (Q + 0.5 * u).bfloat16()
    K = K.bfloat16()
    opts = [dict(), dict(flags=0, offset_mode="hybrid", layer=5, sink_blocks=1, recent_blocks=2)]
    for more in opts:
        print(f"[short estimate] R={R} L={L} {Hq}/{Hkv} x {batch} {more}", flush=True)
        got, ref = (rr.BlockMask.allocate(batch, Hq, Nb, B, dev, block_mass=True, Hkv=Hkv) for _ in range(2))
        rr.rr_estimate(Q, K, S, B, tau, out=got, **more)
        rr.rr_estimate(Q, K, S, B, tau, out=ref, seq_first=torch.zeros(Nb, dtype=torch.int32, device=dev), **more)
        torch.cuda.synchronize()
        # A mass is a sum of exponentials of scores below 2^7 in log2 units, rounded to 2^-17, and of up to 1024 terms: either
        # form is within 2^-17 of its value; the fractions of a row add up to one.
        a, b = got.block_mass.double(), ref.block_mass.double()
        assert ((a - b).abs() <= 2.0 ** -16 * b + 2.0 ** -24).all()
        # lists, counts and dense rows describe one mask
        n = torch.arange(Nb, device=dev)
        assert torch.equal(got.dense.sum(-1).int(), got.row_count)
        listed = torch.zeros_like(got.dense)
        live = n < got.row_count[..., None]
        listed.scatter_add_(-1, torch.where(live, got.row_list, 0).long(), live.to(torch.uint8))
        assert torch.equal(listed, got.dense)
        # rows that differ meet tau, or the next mass, to rounding
        for i in (got.dense != ref.dense).any(-1).nonzero():
            row = b[tuple(i)].sort(descending=True).values
            cum = row.cumsum(0)
            k = int(ref.row_count[tuple(i)])
            near = (cum - tau).abs().min() < 2.0 ** -15
            tied = k < Nb and float(row[k - 1] - row[k]) <= 2.0 ** -15 * float(row[k - 1])
            assert near or tied, (i.tolist(), cum[k - 1].item())


# steps whose heads hold a sampled query only in part, or not at all (those that complete no stride): workgroups of 64 / R rows without a
# single one skip the scores, with others that do not
@pytest.mark.parametrize("R,L,Lq,Hq,Hkv,batch", [(4, 32000 + 3, 3, 32, 8, 1), (4, 32000, 9, 64, 2, 1), (8, 16007, 1, 8, 2, 2), (8, 16000, 3, 32, 2, 1),
                                                 (16, 8003, 2, 8, 1, 1), (16, 4000, 1, 16, 2, 1), (32, 4002, 1, 8, 2, 1), (32, 2004, 2, 8, 1, 3)])
def test_steps_with_few_sampled_queries(R, L, Lq, Hq, Hkv, batch):
    import paper_2602_05853_amd as rr
    dev, B, tau = "cuda:0", 128, 0.9
    S, Nb, q0, G = B // R, -(-L // B), L - Lq, Hq // Hkv
    g = torch.Generator(device=dev).manual_seed(L + Lq)
    Q = (2.0 * torch.randn(batch, Hq, Lq, 128, generator=g, device=dev)).bfloat16()
    K = (torch.randn(batch, Hkv, L, 128, generator=g, device=dev) + 2.0 * (torch.arange(L, device=dev) < L // 5)[:, None]).bfloat16()
    rows = Nb - q0 // B
    mask = rr.BlockMask.allocate(batch, Hq, Nb, B, dev, block_mass=True, Hkv=Hkv, rows=rows)
    mask.block_mass.fill_(float("nan"))
    mask.dense.fill_(7)
    print(f"[short step] R={R} {Lq} of {L} {Hq}/{Hkv} x {batch}", flush=True)
    rr.rr_estimate(Q, K, S, B, tau, flags=0, out=mask)
    torch.cuda.synchronize()
    n = torch.arange(Nb, device=dev)
    held = 0
    for b in range(batch):
        for h in range(Hq):
            ref = gu.stride_masses(Q[b, h], K[b, h // G], S, B, q0, h)
            assert ((mask.block_mass[b, h].double() - ref).abs() <= 2.0 ** -16 * ref + 2.0 ** -24).all()
            for r in range(rows):
                kept, m = mask.dense[b, h, r], q0 // B + r
                if not bool(ref[r].any()):
                    assert torch.equal(kept.bool(), n <= m) and int(kept.max()) == 1
                    continue
                held += 1
                a, rest = ref[r][kept.bool()], ref[r][~kept.bool()]
                assert a.sum() >= tau - 1e-5 and a.sum() - a.min() < tau + 1e-5 and (rest <= a.min() * (1 + 2.0 ** -15)).all()
    sampled = sum(i * S + S - 1 - h % S >= q0 for h in range(Hq) for i in range(q0 // S, L // S))
    assert (held > 0) == (sampled > 0)
