"""The estimate of bf16 tensors in two sweeps over the key strides (contexts or launches beyond what one launch takes, steps included
that hold many sampled queries), for every number of sampled queries to a block: unsplit, with the key tiles shared out among workgroups,
and with stride sums kept from call to call.  Which form a call takes is a rule on its shape; the tests tell by what it leaves in
the workspace, whose parts in order are the planes of stride sums, the block masses, the softmax states of a split launch."""
import pytest
import torch

import gpu_util as gu

pytestmark = pytest.mark.gpu

B = 128


def _context(batch, Hq, Hkv, L, Lq, seed):
    g = torch.Generator(device="cuda:0").manual_seed(seed)
    K = torch.randn(batch, Hkv, L, 128, generator=g, device="cuda:0")
    K = (K + 1.5 * torch.randn(batch, Hkv, -(-L // 512), 128, generator=g, device="cuda:0").repeat_interleave(512, 2)[:, :, :L]).bfloat16()
    return (1.5 * torch.randn(batch, Hq, Lq, 128, generator=g, device="cuda:0")).bfloat16(), K


def _parts(batch, Hq, Hkv, L, rows, S):
    """bytes of the planes and of the masses"""
    Nb = -(-L // B)
    pad = lambda n: -(-n // 256) * 256
    return pad(3 * batch * Hkv * (Nb * B // S) * 128 * 2), pad(4 * batch * Hq * rows * Nb)


# R = 128 / S; batch, Hq, Hkv, L, split: prompts of 8 to 15 tiles of key strides by the hundred, and single ones of more than 32 tiles
@pytest.mark.parametrize("R,batch,Hq,Hkv,L,split", [(4, 15, 12, 3, 128 * 64, False), (8, 13, 14, 2, 128 * 48 - 5, False),
                                                    (16, 15, 12, 4, 128 * 15, False), (32, 11, 8, 8, 128 * 15 - 3, False),
                                                    (4, 1, 4, 2, 128 * 300 - 40, True), (8, 2, 3, 1, 128 * 140, True),
                                                    (16, 1, 6, 2, 128 * 70, True), (32, 1, 4, 2, 128 * 36 - 1, True)])
@pytest.mark.parametrize("mode,layer", [("head", 0), ("hybrid", 3)])
def test_block_masses(R, batch, Hq, Hkv, L, split, mode, layer):
    import paper_2602_05853_amd as rr
    S, tau, Nb, G = B // R, 0.9, -(-L // B), Hq // Hkv
    Q, K = _context(batch, Hq, Hkv, L, L, 10 * L + R)
    ws = torch.full((rr.rr_workspace_bytes(Q, K, S, B),), 0xFF, dtype=torch.uint8, device="cuda:0")
    print(f"[sweeps] R {R}: {batch} x {Hq}/{Hkv} heads of {L}, {mode}", flush=True)
    mask = rr.rr_estimate(Q, K, S, B, tau, workspace=ws, block_mass=True, offset_mode=mode, layer=layer)
    torch.cuda.synchronize()
    planes, masses = _parts(batch, Hq, Hkv, L, Nb, S)
    assert not bool((ws[planes:planes + 4] == 0xFF).all())          # the one launch of short contexts leaves no masses there
    assert (ws.numel() > planes + masses) == split
    gu.check_mask_structures(mask)
    n = torch.arange(Nb)
    for b in {0, batch // 2, batch - 1}:
        for h in {0, G - 1, Hq // 2, Hq - 1}:
            ref = gu.stride_masses(Q[b, h], K[b, h // G], S, B, 0, h + layer)
            got = mask.block_mass[b, h].double()
            # sums of at most 1280 fp32 terms 2^(score - reference), scores below 2^7 to 2^-17 of their value: within 2^-16 of a mass
            assert ((got - ref).abs() <= 2.0 ** -16 * ref + 2.0 ** -24).all(), (b, h)
            ref, dense = ref.cpu(), mask.dense[b, h].bool().cpu()
            for m in range(Nb):
                kept = dense[m]
                if m == Nb - 1 or not ref[m].any():
                    assert torch.equal(kept, n <= m)
                    continue
                a, rest = ref[m][kept], ref[m][~kept]
                assert a.sum() >= tau - 1e-5 and a.sum() - a.min() < tau + 1e-5 and (rest <= a.min() * (1 + 2.0 ** -15)).all(), (b, h, m)


@pytest.mark.parametrize("Hq,Hkv,S,batch", [(8, 2, 16, 1), (6, 3, 8, 2), (4, 2, 32, 1), (4, 2, 4, 1)])
def test_kept_stride_sums_deep_in_a_context(Hq, Hkv, S, batch):
    """Planes laid out for more strides than the context has, the leading ones kept, everything behind them of an earlier call: a prompt, chunks
    and short steps beyond 1024 key strides give, bit for bit, what the same call gives when it forms all sums itself."""
    import paper_2602_05853_amd as rr
    first = 1025 * S + 3
    lengths = [first]
    for more in (300, 1, S, 5, 2000 + S // 2, 2 * S + 1, 1, 3, 129, S):
        lengths.append(lengths[-1] + more)
    cap = -(-(lengths[-1] + B) // 4096) * 4096
    Q, K = _context(batch, Hq, Hkv, lengths[-1], lengths[-1], 7 * S + Hq)
    room = K.new_empty((batch, Hkv, cap, 128), device="meta")
    need = max(rr.rr_workspace_bytes(Q.new_empty((batch, Hq, b - a + B, 128), device="meta"), room, S, B) for a, b in zip([0] + lengths, lengths))
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda:0")
    at = 3 * batch * Hkv * (cap // S) * 128 * 2
    forms = set()
    for prev, L in zip([0] + lengths, lengths):
        Qc, Kv = Q[:, :, prev:L].contiguous(), K[:, :, :L]
        if L % 2:
            ws[at:].fill_(0xFF)                              # behind the planes: of the call before, or no numbers
        kept = rr.rr_estimate(Qc, Kv, S, B, 0.9, flags=0, workspace=ws, block_mass=True, ksum_capacity=cap, ksum_valid=prev)
        own = torch.full((rr.rr_workspace_bytes(Qc, Kv, S, B),), 0xFF, dtype=torch.uint8, device="cuda:0")
        plain = rr.rr_estimate(Qc, Kv, S, B, 0.9, flags=0, workspace=own, block_mass=True)
        torch.cuda.synchronize()
        one = bool((own[-2048:] == 0xFF).all())
        forms.add((one, L - prev))
        print(f"[kept sums] S {S}: {L - prev} of {L}, {'one sweep' if one else 'two sweeps'}", flush=True)
        for name in ("row_count", "dense", "block_mass", "row_order"):
            assert torch.equal(getattr(kept, name), getattr(plain, name)), (name, prev, L)
        live = torch.arange(plain.Nb, device="cuda:0") < plain.row_count[..., None]
        assert torch.equal(torch.where(live, kept.row_list, -1), torch.where(live, plain.row_list, -1))
    assert sum(one for one, _ in forms) >= 3 and sum(not one for one, _ in forms) >= 2


# key strides shared out among 7, 8, 9, 31, 33 and 39 workgroups, whose softmax states the second launch reads 8 to 32 at a time
@pytest.mark.parametrize("S,L,parts", [(16, 30000, 7), (16, 128 * 256, 8), (16, 37000, 9), (4, 31800, 31), (4, 33900, 33), (4, 40000, 39)])
def test_states_of_many_parts(S, L, parts):
    import paper_2602_05853_amd as rr
    Hq, Hkv, Lq, Nb = 4, 2, 600, -(-L // B)
    Q, K = _context(1, Hq, Hkv, L, Lq, L + S)
    rows = Nb - (L - Lq) // B
    ws = torch.full((rr.rr_workspace_bytes(Q, K, S, B),), 0xFF, dtype=torch.uint8, device="cuda:0")
    print(f"[states] S {S}, {L} tokens", flush=True)
    mask = rr.rr_estimate(Q, K, S, B, 0.9, workspace=ws, block_mass=True)
    torch.cuda.synchronize()
    planes, masses = _parts(1, Hq, Hkv, L, rows, S)
    groups = -(-rows // min(rows, 256 // (Hq // Hkv * (B // S))))
    assert ws.numel() - planes - masses >= Hkv * groups * parts * 256 * 8 > ws.numel() - planes - masses - 2048
    for h in range(Hq):
        ref = gu.stride_masses(Q[0, h], K[0, h // (Hq // Hkv)], S, B, L - Lq, h)
        assert ((mask.block_mass[0, h].double() - ref).abs() <= 2.0 ** -16 * ref + 2.0 ** -24).all(), h      # as above
