"""Top-tau selection against its definition, applied on the host to the block masses the same call reports: rows of one to
five chunks of 64 key blocks, rows in registers and in LDS, rows of equal masses (ties go to the smaller index), a row
with one dominant block.  The definition ranks by mass and keeps the shortest prefix whose sum reaches tau; rows whose
prefix sum comes within 2^-25 per candidate (3.1e-5 for 1025) of tau are left out: the kernel adds 32-bit masses up one
after the other where they tie, sums stay below 1, and each addition rounds by at most 2^-25."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _expected(frac, m, tau):
    order = np.lexsort((np.arange(m + 1), -frac[: m + 1]))
    sums = np.cumsum(frac[: m + 1][order].astype(np.float64))
    if np.abs(sums - tau).min() < max(2e-6, (m + 1) * 2.0 ** -25):
        return None
    k = int(np.searchsorted(sums, tau)) + 1
    keep = np.zeros(frac.shape[0], dtype=np.uint8)
    keep[order[:k]] = 1
    return keep


@pytest.mark.parametrize("Nb,dtype,d,B", [(5, "bf16", 128, 128), (64, "bf16", 128, 128), (65, "bf16", 128, 128),
                                          (257, "bf16", 128, 128), (513, "bf16", 128, 128), (1025, "bf16", 128, 128),
                                          (64, "f32", 64, 32), (257, "f32", 64, 32), (300, "bf16", 64, 32)])
@pytest.mark.parametrize("kind", ["random", "ties", "dominant"])
def test_selection_follows_its_definition(kind, Nb, dtype, d, B):
    import paper_2602_05853_amd as rr
    L, S = Nb * B, 8
    g = torch.Generator(device="cuda:0").manual_seed(Nb)
    Q = torch.randn(1, 2, L, d, generator=g, device="cuda:0") * 2.0
    K = torch.randn(1, 1, L, d, generator=g, device="cuda:0")
    if kind == "ties":
        K[:] = K[:, :, :1]                                  # every key the same: every block before the row's own weighs the same
    if kind == "dominant":
        K[:, :, :B] = 0.5 * Q.mean(dim=(1, 2), keepdim=True) + 40.0 / d ** 0.5
        Q += 3.0 / d ** 0.5
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    tau = 0.87
    mask = rr.rr_estimate(Q.to(tdt), K.to(tdt), S, B, tau, flags=0, block_mass=True)
    torch.cuda.synchronize()
    frac, dense = mask.block_mass.cpu().numpy()[0], mask.dense.cpu().numpy()[0]
    count, lists = mask.row_count.cpu().numpy()[0], mask.row_list.cpu().numpy()[0]
    checked = 0
    for h in range(2):
        for m in range(Nb):
            want = _expected(frac[h, m], m, tau)
            assert np.array_equal(lists[h, m, : count[h, m]], np.nonzero(dense[h, m])[0]), (h, m)
            if want is not None:
                checked += 1
                assert np.array_equal(dense[h, m], want), (h, m, int(dense[h, m].sum()), int(want.sum()))
    print(f"[selection] {kind} Nb={Nb}: {checked} of {2 * Nb} rows", flush=True)
    assert checked >= Nb                                    # nearly all rows, in every case
