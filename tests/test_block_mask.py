"""BlockMask.allocate: the arrays of small masks (views of one buffer) and of large ones (tensors of their own) have the same
shapes, types and contents, start at 256-byte steps of one another and do not overlap."""
import pytest
import torch


@pytest.mark.parametrize("Nb,rows", [(3, None), (9, 5), (300, None)])
@pytest.mark.parametrize("dense,mass,Hkv", [(True, True, 2), (False, False, None), (True, False, 4), (False, True, 1)])
def test_allocated_arrays(Nb, rows, dense, mass, Hkv):
    import paper_2602_05853_amd as rr
    m = rr.BlockMask.allocate(2, 4, Nb, 64, "cpu", dense=dense, block_mass=mass, Hkv=Hkv, rows=rows)
    Nq = rows or Nb
    want = {"row_count": ((2, 4, Nq), torch.int32), "row_list": ((2, 4, Nq, Nb), torch.int32),
            "dense": ((2, 4, Nq, Nb), torch.uint8) if dense else None,
            "block_mass": ((2, 4, Nq, Nb), torch.float32) if mass else None,
            "row_order": ((2, Hkv, 4 // Hkv * Nq), torch.int32) if Hkv else None,
            "queue": ((rr.binding.RR_QUEUE_WORDS,), torch.int32) if Hkv else None}
    arrays = {}
    for k, w in want.items():
        t = getattr(m, k)
        if w is None:
            assert t is None
            continue
        assert tuple(t.shape) == w[0] and t.dtype == w[1] and t.is_contiguous() and not t.any()
        arrays[k] = t
    for i, t in enumerate(arrays.values()):
        t.fill_(i + 1)                                      # every array keeps its own value: no overlap
    for i, t in enumerate(arrays.values()):
        assert (t == i + 1).all()
