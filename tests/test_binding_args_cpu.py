"""The binding's pointer tables against the element-by-element form (CPU)."""
import ctypes

import pytest
import torch

from paper_2606_09200_amd import binding as occ


def test_perm_array_in_place_and_copied_agree():
    base = torch.randperm(37).to(torch.int32)
    forms = [base, base.tolist(), base.to(torch.int64), base.numpy(), torch.stack([base, base], 1)[:, 0],
             torch.cat([base, base])[37:]]
    for f in forms:
        arr, n = occ._perm_arr(f)
        assert n == 37 and list(arr)[:n] == base.tolist()
        assert isinstance(arr, ctypes.Array) and arr._type_ is ctypes.c_int32
    assert occ._perm_arr([])[1] == 0 and occ._perm_arr(torch.empty(0, dtype=torch.int32))[1] == 0


def test_perm_array_is_a_snapshot():
    # what the caller writes afterwards (from
    # another thread, say) cannot reach a launch
    base = torch.randperm(37).to(torch.int32)
    want = base.tolist()
    for f in (base, base.numpy(), torch.cat([base, base])[37:], torch.stack([base, base], 1)[:, 0]):
        arr, n = occ._perm_arr(f)
        saved = torch.as_tensor(f).clone()
        f[...] = 1 << 20
        assert list(arr)[:n] == want
        f[...] = saved if isinstance(f, torch.Tensor) else saved.numpy()
    # a lazily negated view holds other values than its memory
    assert list(occ._perm_arr(torch._neg_view(-base))[0]) == want
    with pytest.raises((RuntimeError, NotImplementedError)):
        occ._perm_arr(torch.empty(4, dtype=torch.int32, device="meta"))


def test_row_pointers_only_for_rows_that_can_be_read_as_chunks():
    # the table itself needs no GPU: a stand-in with a tensor's shape and strides
    class Fake:
        dtype, is_cuda = torch.float32, True

        def __init__(self, t):
            self.t, self.shape = t, t.shape

        def __getattr__(self, k):
            return getattr(self.t, k)

    t = torch.zeros(6, 11)
    for v in (t, t[1:4], t[:, :7], t[:, 2:], t[::2]):
        arr = occ._row_ptrs(Fake(v))
        assert list(arr) == [r.data_ptr() for r in v.unbind(0)]
    for v in (t.t(), t[:, ::2], t[:0], t[:, :0], t[0], t[0].expand(3, 11)):
        assert occ._row_ptrs(Fake(v)) is None
    assert occ._row_ptrs(t) is None and occ._row_ptrs(t.double()) is None
