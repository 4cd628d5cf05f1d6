"""Host side of the binding: what a table of addresses keeps alive."""
import weakref

import torch

import paper_2109_10060_amd as ds


class _Tensor:
    """As much of a device tensor as make_groups looks at."""
    is_cuda, dtype = True, torch.int32

    def is_contiguous(self):
        return True

    def data_ptr(self):
        return 4096


def test_groups_keep_their_tensors():
    # a table outlives the names its tensors had: with the memory handed to another tensor the kernels would take that
    # tensor's contents for slot offsets
    off, perm = _Tensor(), _Tensor()
    alive = [weakref.ref(off), weakref.ref(perm)]
    g = ds.make_groups(off, perm, [8, 16], [8, 24])
    del off, perm
    assert all(r() is not None for r in alive) and g.offsets == g.perm == 4096
    assert list(g.k_in[:2]) == [8, 16] and list(g.k_out[:2]) == [8, 24] and list(g.table_row[:2]) == [0, 1]
    del g
    assert all(r() is None for r in alive)
