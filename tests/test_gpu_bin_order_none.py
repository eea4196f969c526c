"""A partition without split slices keeps no launch order of its bins."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_no_order_without_split_slices(tk):
    """Mode 0 has 5000 slices of 16 elements and bins of 16: each bin is one slice.
    The blocks that set_ranks leaves in use are counted by the allocator hook;
    an order of the bins would be one of 4 bytes per bin."""
    import torch
    from paper_1804_09494_amd import _lib
    P = 5000
    dims, ranks = (P, 61, 53), (2, 3, 2)
    e = np.arange(16 * P)
    idx = [(e // 16).astype(np.int32), (e % 61).astype(np.int32), (e % 53).astype(np.int32)]
    vals = np.ones(len(e), np.float32)
    print("case", P, flush=True)
    live = {}

    def alloc(n, user):
        p = torch.cuda.caching_allocator_alloc(int(n), 0, 0)
        live[p] = int(n)
        return p

    def free(p, n, user):
        live.pop(p)
        torch.cuda.caching_allocator_delete(p)

    hook = _lib.tk_allocator(_lib.TK_ALLOC_FN(alloc), _lib.TK_FREE_FN(free), None)
    L, h = _lib.load(), ctypes.c_void_p()
    assert L.tk_create(0, None, ctypes.byref(hook), ctypes.byref(h)) == 0
    ctx = tk.TuckerContext(0)
    ctx.close()
    ctx._h = h                      # the same calls on the hooked context
    ctx.set_options(wg_nnz_target=16, keep_elem_order=0)
    ctx.load_coo(idx, vals, dims)
    before = dict(live)
    ctx.set_ranks(ranks)
    st = ctx.partition_stats(0)
    assert st["P"] == P and st["n_bad"] == 0 and st["R_sum"] == P
    new = sorted(n for p, n in live.items() if p not in before)
    # of P int32 entries: mode 0's row_slice, row_of, label, seg_row and seg_slot, and
    # the bin orders of the other modes, whose slices are all split
    others = [ctx.partition_stats(n) for n in (1, 2)]
    assert all(o["P"] == P and o["n_bad"] == o["L_nonempty"] and o["R_sum"] > P for o in others), others
    assert new.count(4 * P) == 5 + 2, new
    ctx.close()
    assert not live
