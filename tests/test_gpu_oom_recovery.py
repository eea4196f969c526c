"""Allocations that fail (an allocator hook with a budget): the call says so, what
does not need the memory still runs, and nothing is taken to be allocated."""
import ctypes

import numpy as np
import pytest

import synth
from oracle import coo
from tests.gpu_common import oracle_Y, rel_fro, zipf_tensor

pytestmark = pytest.mark.gpu

TK_ERR_OOM = 3


class Hook:
    """Torch's allocator behind the library's hook: counts, and refuses above `budget`."""

    def __init__(self, tk):
        import torch
        from paper_1804_09494_amd import _lib
        self.budget, self.live, self.used, self.peak = 1 << 60, {}, 0, 0

        def alloc(n, user):
            n = int(n)
            if self.used + n > self.budget:
                return None
            p = torch.cuda.caching_allocator_alloc(n, 0, 0)
            self.live[p] = n
            self.used += n
            self.peak = max(self.peak, self.used)
            return p

        def free(p, n, user):
            self.used -= self.live.pop(p)
            torch.cuda.caching_allocator_delete(p)

        self.hook = _lib.tk_allocator(_lib.TK_ALLOC_FN(alloc), _lib.TK_FREE_FN(free), None)
        h = ctypes.c_void_p()
        assert _lib.load().tk_create(0, None, ctypes.byref(self.hook), ctypes.byref(h)) == 0
        self.ctx = tk.TuckerContext(0)
        self.ctx.close()
        self.ctx._h = h             # the same calls on the hooked context


def test_smaller_call_after_a_failed_one(tk):
    """Y of mode 0 does not fit; mode 2's, which is smaller, does."""
    dims, ranks = (9000, 500, 40), (4, 6, 5)
    idx, vals = zipf_tensor(dims, 40_000, seed=971)
    print("case", dims, flush=True)
    h = Hook(tk)
    ctx = h.ctx
    ctx.load_coo(idx, vals, dims)
    ctx.set_ranks(ranks)
    F = [synth.normal(972, 200 + n, d * k).reshape(d, k) for n, (d, k) in enumerate(zip(dims, ranks))]
    for n in range(3):
        ctx.set_factor(n, F[n])
    need = [4 * int(np.prod(ctx.ttm_shape(n))) for n in range(3)]
    assert need[2] < need[0] // 4
    h.budget = h.used + need[0] - 4     # no room for mode 0's, room for mode 2's and its partial rows
    with pytest.raises(tk.TuckerError) as e:
        ctx.ttm_chain(0)
    assert e.value.status == TK_ERR_OOM
    Y, _ = ctx.ttm_chain(2)
    ic, vc, _ = coo.coalesce_fast(idx, vals)
    want, _ = oracle_Y(ic, vc, [f.astype(np.float32).astype(np.float64) for f in F], 2, dims)
    assert rel_fro(Y, want) <= 1e-5
    ctx.close()
    assert not h.live
