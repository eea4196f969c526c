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


def test_observations_without_room_for_the_two_pass_table(tk):
    """The forward's table of positions (4 bytes per observation) is the last thing
    tk_load_obs takes; a byte too little for it leaves the one-pass form, with the
    same values."""
    import torch
    dims, ranks, m = (400_000, 300, 20), (4, 3, 5), (1 << 20) + 77
    print("case", dims, flush=True)
    idx = [torch.from_numpy(i).cuda() for i in synth.coordinates(973, dims, m, "zipf", (0.3, 0.5, 0.5))]
    rng = np.random.default_rng(974)
    G = torch.from_numpy(rng.standard_normal(int(np.prod(ranks))).astype(np.float32)).cuda()
    F = [torch.from_numpy(rng.standard_normal((L, K)).astype(np.float32)).cuda() for L, K in zip(dims, ranks)]
    full = Hook(tk)
    full.ctx.load_obs(idx, dims, ranks)
    assert full.used == full.peak - 4           # the end of the call needs most (with a flag of 4 bytes)
    want = full.ctx.tucker_eval(G, F).cpu().numpy()
    total = full.peak
    full.ctx.close()
    h = Hook(tk)
    h.budget = total - 1
    h.ctx.load_obs(idx, dims, ranks)
    assert h.used <= total - 4 * m
    np.testing.assert_array_equal(h.ctx.tucker_eval(G, F).cpu().numpy(), want)
    h.ctx.close()
    assert not h.live and not full.live


def test_loading_observations_again(tk):
    """What the observations before leave during the next load: the work buffers for
    the adjoint's Y (300 rows of 15 floats at most) and the core, not the forward's
    table and values (8 bytes per observation and padding)."""
    import torch
    dims, ranks, m = (300, 200, 20), (4, 3, 5), (1 << 20) + 77
    print("case", dims, flush=True)
    idx = [torch.from_numpy(i).cuda() for i in synth.coordinates(975, dims, m, "zipf", (0.3, 0.5, 0.5))]
    h = Hook(tk)
    h.ctx.load_obs(idx, dims, ranks)
    first = h.peak
    assert first > h.used + 4               # the partition of the observations needs most
    h.peak = 0
    h.ctx.load_obs(idx, dims, ranks)
    assert h.peak - first <= 4 * (300 * 15 + 60 + 8)
    h.ctx.close()
    assert not h.live


def test_ranks_without_room_for_the_bin_order(tk):
    """The sort of the bins' launch order comes while the plan is at its largest; a
    byte too little for it leaves the bins as they are numbered."""
    dims, ranks = (3000, 2000, 700), (10, 10, 10)
    idx, vals = zipf_tensor(dims, 90_000, s=(0.4, 1.3, 1.5), seed=83)
    dims = tuple(int(i.max()) + 1 for i in idx)
    print("case", dims, flush=True)
    F = [synth.normal(84, 200 + n, d * k).reshape(d, k) for n, (d, k) in enumerate(zip(dims, ranks))]
    Y, peak, used = [], 0, 0
    for tight in (False, True):
        h = Hook(tk)
        h.ctx.set_options(wg_nnz_target=16, keep_elem_order=0)
        h.ctx.load_coo(idx, vals, dims)
        if tight:
            h.budget = peak - 1
        h.peak = 0
        h.ctx.set_ranks(ranks)
        if tight:
            assert h.used < used        # an order fewer
        peak, used = h.peak, h.used
        h.budget = 1 << 60
        for n in range(3):
            h.ctx.set_factor(n, F[n])
        Y.append([h.ctx.ttm_chain(n)[0] for n in range(3)])
        h.ctx.close()
        assert not h.live
    for a, b in zip(*Y):
        np.testing.assert_array_equal(a, b)
