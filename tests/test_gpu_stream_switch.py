"""A context moved to another stream while its TTM-chains are still queued on the
former one: what it releases and loads next must not touch what they read."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _tensor(dims, nnz, seed):
    import torch
    g = torch.Generator(device="cuda:0")
    g.manual_seed(seed)
    idx = [torch.randint(0, L, (nnz,), generator=g, device="cuda:0", dtype=torch.int32) for L in dims]
    return idx, torch.randn(nnz, generator=g, device="cuda:0").exp_()


@pytest.mark.parametrize("noalloc", [False, True], ids=["chain", "noalloc"])
def test_reload_after_switch_leaves_queued_chains_alone(tk, noalloc):
    import torch
    dims, ranks, nnz = (40_000, 30_000, 20_000), (10, 10, 10), 4_000_000
    print("case", noalloc, flush=True)
    first, second = _tensor(dims, nnz, 901), _tensor(dims, nnz, 902)
    F = [synth.normal(903, 200 + n, d * k).reshape(d, k) for n, (d, k) in enumerate(zip(dims, ranks))]
    A, B = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()

    def load(ctx, t):
        ctx.load_coo(*t, dims)
        ctx.set_ranks(ranks)
        for n in range(3):
            ctx.set_factor(n, F[n])

    with torch.cuda.stream(A):
        ctx = tk.TuckerContext(0)
        load(ctx, first)
        R, kh = ctx.ttm_shape(0)
        out = [torch.full((R, kh), float("nan"), device="cuda:0") for _ in range(24)]
        chain = ctx.ttm_chain_noalloc if noalloc else ctx.ttm_chain
        chain(0, out[0])
        torch.cuda.synchronize()
        want = out[0].cpu().numpy()
        for Y in out:
            chain(0, Y)
    ctx.set_stream(B)
    load(ctx, second)          # releases the first tensor's plan, takes blocks for its own
    torch.cuda.synchronize()
    for Y in out:
        np.testing.assert_array_equal(Y.cpu().numpy(), want)
    with torch.cuda.stream(B):
        got = ctx.ttm_chain(0)[0]
        ref = tk.TuckerContext(0)
    load(ref, second)
    np.testing.assert_array_equal(got, ref.ttm_chain(0)[0])


def test_switch_inside_a_capture(tk):
    """The context moves to the capturing stream inside the capture, and back after
    it; every replay gives the eager rows, with eager work, releases and new
    factors between them."""
    import torch
    dims, ranks, nnz = (3000, 2000, 700), (10, 8, 5), 200_000
    print("case", dims, flush=True)
    t = _tensor(dims, nnz, 904)
    F = [[synth.normal(s, 200 + n, d * k).reshape(d, k) for n, (d, k) in enumerate(zip(dims, ranks))]
         for s in (905, 906)]
    torch.cuda.synchronize()
    ctx, other = tk.TuckerContext(0), tk.TuckerContext(0)
    for c in (ctx, other):
        c.load_coo(*t, dims)
        c.set_ranks(ranks)
    Y = torch.empty(ctx.ttm_shape(0), device="cuda:0")
    home = torch.cuda.current_stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        ctx.set_stream(torch.cuda.current_stream())
        ctx.ttm_chain_noalloc(0, Y)
    ctx.set_stream(home)
    for rep in range(4):
        for n in range(3):
            ctx.set_factor(n, F[rep % 2][n])
            other.set_factor(n, F[rep % 2][n])
        want = other.ttm_chain(0)[0]
        ctx.ttm_chain(1)               # eager work on the context between the replays
        Y.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(Y.cpu().numpy(), want)
        np.testing.assert_array_equal(ctx.ttm_chain(0)[0], want)
