"""Completion forward and adjoint where their forms change: the forward's parts of
128 positions and its two passes, the adjoint with many bins (one wave each)
and few (several waves), against FP64."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

# dims, observations, ranks, elements per bin (0: default)
CASES = {
    "one": ((5, 4, 3), 1, (2, 2, 2), 0),
    "part_edges": ((40, 30, 3), 4_000, (16, 5, 9), 1024),
    "tiny_slices": ((3000, 2500, 2000), 9_000, (7, 16, 3), 0),
    "many_bins": ((400, 300, 50), 40_000, (10, 16, 4), 16),
    "ordered_bins": ((4000, 300, 20), 90_000, (5, 6, 7), 16),
    "two_pass": ((2000, 900, 77), (1 << 20) + 333, (8, 3, 5), 0),
    "one_pass_many_slices": ((150_000, 140_000, 160_000), 1_300_000, (4, 5, 3), 0),
}


@pytest.mark.parametrize("name", list(CASES))
def test_forward_and_adjoint(tk, name):
    import torch
    dims, m, ranks, wg = CASES[name]
    print("case", name, flush=True)
    idx = synth.coordinates(91, dims, m, "zipf", (0.8, 0.9, 1.0))
    rng = np.random.default_rng(92)
    G = rng.standard_normal(ranks).astype(np.float32)
    F = [(rng.standard_normal((L, K)) / np.sqrt(K)).astype(np.float32) for L, K in zip(dims, ranks)]
    g = rng.standard_normal(m).astype(np.float32)
    ctx = tk.TuckerContext(0, wg_nnz_target=wg)
    ctx.load_obs([torch.from_numpy(i).cuda() for i in idx], dims, ranks)
    Gt = torch.from_numpy(G.ravel(order="F").copy()).cuda()
    Ft = [torch.from_numpy(f).cuda() for f in F]
    model = ctx.tucker_eval(Gt, Ft).cpu().numpy().astype(np.float64)
    dcore, dF = ctx.tucker_adjoint(torch.from_numpy(g).cuda(), Gt, Ft)
    # the same in FP64: rows gathered, the core contracted mode by mode
    G64, rows = G.astype(np.float64), [f[i].astype(np.float64) for f, i in zip(F, idx)]
    t01 = np.einsum("ma,mb->mab", rows[0], rows[1]).reshape(m, -1)
    GM = G64.reshape(-1, ranks[2])                       # (a, b) x c
    want = ((t01 @ GM) * rows[2]).sum(1)
    scale = np.linalg.norm(want)
    assert np.linalg.norm(model - want) <= 1e-5 * scale
    np.testing.assert_array_equal(ctx.tucker_eval(Gt, Ft).cpu().numpy(), model.astype(np.float32))
    gd = g.astype(np.float64)[:, None]
    wG = (t01 * gd).T @ rows[2]
    d = [None] * 3
    gr = (rows[2] * gd) @ GM.T                           # g sum_c G F_c, (a, b)
    gr = gr.reshape(m, ranks[0], ranks[1])
    d[0] = np.einsum("mab,mb->ma", gr, rows[1])
    d[1] = np.einsum("mab,ma->mb", gr, rows[0])
    d[2] = (t01 @ GM) * gd
    got = dcore.cpu().numpy().astype(np.float64).reshape(ranks, order="F").reshape(-1, ranks[2])
    assert np.linalg.norm(got - wG) <= 1e-5 * max(np.linalg.norm(wG), 1e-30)
    for n in range(3):
        w = np.zeros((dims[n], ranks[n]))
        for k in range(ranks[n]):
            w[:, k] = np.bincount(idx[n], weights=d[n][:, k], minlength=dims[n])
        e = np.linalg.norm(dF[n].cpu().numpy().astype(np.float64) - w)
        assert e <= 1e-5 * np.linalg.norm(w), (n, e, np.linalg.norm(w))
