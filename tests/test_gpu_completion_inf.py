"""Model values where a factor row is infinite (a diverged step): ranks below 16
leave padding in the forward's tiles, which must not turn an infinity into NaN."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ranks", [(3, 5, 7), (16, 16, 3), (15, 16, 16), (16, 1, 16)],
                         ids=lambda r: "x".join(map(str, r)))
def test_infinite_row_of_the_walked_mode(tk, ranks):
    """Positive core and factors, one row of the mode with the fewest slices (the
    one the forward walks) infinite: its observations' values are +inf, the
    others' are the finite model values."""
    import torch
    dims, m = (400, 300, 6), 5_000
    print("case", ranks, flush=True)
    rng = np.random.default_rng(95)
    idx = [rng.integers(0, L, m).astype(np.int32) for L in dims]
    G = rng.uniform(0.5, 1.5, ranks).astype(np.float32)
    F = [rng.uniform(0.5, 1.5, (L, K)).astype(np.float32) for L, K in zip(dims, ranks)]
    F[2][4] = np.inf
    ctx = tk.TuckerContext(0)
    ctx.load_obs([torch.from_numpy(i).cuda() for i in idx], dims, ranks)
    got = ctx.tucker_eval(torch.from_numpy(G.ravel(order="F").copy()).cuda(),
                          [torch.from_numpy(f).cuda() for f in F]).cpu().numpy()
    at = idx[2] == 4
    assert at.any() and not at.all()
    assert np.all(np.isposinf(got[at]))
    rows = [f[i].astype(np.float64) for f, i in zip(F, idx)]
    want = np.einsum("abc,ma,mb,mc->m", G.astype(np.float64), *[r[~at] for r in rows], optimize=True)
    np.testing.assert_allclose(got[~at], want, rtol=1e-5)
