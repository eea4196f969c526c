"""The four-mode matrix-core TTM-chain over the shapes of its column-to-lane map
(tiles, lanes above K_b, rows staged or not) and of its slices (inside a wave,
across waves, across bins), FP32 against the oracle, reruns bit-identical."""
import numpy as np
import pytest

import synth
from oracle import coo
from tests.gpu_common import U32, oracle_Y

pytestmark = pytest.mark.gpu

# ranks; mode 0's K_a, K_b, K_c are the last three
RANKS = [(3, 1, 1, 1), (2, 3, 2, 5), (4, 4, 4, 8), (2, 5, 4, 9), (2, 5, 6, 6), (3, 16, 3, 16), (3, 7, 16, 3), (2, 10, 10, 10),
         (2, 9, 8, 10), (2, 11, 12, 12), (2, 6, 13, 13), (2, 16, 11, 11), (2, 15, 16, 15), (2, 13, 15, 16), (1, 2, 16, 16)]


@pytest.mark.parametrize("bins", [0, 64, 3000], ids=lambda b: f"bins{b}")
@pytest.mark.parametrize("ranks", RANKS, ids=lambda r: "x".join(map(str, r)))
def test_ttm4_tiles(tk, ranks, bins):
    """An entry of Y sums products of a value and three FP32 factor entries:
    with nnz_row terms its error is at most (nnz_row + 3) u times the sum of
    their magnitudes."""
    dims = (90, 70, 60, 50)
    idx, vals = synth.make_tensor(dims, 6_000, "zipf", (1.2, 0.4, 0.6, 0.5), "lognormal", seed=841)
    print("case", ranks, bins, flush=True)
    ctx = tk.TuckerContext(0, wg_nnz_target=bins)
    ctx.load_coo(idx, vals, dims)
    ctx.set_ranks(ranks)
    F0 = [f.astype(np.float32).astype(np.float64) for f in synth.orthonormal_init(842, dims, ranks)]
    for n in range(4):
        ctx.set_factor(n, np.ascontiguousarray(F0[n]))
    ic, vc, _ = coo.coalesce_fast(idx, vals)
    for n in range(4):
        Y, rows = ctx.ttm_chain(n)
        Y2, _ = ctx.ttm_chain(n)
        np.testing.assert_array_equal(Y, Y2)
        want, present = oracle_Y(ic, vc, F0, n, dims)
        mag, _ = oracle_Y(ic, np.abs(vc), [np.abs(f) for f in F0], n, dims)
        np.testing.assert_array_equal(rows, present)
        terms = np.bincount(ic[n], minlength=dims[n])[present]
        assert np.all(np.abs(Y - want) <= (terms[:, None] + 3) * U32 * mag + 1e-300)
