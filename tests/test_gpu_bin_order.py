"""TTM-chains whose bins are launched in another order than they are numbered
(many bins, slices of many pieces), against the oracle, for each kernel that
walks the bins of a three-mode tensor."""
import numpy as np
import pytest

import synth
from oracle import coo
from tests.gpu_common import oracle_Y, rel_fro, zipf_tensor

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel", ["auto", "vector"])
@pytest.mark.parametrize("ranks", [(10, 10, 10), (3, 20, 5)], ids=["k10", "k20"])
def test_many_bins_of_split_slices(tk, kernel, ranks):
    idx, vals = zipf_tensor((3000, 2000, 700), 90_000, s=(0.4, 1.3, 1.5), seed=83)
    dims = tuple(int(i.max()) + 1 for i in idx)
    print("case", kernel, ranks, dims, flush=True)
    ctx = tk.TuckerContext(0, wg_nnz_target=16, ttm_kernel=kernel)
    ctx.load_coo(idx, vals, dims)
    ctx.set_ranks(ranks)
    F = [synth.normal(84, 200 + n, d * k).reshape(d, k) for n, (d, k) in enumerate(zip(dims, ranks))]
    for n in range(3):
        ctx.set_factor(n, F[n])
    ic, vc, _ = coo.coalesce_fast(idx, vals)
    F32 = [f.astype(np.float32).astype(np.float64) for f in F]
    ordered = 0
    for n in range(3):
        st = ctx.partition_stats(n)
        slots = st["R_sum"] - st["L_nonempty"] + st["n_bad"]
        ordered += st["P"] >= 4096 and slots >= 8 * st["n_bad"]
        Y, rows = ctx.ttm_chain(n)
        Yo, rows_o = oracle_Y(ic, vc, F32, n, dims)
        np.testing.assert_array_equal(rows, rows_o)
        assert rel_fro(Y, Yo) <= 1e-5, n
    assert ordered > 0   # the case is one of these
