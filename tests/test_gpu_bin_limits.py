"""Bins too large for a CU's LDS are refused, whichever matrix-core kernel the
number of bins and the precision lead to, and those below the limit are not."""
import numpy as np
import pytest

from oracle import coo
from tests.gpu_common import oracle_Y, rel_fro, uniform_tensor

pytestmark = pytest.mark.gpu

TK_ERR_UNSUPPORTED = 6

# dims, elements, ranks, elements per bin, whether mode 0's bins fit.
# Three modes: 12 bytes per element and K-hat floats per slice beside 2 KB; four
# modes: 16 bytes per element beside 12 KB, 160 KB altogether.
CASES = {
    "three_over": ((40, 300, 200), 60_000, (4, 5, 5), 30_000, False),
    "three_under": ((40, 300, 200), 60_000, (4, 5, 5), 9_000, True),
    "four_over": ((12, 80, 60, 50), 60_000, (2, 8, 6, 7), 11_000, False),
    "four_under": ((12, 80, 60, 50), 60_000, (2, 8, 6, 7), 5_000, True),
    # many short slices: the rows a bin may hold keep its elements few
    "four_short_slices": ((4000, 80, 60, 50), 60_000, (2, 10, 10, 10), 20_000, True),
}


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("name", list(CASES))
def test_bin_limit(tk, name, prec):
    dims, nnz, ranks, wg, fits = CASES[name]
    print("case", name, prec, flush=True)
    idx, vals = uniform_tensor(dims, nnz, seed=87)
    ctx = tk.TuckerContext(0, wg_nnz_target=wg, prec=prec)
    ctx.load_coo(idx, vals, dims)
    ctx.set_ranks(ranks)
    rng = np.random.default_rng(88)
    F = [rng.standard_normal((L, K)) for L, K in zip(dims, ranks)]
    for n in range(len(dims)):
        ctx.set_factor(n, F[n])
    if fits:
        ic, vc, _ = coo.coalesce_fast(idx, vals)
        want, _ = oracle_Y(ic, vc, [f.astype(np.float32).astype(np.float64) for f in F], 0, dims)
        assert rel_fro(ctx.ttm_chain(0)[0], want) <= (1e-5 if prec == "fp32" else 1e-2)
    else:
        with pytest.raises(tk.TuckerError) as e:
            ctx.ttm_chain(0)
        assert e.value.status == TK_ERR_UNSUPPORTED
        ctx.set_options(ttm_kernel="vector")       # whatever the bin sizes
        ctx.ttm_chain(0)
