"""The four-mode TTM-chain's BF16 tiles entry by entry: its own LDS row order, slice
masks per quad of elements and operand packing, over the FP32 form's shapes."""
import numpy as np
import pytest

import synth
from oracle import coo
from tests.gpu_common import U32, oracle_Y
from tests.test_gpu_ttm4_tiles import RANKS

pytestmark = pytest.mark.gpu

U16 = 2.0 ** -8   # BF16 unit roundoff (8 significant bits)


@pytest.mark.parametrize("bins", [0, 64, 3000], ids=lambda b: f"bins{b}")
@pytest.mark.parametrize("ranks", RANKS, ids=lambda r: "x".join(map(str, r)))
def test_ttm4_tiles_bf16(tk, ranks, bins):
    """A term is bf16(value F_a) times bf16(F_b F_c), each product rounded to FP32
    before: two roundings of 2^-8 and three of 2^-24 in a term, FP32 sums."""
    dims = (90, 70, 60, 50)
    idx, vals = synth.make_tensor(dims, 6_000, "zipf", (1.2, 0.4, 0.6, 0.5), "lognormal", seed=841)
    print("case", ranks, bins, flush=True)
    ctx = tk.TuckerContext(0, wg_nnz_target=bins, prec="bf16")
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
        bound = 2 * U16 + U16 * U16 + (terms[:, None] + 4) * U32
        assert np.all(np.abs(Y - want) <= bound * mag + 1e-300)
