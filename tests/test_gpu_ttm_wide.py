"""The three-mode matrix-core TTM-chain for ranks 17 to 32: edges of its 16-column
planes, one to eight waves per bin, slices that straddle the waves of a bin
and the bins themselves."""
import numpy as np
import pytest

import synth
from oracle import coo
from tests.gpu_common import oracle_Y, rel_fro, zipf_tensor

pytestmark = pytest.mark.gpu


def _slices(sizes, seed):
    """Mode-0 slices of the given sizes, distinct coordinates in the other modes."""
    i0 = np.repeat(np.arange(len(sizes), dtype=np.int32), sizes)
    j = np.arange(len(i0))
    vals = np.random.default_rng(seed).standard_normal(len(i0)).astype(np.float32)
    return [i0, (j % 397).astype(np.int32), (j // 397 % 211).astype(np.int32)], vals


CASES = {
    "k32": (lambda: zipf_tensor((500, 400, 300), 40_000, seed=61), (32, 32, 32), 0),
    "k17": (lambda: zipf_tensor((500, 400, 300), 40_000, seed=62), (17, 17, 17), 0),
    "mixed": (lambda: zipf_tensor((500, 400, 300), 40_000, seed=63), (16, 20, 1), 2048),
    "odd_narrow": (lambda: zipf_tensor((300, 200, 100), 20_000, seed=64), (3, 31, 18), 1024),
    "bins_of_16": (lambda: zipf_tensor((300, 200, 100), 6_000, seed=65), (20, 24, 18), 16),
    "bins_of_300": (lambda: zipf_tensor((300, 200, 100), 20_000, seed=66), (20, 24, 18), 300),
    # slices over several waves of one bin, ending at and next to wave edges (512 elements a wave)
    "straddle": (lambda: _slices([511, 1, 1, 1600, 12, 499, 1024, 512, 3, 700, 17, 4000, 9000], 67), (18, 20, 22), 4096),
    # every bin inside one slice
    "one_slice": (lambda: _slices([70_000], 68), (1, 17, 32), 4096),
    # above the kernel's range: the vector ALUs
    "k33": (lambda: zipf_tensor((300, 200, 100), 10_000, seed=69), (33, 20, 17), 1024),
}


@pytest.mark.parametrize("name", list(CASES))
def test_wide_ttm_matches_oracle(tk, name):
    make, ranks, wg = CASES[name]
    idx, vals = make()
    dims = tuple(max(int(i.max()) + 1, k) for i, k in zip(idx, ranks))
    print("case", name, dims, len(vals), ranks, wg, flush=True)
    ctx = tk.TuckerContext(0, wg_nnz_target=wg)
    ctx.load_coo(idx, vals, dims)
    ctx.set_ranks(ranks)
    F = [synth.normal(71, 200 + n, d * k).reshape(d, k) for n, (d, k) in enumerate(zip(dims, ranks))]
    for n in range(3):
        ctx.set_factor(n, F[n])
    ic, vc, _ = coo.coalesce_fast(idx, vals)
    F32 = [f.astype(np.float32).astype(np.float64) for f in F]
    for n in range(3):
        Y, rows = ctx.ttm_chain(n)
        Yo, rows_o = oracle_Y(ic, vc, F32, n, dims)
        np.testing.assert_array_equal(rows, rows_o)
        assert rel_fro(Y, Yo) <= 1e-5, n
        np.testing.assert_array_equal(ctx.ttm_chain(n)[0], Y)   # fixed order: the same bits again
