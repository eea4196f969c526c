"""The factor step (U = Y W, CholeskyQR2) at the edges of its routes: one
workgroup for few rows (256 rows, 2^15 entries of Y), 16-row tiles dealt to at
most 256 workgroups of 4 to 16 waves, Cholesky steps of 8, 16 and 32 columns."""
import numpy as np
import pytest

import synth
from oracle import coo
from tests.gpu_common import U32, oracle_Y

pytestmark = pytest.mark.gpu

# (rows of mode 0, ranks): K-hat of mode 0 is the product of the other two
CASES = [(1, (1, 2, 3)), (15, (2, 3, 3)), (16, (7, 4, 4)), (17, (8, 3, 7)), (65, (9, 5, 5)), (256, (16, 16, 8)),
         (255, (10, 8, 16)), (256, (5, 11, 12)),
         (257, (16, 9, 13)), (1023, (10, 8, 16)), (1024, (10, 8, 16)), (1025, (10, 8, 16)), (1024, (12, 11, 12)),
         (1024, (5, 1, 5)), (2500, (8, 5, 5)), (4097, (10, 10, 10)), (16400, (3, 7, 5)), (70000, (16, 4, 5)),
         (400, (17, 5, 5)), (1100, (20, 6, 7)), (300, (32, 6, 6))]


@pytest.mark.parametrize("rows, ranks", CASES, ids=[f"r{r}_k{k[0]}_khat{k[1] * k[2]}" for r, k in CASES])
def test_factor_step_edges(tk, rows, ranks):
    """Mode 0's new factor has orthonormal columns and spans a leading left
    singular subspace of Y_(0): ||U^T Y||_F^2 is the sum of the leading squared
    singular values, to 2 sqrt(K) ||E||_F with ||E||_F <= c u ||Y||_F^2, c = 4
    (Y in FP32, the Gram route and W rounded to FP32)."""
    dims = (rows, 60, 50)
    nnz = max(4 * rows, 9_000)
    idx, vals = synth.make_tensor(dims, nnz, "zipf", (0.0, 0.7, 0.8), "lognormal", seed=831)
    idx = [np.ascontiguousarray(i) for i in idx]
    idx[0][:rows] = np.arange(rows)                  # no empty slice: exactly `rows` rows
    print("case", rows, ranks, flush=True)
    ctx = tk.TuckerContext(0)
    ctx.load_coo(idx, vals, dims)
    ctx.set_ranks(ranks)
    F0 = synth.orthonormal_init(832, (max(rows, ranks[0]),) + dims[1:], ranks)
    for n in range(3):
        ctx.set_factor(n, np.ascontiguousarray(F0[n][:dims[n]]))
    ctx.hooi_iterate(1)
    U = ctx.get_factor(0)
    np.testing.assert_allclose(U.T @ U, np.eye(ranks[0]), atol=1e-12)
    ic, vc, _ = coo.coalesce_fast(idx, vals)
    Y, present = oracle_Y(ic, vc, [f.astype(np.float32).astype(np.float64) for f in F0], 0, dims)
    assert len(present) == rows
    s2 = np.linalg.svd(Y, compute_uv=False) ** 2
    lead = s2[:ranks[0]].sum()
    got = np.linalg.norm(U[present].T @ Y) ** 2
    assert abs(got - lead) <= 2 * np.sqrt(ranks[0]) * 4 * U32 * s2.sum()
