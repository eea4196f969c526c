"""The one-workgroup eigensolver of the SVD step at the edges of its 16-row
groups and 64-column halves, through one HOOI invocation (K-hat from 1 to 128)."""
import numpy as np
import pytest

import synth
from oracle import coo
from tests.gpu_common import U32, oracle_Y

pytestmark = pytest.mark.gpu

# K-hat of mode 0 is the product of the other two ranks
RANKS = [(1, 1, 1), (2, 1, 2), (1, 3, 1), (3, 3, 5), (16, 4, 4), (4, 1, 16), (5, 2, 9), (8, 2, 16), (11, 3, 11),
         (7, 4, 12), (16, 4, 16), (10, 5, 13), (9, 5, 16), (12, 9, 9), (11, 8, 12), (10, 7, 14), (10, 10, 10),
         (16, 7, 16), (13, 8, 15), (16, 8, 16)]


@pytest.mark.parametrize("ranks", RANKS, ids=[f"khat{b * c}_k{a}" for a, b, c in RANKS])
def test_factor_spans_leading_subspace(tk, ranks):
    """The new factor of mode 0 holds leading left singular vectors of Y_(0):
    with U orthonormal, ||U^T Y||_F^2 is the sum of the leading squared singular
    values.  Y in FP32 and the Gram route perturb Y^T Y by E with ||E||_F at most
    c u ||Y||_F^2, c = 4, and a K-subspace that is optimal for the perturbed
    Gram loses at most 2 sqrt(K) ||E||_F."""
    dims = (150, 60, 50)
    idx, vals = synth.make_tensor(dims, 9_000, "zipf", (0.6, 0.7, 0.8), "lognormal", seed=811)
    print("case", ranks, flush=True)
    ctx = tk.TuckerContext(0)
    ctx.load_coo(idx, vals, dims)
    ctx.set_ranks(ranks)
    F0 = synth.orthonormal_init(812, dims, ranks)
    for n in range(3):
        ctx.set_factor(n, np.ascontiguousarray(F0[n]))
    ctx.hooi_iterate(1)
    U = ctx.get_factor(0)
    np.testing.assert_allclose(U.T @ U, np.eye(ranks[0]), atol=1e-12)
    ic, vc, _ = coo.coalesce_fast(idx, vals)
    Y, rows = oracle_Y(ic, vc, [f.astype(np.float32).astype(np.float64) for f in F0], 0, dims)
    s2 = np.linalg.svd(Y, compute_uv=False) ** 2
    lead = s2[:ranks[0]].sum()
    got = np.linalg.norm(U[rows].T @ Y) ** 2
    assert abs(got - lead) <= 2 * np.sqrt(ranks[0]) * 4 * U32 * s2.sum()
