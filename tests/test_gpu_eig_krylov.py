"""The block-Krylov eigensolver's one-workgroup orthonormalisation at the edges
of its row tiles (a wave holds 2, 4, 8 or 16 of them; 2048 rows at most),
through one HOOI invocation (K-hat from 192 to 2080), with Y of full and of
low rank (dependent Krylov blocks)."""
import numpy as np
import pytest

import synth
from oracle import coo
from tests.gpu_common import U32, oracle_Y

pytestmark = pytest.mark.gpu

# K-hat of mode 0 is the product of the other three ranks
RANKS = [(4, 4, 6, 8), (7, 5, 5, 8), (3, 16, 16, 1), (16, 4, 5, 13), (10, 8, 8, 8), (5, 5, 8, 13), (10, 10, 10, 10),
         (12, 8, 8, 16), (9, 8, 10, 13), (8, 16, 16, 8), (8, 16, 13, 10)]


@pytest.mark.parametrize("ranks, rows", [(r, 150) for r in RANKS] + [(RANKS[6], 24), (RANKS[0], 9)],
                         ids=lambda x: "x".join(map(str, x)) if isinstance(x, tuple) else f"rows{x}")
def test_factor_spans_leading_subspace(tk, ranks, rows):
    """The new factor of mode 0 holds leading left singular vectors of Y_(0):
    ||U^T Y||_F^2 is the sum of the leading squared singular values.  Y in FP32
    and the Gram route perturb Y^T Y by E with ||E||_F at most c u ||Y||_F^2,
    c = 4, and a K-subspace that is optimal for the perturbed Gram loses at most
    2 sqrt(K) ||E||_F; an accepted residual adds its square, far below."""
    dims = (rows, 40, 36, 32)
    idx, vals = synth.make_tensor(dims, 9_000, "zipf", (0.6, 0.7, 0.8, 0.5), "lognormal", seed=821)
    print("case", ranks, rows, flush=True)
    ctx = tk.TuckerContext(0)
    ctx.load_coo(idx, vals, dims)
    ctx.set_ranks(ranks)
    F0 = synth.orthonormal_init(822, dims, ranks)
    for n in range(4):
        ctx.set_factor(n, np.ascontiguousarray(F0[n]))
    ctx.hooi_iterate(1)
    assert ctx.counters()["eig_krylov_solves"] > 0
    U = ctx.get_factor(0)
    np.testing.assert_allclose(U.T @ U, np.eye(ranks[0]), atol=1e-12)
    ic, vc, _ = coo.coalesce_fast(idx, vals)
    Y, present = oracle_Y(ic, vc, [f.astype(np.float32).astype(np.float64) for f in F0], 0, dims)
    s2 = np.linalg.svd(Y, compute_uv=False) ** 2
    lead = s2[:ranks[0]].sum()
    got = np.linalg.norm(U[present].T @ Y) ** 2
    assert abs(got - lead) <= 2 * np.sqrt(ranks[0]) * 4 * U32 * s2.sum()
