"""What the one-workgroup eigensolver's eigenvectors and eigenvalues are accurate
to: first-order subspace errors on planted spectra (isolated and clustered), and
Ritz values down to FP64's resolution where a residual depends on them."""
import numpy as np
import pytest

import synth
from tests.gpu_common import U32

pytestmark = pytest.mark.gpu


def _dense(T):
    """The element list of a dense array."""
    idx = [i.ravel().astype(np.int32) for i in np.indices(T.shape)]
    return idx, T.ravel().astype(np.float32)


def _orth(seed, stream, n, k):
    return np.linalg.qr(synth.normal(seed, stream, n * k).reshape(n, k))[0]


# squared singular values, K of them leading
SPECTRA = {
    "isolated": lambda K, n: np.concatenate([np.linspace(1.0, 0.5, K), np.linspace(0.2, 0.01, n - K)]),
    # spacings below 1e-3 of the norm inside the leading K
    "cluster": lambda K, n: np.concatenate([1.0 - 1e-4 * np.arange(K), np.linspace(0.5, 0.01, n - K)]),
    "equal": lambda K, n: np.concatenate([np.ones(K), np.full(n - K, 0.25)]),
}


@pytest.mark.parametrize("spectrum", list(SPECTRA))
@pytest.mark.parametrize("ranks", [(5, 5, 5), (10, 10, 10), (10, 8, 13), (16, 8, 12), (16, 16, 8)],
                         ids=lambda r: "x".join(map(str, r)))
def test_planted_spectrum(tk, ranks, spectrum):
    """Factors of modes 1 and 2 are identities, so Y_(0) is the planted matrix in
    FP32.  Y's rounding and the Gram route perturb Y^T Y by E, ||E|| <= 4 u
    sigma_1^2; the sin-theta theorem bounds the leading subspace's distance by
    sqrt(2) ||E|| / (lambda_K - lambda_{K+1}) and an isolated vector's by
    sqrt(2) ||E|| over its gap; V's columns are rounded to FP32 on the way (a
    further u each, sqrt(K) u sigma_1 / sigma_K together)."""
    K, n, rows = ranks[0], ranks[1] * ranks[2], 150
    lam = SPECTRA[spectrum](K, n)
    Y = (_orth(921, 1, rows, n) * np.sqrt(lam)) @ _orth(921, 2, n, n).T
    print("case", ranks, spectrum, flush=True)
    # Y_(0)'s columns: the first remaining mode fastest
    idx, vals = _dense(Y.reshape(rows, ranks[2], ranks[1]).transpose(0, 2, 1))
    ctx = tk.TuckerContext(0)
    dims = (rows,) + ranks[1:]
    ctx.load_coo(idx, vals, dims)
    ctx.set_ranks(ranks)
    ctx.set_factor(0, _orth(921, 3, rows, K))
    for j in (1, 2):
        ctx.set_factor(j, np.eye(ranks[j]))
    ctx.hooi_iterate(1)
    U = ctx.get_factor(0)
    np.testing.assert_allclose(U.T @ U, np.eye(K), atol=1e-12)
    ref, s, _ = np.linalg.svd(Y.astype(np.float32).astype(np.float64), full_matrices=False)
    E = 4 * U32 * s[0] ** 2
    more = np.sqrt(K) * U32 * s[0] / s[K - 1]
    P = ref[:, :K]
    dist = np.linalg.norm(U - P @ (P.T @ U), 2)
    print("  subspace distance", dist, flush=True)
    assert dist <= np.sqrt(2) * E / (s[K - 1] ** 2 - s[K] ** 2) + more
    if spectrum == "isolated":
        for k in range(K):
            gap = min(abs(s[k] ** 2 - s[j] ** 2) for j in range(len(s)) if j != k)
            c = abs(P[:, k] @ U[:, k])
            # (CholeskyQR2 subtracts the columns before it: as much again)
            assert np.sqrt(max(0.0, 1 - c * c)) <= 2 * (np.sqrt(2) * E / gap + more), k


def test_ritz_values_at_fp64_resolution(tk):
    """Ranks 13 and 15 at K-hat 195 and 225: the block-Krylov solver's Rayleigh-Ritz
    steps are 96 x 96 problems for 14 and 16 pairs.  Y has 13 (15) large singular
    values and the rest at 1e-6 of them, so what stops the estimated error,
    sqrt(2) residual theta_1 / gap (the ratio below 10 here), is rounding: with the
    general dense solver (FP64 resolution) in the Rayleigh-Ritz step it comes to
    between 1e-13 and 3e-13 on this tensor.  An eig_tol of 6e-13 accepts that in every
    mode; Ritz values known to 1e-11 of the norm (errors up to 5e-13 of it and
    more, times the ratio) need the dense solver instead."""
    dims, ranks = (40, 36, 32), (13, 15, 15)
    G = synth.normal(931, 1, 13 * 15 * 15).reshape(13, 15, 15)
    A = [_orth(931, 2 + n, L, K) for n, (L, K) in enumerate(zip(dims, ranks))]
    T = np.einsum("abc,ia,jb,kc->ijk", G, *A, optimize=True)
    T += 1e-6 * np.linalg.norm(T) / np.sqrt(T.size) * synth.normal(931, 5, T.size).reshape(T.shape)
    print("case", ranks, flush=True)
    idx, vals = _dense(T)
    ctx = tk.TuckerContext(0, eig_tol=6e-13)
    ctx.load_coo(idx, vals, dims)
    ctx.set_ranks(ranks)
    for n in range(3):
        ctx.set_factor(n, np.ascontiguousarray(A[n]))
    for n in range(3):
        Y, _ = ctx.ttm_chain(n)
        s2 = np.linalg.svd(Y.astype(np.float64), compute_uv=False) ** 2
        K = ranks[n]
        assert s2[0] < 10 / np.sqrt(2) * (s2[K - 1] - (s2[K] if len(s2) > K else 0.0)), n
    ctx.hooi_iterate(1)
    c = ctx.counters()
    print("  ", c, flush=True)
    assert c["eig_krylov_solves"] == 3
    assert c["eig_dense_fallbacks"] == 0
