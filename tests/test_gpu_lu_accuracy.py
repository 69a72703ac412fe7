"""Rounding errors of an LU plan's diagonal blocks in its single-wavefront nodes.
X_KK = Dt^{-1} - Uhat X_{C,K}: the product is summed by itself and Dt^{-1} enters
once, so that the error is the product's own and one rounding of X_KK, and does
not grow with the number of rows where the product is small beside Dt^{-1}."""

import numpy as np
import pytest


@pytest.mark.gpu
@pytest.mark.parametrize("c", [16, 33, 64])
def test_small_product_beside_the_diagonal_block(c):
    from paper_1604_02528_amd import SelInv

    # leaves of one column over a common clique of c rows
    m, rng = 64, np.random.default_rng(c)
    n = m + c
    rows = [np.concatenate([[j], np.arange(m, n)]) if j < m else np.arange(j, n) for j in range(n)]
    colptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
    rowind = np.concatenate(rows).astype(np.int64)
    cols = np.repeat(np.arange(n), np.diff(colptr))
    lo, up = rng.uniform(0.5, 1.0, (2, rowind.size)) / 8
    d = rowind == cols
    lo[d] = up[d] = rng.uniform(2.0, 3.0, n) + np.where(np.arange(n) >= m, 16.0, 0.0)
    A = np.zeros((n, n), np.longdouble)
    A[rowind, cols], A[cols, rowind] = lo, up
    S = SelInv(n, colptr, rowind, None, dtype="lu64", batch=1, relax=0.0)
    S.factor(np.concatenate([lo, up])[None])
    S.run()
    k = m - 1  # (the last leaf is a column of the root's supernode)
    assert S.symbolic()["xsuper"][k] == k
    got = S.extract().cpu().numpy()[0, :rowind.size][d][:k]
    # the exact diagonal of the leaves: 1 / d_j + (A_jC / d_j) X_CC (A_Cj / d_j)
    schur = A[m:, m:] - (A[m:, :m] / np.diag(A)[:m]) @ A[:m, m:]
    X = np.eye(c, dtype=np.longdouble)
    F = schur.copy()
    for j in range(c):  # Gauss-Jordan
        p = F[j, j]
        F[j] /= p
        X[j] /= p
        f = F[:, j].copy()
        f[j] = 0.0
        F -= np.outer(f, F[j])
        X -= np.outer(f, X[j])
    dl = np.diag(A)[:k]
    exact = 1 / dl + np.sum((A[:k, m:] @ X) * A[m:, :k].T, axis=1) / dl ** 2
    share = float(np.max(np.abs(exact - 1 / dl) * dl))
    rms = float(np.sqrt(np.mean(((got - exact) / exact) ** 2)))
    eps = np.finfo(float).eps
    # half an ulp (uniform: eps / (2 sqrt 3) at most) each for Dt^{-1} and for the
    # sum; the product's error: at most c + 3 roundings of its share
    bound = eps / np.sqrt(6.0) + (c + 3) * eps * share
    print(f"c={c}: rms {rms:.2e}, bound {bound:.2e}, share of the product {share:.2e}", flush=True)
    assert rms <= bound
    S.close()
