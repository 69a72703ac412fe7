"""Imaginary parts of nearly real complex-symmetric matrices (the spectral
function of a pole expansion with small shifts): their rounding errors have to
be of their own size, not of the real parts'."""

import numpy as np
import pytest

from oracle import factor, selinv, symbolic
from tests.test_gpu_factor_blocks import _clique

DELTA = 1e-10  # size of the imaginary parts; the real parts' rounding errors are 1e6 times smaller only


def _nearly_real(s, c, seed):
    n, colptr, rowind, v = _clique(s, c, 1, "c128", seed)
    return n, colptr, rowind, v[0].real + 1j * DELTA * v[0].imag


@pytest.mark.gpu
@pytest.mark.parametrize("s,c", [(16, 120), (17, 64), (64, 130), (129, 70), (200, 150), (256, 200)])
def test_device_factorization(s, c):
    """Im(L D L^T - A), entry by entry, against the products with one imaginary
    factor that the factorization sums there: n terms of a few roundings each."""
    from paper_1604_02528_amd import SelInv

    print(f"imaginary parts of the factorization s={s} c={c}", flush=True)
    n, colptr, rowind, v = _nearly_real(s, c, 100 * s + c)
    sym = symbolic.analyze(n, colptr, rowind, None, cap=256, relax=0.0)
    S = SelInv(n, colptr, rowind, None, dtype="c128", batch=1, relax=0.0)
    P = S.factor_device(v[None]).cpu().numpy()[0, S.packed_index()]
    S.sync()
    L, D = factor.to_dense_L(sym, selinv.unflatten(sym, P))
    L, D = L.astype(np.clongdouble), D.astype(np.clongdouble)
    A = np.zeros((n, n), np.clongdouble)
    cols = np.repeat(np.arange(n), np.diff(colptr))
    A[rowind, cols] = A[cols, rowind] = v
    err = np.abs(((L * D) @ L.T - A).imag)
    Lr, Li, Dr, Di = np.abs(L.real), np.abs(L.imag), np.abs(D.real), np.abs(D.imag)
    terms = (Li * Dr) @ Lr.T + (Lr * Di) @ Lr.T + (Lr * Dr) @ Li.T + np.abs(A.imag)
    bound = 8 * n * np.finfo(float).eps * terms
    worst = float(np.max(err[terms > 0] / bound[terms > 0]))
    print(f"  worst error / bound {worst:.2e}", flush=True)
    assert worst <= 1.0
    S.close()


def _ldl(A):
    """Dense L D L^T in extended precision: unit lower L, D."""
    F, n = A.copy(), len(A)
    for j in range(n):
        col = F[j + 1:, j] / F[j, j]
        F[j + 1:, j + 1:] -= np.outer(col, F[j + 1:, j])
        F[j + 1:, j] = col
    return np.tril(F, -1) + np.eye(n), np.diag(F).copy()


def _inv_unit_lower(L):
    X = np.eye(len(L), dtype=L.dtype)
    for j in range(len(L)):
        X[j + 1:, :j + 1] -= np.outer(L[j + 1:, j], X[j, :j + 1])
    return X


@pytest.mark.gpu
@pytest.mark.parametrize("s,c", [(17, 100), (70, 100), (130, 70), (66, 300)])
def test_adjoint(s, c):
    """The reverse sweep of a node below the root from exact panels and X (the
    traversal's own products are not looked at): the imaginary parts of the
    gradient in the root's block and in the node's rows below its diagonal
    block, against the products with one imaginary factor; a few chained products
    of at most n terms, each within 8 roundings a term, on a dominant matrix."""
    import torch

    from paper_1604_02528_amd import SelInv

    print(f"imaginary parts of the adjoint s={s} c={c}", flush=True)
    n, colptr, rowind, v = _nearly_real(s, c, 100 * s + c)
    S = SelInv(n, colptr, rowind, None, dtype="c128", batch=1, relax=0.0)
    S.factor(v[None], want_dtilde=True)
    S.run()
    S.sync()
    sym = S.symbolic()
    assert np.array_equal(sym["perm"], np.arange(n)) and sym["xsuper"][1] == s
    cols = np.repeat(np.arange(n), np.diff(colptr))
    A = np.zeros((n, n), np.clongdouble)
    A[rowind, cols] = A[cols, rowind] = v
    L, D = _ldl(A)
    Li = _inv_unit_lower(L)
    X = Li.T @ (Li / D[:, None])
    panels, x = S.panels_view("panels"), S.panels_view("x")
    for K in range(sym["nsuper"]):
        a, b = sym["xsuper"][K], sym["xsuper"][K + 1]
        below = sym["rowind_L"][sym["rowptr"][K]:sym["rowptr"][K + 1]]
        Ki = _inv_unit_lower(L[a:b, a:b])
        top = Ki.T @ (Ki / D[a:b, None])
        for view, block in ((panels, np.concatenate([top, L[below, a:b] @ Ki])),
                            (x, np.concatenate([X[a:b, a:b], X[below, a:b]]))):
            flat = np.ascontiguousarray(block.T.reshape(-1).astype(np.complex128))
            view[0, sym["panel_off"][K]:sym["panel_off"][K] + flat.size] = torch.from_numpy(flat).cuda()
    rng = np.random.default_rng(s)
    g = rng.standard_normal((2, rowind.size))
    g, wl = g[0] + 1j * DELTA * g[1], np.array([0.7 + 0.3j * DELTA])
    got = S.backward(S.scatter(torch.from_numpy(g[None]).cuda()), torch.from_numpy(wl).cuda()).cpu().numpy()[0]
    half = np.where(rowind == cols, 1.0, 0.5)
    W = np.zeros((n, n), np.clongdouble)
    W[rowind, cols] = W[cols, rowind] = g * half
    G = -(X @ W) @ X + wl[0] * X
    Xr, Xi, Wr, Wi = np.abs(X.real), np.abs(X.imag), np.abs(W.real), np.abs(W.imag)
    terms = Xi @ Wr @ Xr + Xr @ Wi @ Xr + Xr @ Wr @ Xi + abs(wl[0].real) * Xi + abs(wl[0].imag) * Xr
    look = (rowind >= s + 2) & ((cols >= s + 2) | (cols < s))
    err = np.abs(got.imag - (G[rowind, cols] / half).imag)[look].max()
    bound = 64 * n * np.finfo(float).eps * float(terms[rowind, cols][look].max())
    print(f"  error {float(err):.2e}, bound {bound:.2e}", flush=True)
    assert err <= bound
    S.close()
