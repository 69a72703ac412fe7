"""Rounding errors of L_KK^{-1} in the normalization of a wide node: the top
block Dt^{-1} = L_KK^{-T} D^{-1} L_KK^{-1} against the same product of an inverse
by forward substitution, column by column, formed in extended precision.  The
device adds the rounding of its own product: a quarter more is allowed."""

import numpy as np
import pytest


def _inv_unit_lower(L):
    X = np.eye(len(L), dtype=L.dtype)
    for j in range(len(L)):
        X[j + 1:, :j + 1] -= np.outer(L[j + 1:, j], X[j, :j + 1])
    return X


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["f64", "c128", "h128"])
def test_wide_node(kind):
    import torch

    from paper_1604_02528_amd import SelInv, capi

    n = 256
    colptr = np.concatenate([[0], np.cumsum(np.arange(n, 0, -1))]).astype(np.int64)
    rowind = np.concatenate([np.arange(j, n) for j in range(n)]).astype(np.int64)
    S = SelInv(n, colptr, rowind, None, dtype=kind, batch=1, adjoint=False, relax=0.0)
    S._alloc(False)
    ext = np.longdouble if kind == "f64" else np.clongdouble
    got, plain = [], []
    for seed in range(4):
        rng = np.random.default_rng(seed)
        L = 2.0 * rng.uniform(-1.0, 1.0, (n, n)) / np.sqrt(n)  # entries of L_KK^{-1} grow by a few orders
        if kind != "f64":
            L = L + 2j * rng.uniform(-1.0, 1.0, (n, n)) / np.sqrt(n)
        L, D = np.tril(L, -1), rng.uniform(1.0, 2.0, n).astype(L.dtype)
        ldlt = torch.zeros_like(S.panels_view("panels"))
        ldlt[0, :n * n] = torch.from_numpy(np.ascontiguousarray((L + np.diag(D)).T.reshape(-1))).cuda()
        capi.selinv_normalize(S.h, ldlt, S._bufs["panels"], S._bufs["work"], None,
                              torch.cuda.current_stream().cuda_stream)
        S.sync()
        top = S.panels_view("panels").cpu().numpy()[0, :n * n].reshape(n, n).T

        def product(X):
            return (X.conj().T if kind == "h128" else X.T) @ (X / D.astype(ext)[:, None])

        exact = product(_inv_unit_lower(L.astype(ext)))
        rms = lambda e: float(np.sqrt(np.mean(np.abs(e) ** 2) / np.mean(np.abs(exact) ** 2)))
        got.append(rms(top - exact))
        plain.append(rms(product(_inv_unit_lower(L).astype(ext)) - exact))
    print(f"{kind}: rms {max(got):.2e}, by columns {max(plain):.2e}", flush=True)
    assert max(got) <= 1.25 * max(plain)
    S.close()
