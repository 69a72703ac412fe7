"""Rounding errors of the device factorization's pivots.  Elimination column by
column rounds an entry once, at the entry's own size, for every column that
updates it.  The device sums the updates of 16 columns first (their roundings
are of the updates' size) and rounds the entry once for all of them, so its
pivots have to be closer to the exact ones than column by column, by a margin
that no run-to-run order of the siblings' updates uses up."""

import numpy as np
import pytest

from workloads import grids


def _matrix(kind, shape, seed):
    rng = np.random.default_rng(seed)
    if kind == "h128":
        colptr, rowind, v = grids.magnetic_laplacian_3d(shape, rng)
    else:
        colptr, rowind, v = grids.weighted_laplacian_3d(shape, 0.05, rng)
    v = np.asarray(v).reshape(-1)
    n = int(np.prod(shape))
    cols = np.repeat(np.arange(n), np.diff(colptr))
    d = rowind == cols
    if kind == "c128":
        v = v + 1j * np.where(d, rng.uniform(0.05, 0.15, v.size), 0.0)
    elif kind == "h128":
        v = v + np.where(d, 0.1, 0.0)
    return n, colptr, rowind, cols, v


def _pivots(B, herm):
    B = B.copy()
    for j in range(len(B)):
        col = B[j + 1:, j].copy()
        B[j + 1:, j + 1:] -= np.outer(col / B[j, j], col.conj() if herm else col)
    return np.diag(B)


@pytest.mark.gpu
@pytest.mark.parametrize("kind,shape", [("f64", (9, 9, 9)), ("f64", (11, 8, 7)), ("c128", (8, 8, 8)),
                                        ("h128", (8, 8, 8)), ("h128", (7, 9, 8))])
def test_pivots_against_elimination_by_columns(kind, shape):
    from paper_1604_02528_amd import SelInv

    print(f"pivot errors {kind} {shape}", flush=True)
    got, plain = [], []
    for seed in range(3):
        n, colptr, rowind, cols, v = _matrix(kind, shape, seed)
        S = SelInv(n, colptr, rowind, grids.nested_dissection(shape), dtype=kind, batch=1, adjoint=False)
        P = S.factor_device(v[None]).cpu().numpy()[0]
        S.sync()
        sym = S.symbolic()
        A = np.zeros((n, n), v.dtype)
        A[cols, rowind] = v.conj() if kind == "h128" else v
        A[rowind, cols] = v
        B = A[np.ix_(sym["perm"], sym["perm"])]
        exact = _pivots(B.astype(np.longdouble if kind == "f64" else np.clongdouble), kind == "h128")
        D = np.empty(n, v.dtype)
        for K in range(sym["nsuper"]):
            a, s = sym["xsuper"][K], sym["xsuper"][K + 1] - sym["xsuper"][K]
            ld = s + sym["rowptr"][K + 1] - sym["rowptr"][K]
            D[a:a + s] = P[sym["panel_off"][K] + (ld + 1) * np.arange(s)]
        got.append(np.abs((D - exact) / exact))
        plain.append(np.abs((_pivots(B, kind == "h128") - exact) / exact))
        S.close()
    got, plain = (float(np.sqrt(np.mean(np.square(e)))) for e in (got, plain))
    print(f"  rms {got:.2e}, by columns {plain:.2e}", flush=True)
    assert got <= 0.6 * plain
