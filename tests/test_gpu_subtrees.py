"""Bottom subtrees of small nodes (one workgroup each) at the edges of their
rule: chains of one-column nodes around the tallest subtree, stars around the
widest, a comb of both, and a batch on either side of the largest launch, for
every scalar type, against numpy's dense inverse."""

import numpy as np
import pytest

from oracle import selinv, symbolic
from tests.test_oracle_lu import dense_original_lu, selected_from_dense_lu


def _pattern(shape, m):
    """Parent of every column but the last (a tree given as its elimination tree)."""
    if shape == "chain":
        return list(range(1, m + 1))
    if shape == "star":  # m leaves under one root
        return [m] * m
    # comb: a spine of m nodes, each but the first with a leaf of its own
    par, spine = [], None
    for i in range(m):
        if i > 0:
            k = len(par)
            par += [k + 1]
            par[spine] = k + 1
            spine = k + 1
        else:
            spine = 0
        par.append(None)
    par[spine] = len(par)
    return par


def _matrix(shape, m, batch, kind, seed):
    par = _pattern(shape, m)
    n = len(par) + 1
    rowind, colptr = [], [0]
    for j in range(n):
        rowind.append(j)
        if j < n - 1:
            rowind.append(par[j])
        colptr.append(len(rowind))
    colptr, rowind = np.array(colptr, np.int64), np.array(rowind, np.int64)
    cols = np.repeat(np.arange(n), np.diff(colptr))
    rng = np.random.default_rng(seed)
    v = rng.uniform(-1.0, 1.0, (batch, rowind.size))
    if kind in ("c128", "h128"):
        v = v + 1j * rng.uniform(-1.0, 1.0, v.shape)
    v /= max(4, n if shape == "star" else 4)
    d = rowind == cols
    v[:, d] = 3.0 + rng.uniform(0.0, 1.0, (batch, n))
    return n, colptr, rowind, cols, d, v


def _check(shape, m, batch, kind, look):
    from paper_1604_02528_amd import SelInv

    print(f"subtree case {shape} m={m} batch={batch} {kind}", flush=True)
    n, colptr, rowind, cols, d, lo = _matrix(shape, m, batch, kind, 7 * m)
    lu = kind == "lu64"
    up = lo.conj() if kind == "h128" else lo
    if lu:
        up = lo[:, ::-1] * 0.5
        up[:, d] = lo[:, d]
    sym = symbolic.analyze(n, colptr, rowind, None, cap=1, relax=0.0)
    S = SelInv(n, colptr, rowind, None, dtype=kind, batch=batch, cap=1, relax=0.0)
    S.factor(np.concatenate([lo, up], axis=1) if lu else lo)
    S.run()
    S.sync()
    X = S.to_host("x")
    for l in look:
        if lu:
            A = dense_original_lu(n, colptr, rowind, lo[l], up[l])
        else:
            A = np.zeros((n, n), lo.dtype)
            A[cols, rowind] = up[l]
            A[rowind, cols] = lo[l]
        RL, RU = selected_from_dense_lu(sym, np.linalg.inv(A))
        ref = selinv.flatten(sym, RL)
        if lu:
            ref = np.concatenate([ref, selinv.flatten(sym, RU)])
        # both inverses are backward stable on a dominant matrix: n eps kappa each, a few such terms
        bound = 8 * n * np.finfo(float).eps * np.linalg.cond(A, np.inf)
        err = np.max(np.abs(X[l] - ref)) / np.max(np.abs(ref))
        print(f"  matrix {l}: {err:.2e}, bound {bound:.2e}", flush=True)
        assert err <= bound
    S.close()


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["f64", "c128", "h128", "lu64"])
@pytest.mark.parametrize("shape,m", [("chain", 1), ("chain", 31), ("chain", 32), ("chain", 70), ("star", 1), ("star", 16),
                                     ("star", 17), ("star", 90), ("comb", 16), ("comb", 40)])
def test_edges_of_the_rule(shape, m, kind):
    _check(shape, m, 1, kind, [0])
    _check(shape, m, 3, kind, [0, 1, 2])


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["f64", "c128"])
@pytest.mark.parametrize("batch", [2047, 2048, 2049, 4100])
def test_largest_launch(batch, kind):
    """32 nodes in the subtree, halves of the batch around 32768 / 32 matrices."""
    _check("chain", 31, batch, kind, [0, 1022, 1023, batch // 2, batch - 1])


@pytest.mark.gpu
def test_infinite_factor_entry_stays_infinite():
    """L_10 = inf in a 2 x 2 matrix: X_10 = -X_11 L_10 and X_00 = 1 / D_0 +
    L_10^2 X_11 are infinite, not NaN (no padding times infinity)."""
    import torch

    from paper_1604_02528_amd import SelInv, capi

    n, colptr, rowind, _, _, lo = _matrix("chain", 1, 1, "f64", 3)
    S = SelInv(n, colptr, rowind, None, batch=1, cap=1, relax=0.0)
    S._alloc(False)
    ldlt = torch.from_numpy(S.factor_host(lo)).cuda()
    at = S.packed_index()
    assert len(at) == 3  # D_0, L_10, D_1
    ldlt[0, int(at[1])] = float("inf")
    st = torch.cuda.current_stream().cuda_stream
    capi.selinv_normalize_run(S.h, ldlt, S._bufs["panels"], S._bufs["x"], S._bufs["work"], None, st)
    S.sync()
    x = S.panels_view("x").cpu().numpy()[0, at]
    print(f"  x = {x}", flush=True)
    assert np.isposinf(x[0]) and np.isneginf(x[1]) and np.isfinite(x[2])
    S.close()
