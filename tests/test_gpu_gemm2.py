"""GEMM-2 as a product over row ranges: nodes of width s with c rows below
around the edges of its rule (s = 64 / 65, three / four row tiles), of its 64
x 64 tiles and of its row ranges, against numpy's dense inverse, for every
scalar type."""

import numpy as np
import pytest

from oracle import selinv, symbolic
from tests.test_gpu_factor_blocks import _clique
from tests.test_oracle_lu import dense_original_lu, selected_from_dense_lu


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["f64", "c128", "h128", "lu64"])
@pytest.mark.parametrize("s,c,batch", [(64, 256, 1), (65, 192, 1), (65, 193, 1), (66, 257, 2), (127, 320, 1),
                                       (128, 385, 3), (129, 511, 1), (200, 700, 1), (256, 449, 2), (255, 832, 1)])
def test_one_node(s, c, batch, kind):
    from paper_1604_02528_amd import SelInv

    print(f"gemm2 case s={s} c={c} batch={batch} {kind}", flush=True)
    lu = kind == "lu64"
    n, colptr, rowind, lo = _clique(s, c, batch, "f64" if lu else kind, 100 * s + c)
    cols = np.repeat(np.arange(n), np.diff(colptr))
    up = lo.conj() if kind == "h128" else lo
    if lu:
        up = lo[:, ::-1] * 0.5
        up[:, rowind == cols] = lo[:, rowind == cols]
    sym = symbolic.analyze(n, colptr, rowind, None, cap=256, relax=0.0)
    assert sym.width(0) == s and sym.rows[0].shape[0] == c
    S = SelInv(n, colptr, rowind, None, dtype=kind, batch=batch, relax=0.0)
    S.factor(np.concatenate([lo, up], axis=1) if lu else lo)
    S.run()
    S.sync()
    X = S.to_host("x")
    for l in range(batch):
        if lu:
            A = dense_original_lu(n, colptr, rowind, lo[l], up[l])
        else:
            A = np.zeros((n, n), lo.dtype)
            A[cols, rowind] = up[l]
            A[rowind, cols] = lo[l]
        Ainv = np.linalg.inv(A)
        RL, RU = selected_from_dense_lu(sym, Ainv)
        ref = selinv.flatten(sym, RL)
        if lu:
            ref = np.concatenate([ref, selinv.flatten(sym, RU)])
        # both inverses are backward stable on a dominant matrix: n eps kappa each, a few such terms
        bound = 8 * n * np.finfo(float).eps * np.linalg.cond(A, np.inf)
        err = np.max(np.abs(X[l] - ref)) / np.max(np.abs(ref))
        print(f"  matrix {l}: {err:.2e}, bound {bound:.2e}", flush=True)
        assert err <= bound
    S.close()
