"""Small nodes of the LU form (one wavefront each) at the edges of their range:
one node of width s with c rows below it, for s around 8 and c around 8, 16,
32 and 64, against numpy's dense inverse; and the plans that must do without
such nodes so that the fixed work area still holds them."""

import numpy as np
import pytest

from oracle import selinv, symbolic
from tests._ref import workload
from tests.test_gpu_factor_blocks import _clique
from tests.test_oracle_lu import dense_original_lu, selected_from_dense_lu


@pytest.mark.gpu
@pytest.mark.parametrize("s,c", [(1, 1), (8, 1), (3, 7), (7, 8), (8, 9), (5, 15), (8, 16), (2, 17), (8, 31), (1, 32),
                                 (8, 33), (6, 63), (8, 64), (8, 65), (9, 64), (9, 8), (16, 20), (17, 20)])
def test_one_lu_node(s, c):
    from paper_1604_02528_amd import SelInv

    print(f"lu node case s={s} c={c}", flush=True)
    n, colptr, rowind, lo = _clique(s, c, 3, "f64", 100 * s + c)
    cols = np.repeat(np.arange(n), np.diff(colptr))
    up = lo[:, ::-1] * 0.5
    up[:, rowind == cols] = lo[:, rowind == cols]
    sym = symbolic.analyze(n, colptr, rowind, None, cap=256, relax=0.0)
    assert sym.width(0) == s and sym.rows[0].shape[0] == c
    S = SelInv(n, colptr, rowind, None, dtype="lu64", batch=3, relax=0.0)
    S.factor(np.concatenate([lo, up], axis=1))
    S.run()
    S.sync()
    X = S.to_host("x")
    for l in range(3):
        A = dense_original_lu(n, colptr, rowind, lo[l], up[l])
        Ainv = np.linalg.inv(A)
        RL, RU = selected_from_dense_lu(sym, Ainv)
        ref = np.concatenate([selinv.flatten(sym, RL), selinv.flatten(sym, RU)])
        # both inverses are backward stable on a dominant matrix: n eps kappa each, a few such terms
        bound = 8 * n * np.finfo(float).eps * np.linalg.cond(A, np.inf)
        err = np.max(np.abs(X[l] - ref)) / np.max(np.abs(ref))
        print(f"  matrix {l}: {err:.2e}, bound {bound:.2e}", flush=True)
        assert err <= bound
    S.close()


def test_offset_tables_leave_the_fixed_work_area_to_the_plan():
    """By batch, the plans of one pattern: those that fit the fixed work area
    have small nodes until their tables would be what exceeds it, then none;
    the first one too large by itself has them again."""
    from paper_1604_02528_amd import SelInv, capi

    w = workload("U3", 16, 1)

    def small_nodes(batch):
        S = SelInv(w.n, w.colptr, w.rowind, w.perm, dtype="lu64", batch=batch, relax=0.0)
        has = bool((capi.selinv_items(S.h, 2)[:, 0] == 1).any())
        S.close()
        return has

    seen = [small_nodes(b) for b in range(8, 18)]
    first = seen.index(False)
    again = seen.index(True, first)
    assert all(seen[:first]) and not any(seen[first:again]) and all(seen[again:])
