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
