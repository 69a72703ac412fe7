"""The device factorization's kernels at the edges of their blocks: one node of
width s with c rows below it, for s and c around 16 (one wavefront's block),
64 and 128 (strips of the single-wavefront kernel, the update's tiles), 128
columns (one column block) and 256 (the widest supernode)."""

import numpy as np
import pytest

from oracle import factor, selinv, symbolic


def _clique(s, c, batch, kind, seed, scale=1.0):
    """s columns coupled to each other and to c rows, a second clique of two
    columns coupled to all but the first of those rows (it keeps the first
    clique a supernode of its own), and the c rows coupled to each other:
    strictly diagonally dominant values."""
    n = s + 2 + c
    full = np.zeros((n, n), bool)
    full[:s, :s] = full[s + 2:, :s] = full[s + 2:, s + 2:] = True
    full[s:s + 2, s:s + 2] = full[s + 3:, s:s + 2] = True
    cols, rows = np.nonzero(np.tril(full).T)  # column by column
    colptr = np.concatenate([[0], np.cumsum(np.bincount(cols, minlength=n))]).astype(np.int64)
    rng = np.random.default_rng(seed)
    v = rng.uniform(-1.0, 1.0, (batch, rows.size))
    if kind != "f64":
        v = v + 1j * rng.uniform(-1.0, 1.0, v.shape)
    v /= n
    d = rows == cols
    v[:, d] = 2.0 + rng.uniform(0.0, 1.0, (batch, n))
    if kind == "c128":
        v[:, d] += 1j * rng.uniform(-0.5, 0.5, (batch, n))
    return n, colptr, rows.astype(np.int64), v * scale


def check_node(s, c, kind, scale=1.0):
    from paper_1604_02528_amd import SelInv

    print(f"factor block case s={s} c={c} {kind} scale={scale}", flush=True)
    n, colptr, rowind, vals = _clique(s, c, 2, kind, 100 * s + c, scale)
    sym = symbolic.analyze(n, colptr, rowind, None, cap=256, relax=0.0)
    assert sym.width(0) == s and sym.rows[0].shape[0] == c
    S = SelInv(n, colptr, rowind, None, dtype=kind, batch=2, relax=0.0)
    P = S.factor_device(vals).cpu().numpy()[:, S.packed_index()]
    S.sync()
    herm = kind == "h128"
    for l in range(2):
        L, D = factor.to_dense_L(sym, selinv.unflatten(sym, P[l]))
        D = D / scale
        Lt = L.conj().T if herm else L.T
        B = np.zeros((n, n), vals.dtype)
        cols = np.repeat(np.arange(n), np.diff(colptr))
        B[cols, rowind] = (vals[l].conj() if herm else vals[l]) / scale
        B[rowind, cols] = vals[l] / scale
        # componentwise backward error of an unpivoted LDL^T: gamma_n |L||D||L^T| (x 4 for complex products)
        bound = 8 * n * np.finfo(float).eps * np.max((np.abs(L) * np.abs(D)) @ np.abs(Lt))
        err = np.max(np.abs((L * D[None, :]) @ Lt - B))
        print(f"  matrix {l}: max |L D L^T - B| {err:.2e}, bound {bound:.2e}", flush=True)
        assert err <= bound
    S.close()


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["f64", "c128", "h128"])
@pytest.mark.parametrize("scale", [1e-190, 1e190])
@pytest.mark.parametrize("s,c", [(7, 20), (16, 100), (40, 30)])
def test_pivots_beyond_the_fast_reciprocal(s, c, scale, kind):
    """Pivots outside 2^-500 .. 2^500 (complex: their squared moduli) take the
    full divisions: L is that of the unscaled matrix, D is scaled."""
    check_node(s, c, kind, scale)


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["f64", "c128", "h128"])
@pytest.mark.parametrize("s,c", [(1, 1), (3, 17), (15, 16), (16, 64), (13, 65), (16, 128), (16, 129), (17, 5),
                                 (48, 63), (64, 130), (127, 3), (128, 70), (129, 64), (144, 200), (255, 33),
                                 (256, 257)])
def test_one_node(s, c, kind):
    check_node(s, c, kind)
