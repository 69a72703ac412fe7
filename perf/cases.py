"""Performance cases of the selected-inversion library.

Four operations, the ones a program of this library runs on the GPU:

* ``solve``     a pole-expansion or marginal-variance program: the values of the
                shifted matrices are on the device, it wants the selected
                entries of their inverses (device factorization, normalization,
                traversal, extraction).
* ``selinv``    the paper's path: LDL^T panels are in device memory (an external
                solver or an earlier factorization), one ``selinv_normalize_run``
                turns them into the selected inverse X.
* ``backward``  the adjoint alone: a gradient on A's pattern goes through
                ``scatter`` and the reverse sweep.
* ``train``     a training step of a Gaussian Markov random field:
                ``SelInvFunction`` forward (selected inverse, log det) and backward.

over six matrix families on grids: ``lap2d`` (5-point Laplacian plus shift),
``gmrf2d`` (GMRF precision), ``lap3d`` (weighted 7-point Laplacian plus shift),
``shift3d`` (complex-symmetric shifts H - z S of it), ``sten27``
(complex-symmetric 27-point stencil minus shifts), ``herm3d`` (Hermitian magnetic
Laplacian plus shifts) and ``conv3d`` (unsymmetric convection-diffusion, LU form).
"""

from __future__ import annotations

import math
from functools import lru_cache

import numpy as np
import torch

from paper_1604_02528_amd import SelInv, SelInvFunction, capi

DTYPE = {"lap2d": "f64", "gmrf2d": "f64", "lap3d": "f64", "shift3d": "c128", "sten27": "c128", "herm3d": "h128",
         "conv3d": "lu64"}


def _case(name, op, family, nx, ny, nz=1, batch=1):
    return {"name": name, "op": op, "family": family, "nx": nx, "ny": ny, "nz": nz, "batch": batch}


def listed():
    return [
        # the smallest real call: one 2-D problem of a thousand unknowns, where launches and latency count
        _case("solve_lap2d_31x31", "solve", "lap2d", 31, 31),
        # a handful of small odd-sized 3-D problems in one batch
        _case("solve_lap3d_21x13x9_b5", "solve", "lap3d", 21, 13, 9, 5),
        # one mid-size real 3-D problem from its values to the selected inverse
        _case("solve_lap3d_40x40x40", "solve", "lap3d", 40, 40, 40),
        # complex shifts of a 27-point operator, odd extents: wide supernodes, ragged tiles
        _case("solve_sten27_23x17x29_b3", "solve", "sten27", 23, 17, 29, 3),
        # a pole expansion over Hermitian matrices, 16 shifts in one batch
        _case("solve_herm3d_30x30x30_b16", "solve", "herm3d", 30, 30, 30, 16),
        # the traversal on one real 3-D problem whose panels come from a solver
        _case("selinv_lap3d_40x40x40", "selinv", "lap3d", 40, 40, 40),
        # the traversal on a pole expansion of 32 complex shifts
        _case("selinv_shift3d_30x30x30_b32", "selinv", "shift3d", 30, 30, 30, 32),
        # the traversal on the largest grid the library is run on, two of its complex shifts
        _case("selinv_sten27_64x64x64_b2", "selinv", "sten27", 64, 64, 64, 2),
        # the LU form: unsymmetric values, both triangles of the inverse
        _case("selinv_conv3d_30x30x30_b4", "selinv", "conv3d", 30, 30, 30, 4),
        # the adjoint of a 2-D GMRF's marginal variances
        _case("backward_gmrf2d_200x200", "backward", "gmrf2d", 200, 200),
        # the adjoint of complex 3-D shifts with log-det terms
        _case("backward_shift3d_20x20x20_b4", "backward", "shift3d", 20, 20, 20, 4),
        # one training step of the GMRF through autograd
        _case("train_gmrf2d_200x200", "train", "gmrf2d", 200, 200),
    ]


# (op, family, shortest and longest extent, most unknowns, most matrices)
_RANGES = [
    ("solve", "lap2d", 20, 300, 40000, 8),
    ("solve", "lap3d", 7, 56, 64000, 5),
    ("solve", "sten27", 6, 32, 16000, 4),
    ("solve", "herm3d", 8, 40, 27000, 16),
    ("selinv", "lap3d", 10, 56, 64000, 4),
    ("selinv", "shift3d", 8, 40, 27000, 32),
    ("selinv", "sten27", 10, 80, 200000, 2),
    ("selinv", "conv3d", 8, 40, 27000, 4),
    ("backward", "gmrf2d", 20, 260, 40000, 2),
    ("backward", "shift3d", 6, 26, 8000, 4),
    ("train", "gmrf2d", 20, 260, 40000, 1),
]


def draw(rng):
    op, family, lo, hi, most, batch = rng.choice(_RANGES)
    ext = lambda: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    while True:
        d = [ext(), ext(), 1 if family.endswith("2d") else ext()]
        if d[0] * d[1] * d[2] <= most:
            break
    b = int(round(math.exp(rng.uniform(0.0, math.log(batch)))))
    return {"op": op, "family": family, "nx": d[0], "ny": d[1], "nz": d[2], "batch": b}


# --------------------------------------------------------------------------
# patterns (one per grid, shared by every seed)
# --------------------------------------------------------------------------

def _dissection(nx, ny, nz):
    """Geometric nested dissection, new -> old: split the longest axis at its
    middle plane, number both halves, then the plane; boxes below 3 are leaves."""
    idx = np.arange(nx * ny * nz, dtype=np.int64).reshape(nz, ny, nx)
    out = []

    def box(a):
        if a.size == 0:
            return
        ax = max((2, 1, 0), key=lambda q: a.shape[q])
        m = a.shape[ax]
        if m < 3:
            out.append(a.ravel())
            return
        cut = [slice(None)] * 3
        for part in (slice(0, m // 2), slice(m // 2 + 1, m)):
            cut[ax] = part
            box(a[tuple(cut)])
        cut[ax] = m // 2
        out.append(a[tuple(cut)].ravel())

    box(idx)
    return np.concatenate(out)


@lru_cache(maxsize=16)
def _pattern(family, nx, ny, nz):
    """Lower CSC pattern with the grid edges behind it: colptr, rowind, perm,
    edge ends a < b, ghost points (one per missing axis neighbour) and the
    position of each [diagonal, edges] entry in CSC order."""
    idx = np.arange(nx * ny * nz, dtype=np.int64).reshape(nz, ny, nx)
    n = idx.size
    if family == "sten27":
        offs = [(z, y, x) for z in (-1, 0, 1) for y in (-1, 0, 1) for x in (-1, 0, 1) if (z, y, x) > (0, 0, 0)]
    else:
        offs = [o for o, m in (((0, 0, 1), nx), ((0, 1, 0), ny), ((1, 0, 0), nz)) if m > 1]
    lo = lambda d, m: slice(max(0, -d), m - max(0, d))
    a = np.concatenate([idx[tuple(lo(d, m) for d, m in zip(o, idx.shape))].ravel() for o in offs])
    b = np.concatenate([idx[tuple(lo(-d, m) for d, m in zip(o, idx.shape))].ravel() for o in offs])
    ghost = np.concatenate([np.take(idx, side, axis=ax).ravel() for ax in range(3) if idx.shape[ax] > 1
                            for side in (0, -1)])
    rows = np.concatenate([idx.ravel(), np.maximum(a, b)])
    cols = np.concatenate([idx.ravel(), np.minimum(a, b)])
    order = np.lexsort((rows, cols))
    colptr = np.concatenate([[0], np.cumsum(np.bincount(cols, minlength=n))]).astype(np.int64)
    return colptr, rows[order], _dissection(nx, ny, nz), a, b, ghost, order


def _dims(case):
    return case["family"], case["nx"], case["ny"], case["nz"]


def _values(case, seed):
    """[batch, nnz] values of the family's matrices (LU: [batch, 2 nnz]: the
    lower entries, then their mirrors)."""
    colptr, rowind, perm, a, b, ghost, order = _pattern(*_dims(case))
    n, m, B, fam = len(perm), len(a), case["batch"], case["family"]
    rng = np.random.default_rng(seed)
    up = None
    ends = lambda w: np.bincount(a, w, n) + np.bincount(b, w, n)
    w = rng.uniform(0.5, 1.5, m)
    ghosts = np.bincount(ghost, rng.uniform(0.5, 1.5, len(ghost)), n)
    z = rng.uniform(-2.0, 2.0, B) + 1j * 10.0 ** rng.uniform(-3.0, 0.0, B)  # complex shifts z_l
    sig = 10.0 ** rng.uniform(-2.0, 0.0, B)                                 # positive shifts
    if fam == "lap2d":
        off, diag, shift = -np.ones(m), ends(np.ones(m)) + np.bincount(ghost, minlength=n), 0.1 * np.ones(B)
        shift = shift + 0.05 * rng.uniform(0, 1, B)
    elif fam == "gmrf2d":
        w = np.exp(rng.normal(0.0, 0.3, m))
        off, diag, shift = -w, ends(w), np.full(B, 0.25)
    elif fam == "lap3d":
        off, diag, shift = -w, ends(w) + ghosts, 0.04 + sig
    elif fam == "shift3d":
        off, diag, shift = -w, ends(w) + ghosts, -z[:, None] * rng.uniform(0.8, 1.2, n)
    elif fam == "herm3d":
        off = -w * np.exp(-1j * rng.uniform(-np.pi, np.pi, m))
        diag, shift = ends(w) + ghosts, sig
    elif fam == "conv3d":
        p = rng.uniform(-0.5, 0.5, m)
        off, up = -w * (1 + p), -w * (1 - p)
        diag, shift = ends(w * (1 + np.abs(p))) + ghosts, sig
    else:  # sten27
        off = rng.uniform(-1.0, 0.0, m) + 1j * rng.uniform(-0.1, 0.1, m)
        diag, shift = ends(np.abs(off)) + 3.0 + 1j * rng.uniform(-0.1, 0.1, n), -z
    shift = shift[:, None] if shift.ndim == 1 else shift
    d = diag[None, :] + shift
    build = lambda o: np.concatenate([d, np.broadcast_to(o, (B, m))], axis=1)[:, order]
    v = build(off) if up is None else np.concatenate([build(off), build(up)], axis=1)
    return np.ascontiguousarray(v)


def _context(case, adjoint, device="cuda", batch=None):
    colptr, rowind, perm = _pattern(*_dims(case))[:3]
    return SelInv(len(perm), colptr, rowind, perm, dtype=DTYPE[case["family"]], batch=batch or case["batch"],
                  adjoint=adjoint, device=device)


def _scalar(case):
    return torch.complex128 if DTYPE[case["family"]] in ("c128", "h128") else torch.float64


def prepare(case, seed):
    op = case["op"]
    S = _context(case, adjoint=op in ("backward", "train"))
    host = _values(case, seed)
    rng = np.random.default_rng(seed + 1)
    st = {"op": op, "S": S}
    if op == "selinv":
        # caller-owned buffers of the C interface; the LDL^T panels as a solver leaves them
        buf = lambda nbytes: torch.zeros(int(nbytes), dtype=torch.uint8, device="cuda")
        size, stream = S.sizes, torch.cuda.current_stream().cuda_stream
        st["panels"], st["x"], st["work"] = buf(size.panels_bytes), buf(size.x_bytes), buf(size.work_bytes)
        if S.is_lu:
            st["ldlt"] = torch.from_numpy(S.factor_host(host)).cuda()
        else:
            st["ldlt"] = buf(size.panels_bytes)
            capi.selinv_factor_device(S.h, torch.from_numpy(host).cuda(), st["ldlt"], st["work"], stream)
            S.sync()
        shape = (case["batch"], S.panel_elems)
        st["X"] = st["x"].view(_scalar(case))[:shape[0] * shape[1]].view(shape)
        return st
    st["values"] = torch.from_numpy(host).cuda()
    if op == "backward":
        S.factor(st["values"], want_dtilde=True, on_device=True)
        S.run()
        g = rng.standard_normal((2,) + host.shape)
        wl = rng.standard_normal((2, case["batch"]))
        cx = _scalar(case).is_complex
        st["gx"] = torch.from_numpy(g[0] + 1j * g[1] if cx else g[0]).cuda()
        st["wl"] = torch.from_numpy(wl[0] + 1j * wl[1] if cx else wl[0]).cuda()
    elif op == "train":
        colptr = _pattern(*_dims(case))[0]
        st["values"].requires_grad_(True)
        st["diag"] = torch.from_numpy(colptr[:-1]).cuda()
        st["c"] = torch.from_numpy(rng.uniform(0.0, 1.0, len(colptr) - 1)).cuda()
    return st


def run(st):
    S, op = st["S"], st["op"]
    if op == "solve":
        S.factor(st["values"], on_device=True)
        S.run()
        return S.extract()
    if op == "selinv":
        capi.selinv_normalize_run(S.h, st["ldlt"], st["panels"], st["x"], st["work"], None,
                                  torch.cuda.current_stream().cuda_stream)
        return st["X"]
    if op == "backward":
        return S.backward(S.scatter(st["gx"]), st["wl"])
    x, logdet = SelInvFunction.apply(st["values"], S)
    loss = (st["c"] * x[:, st["diag"]]).sum() + logdet.sum()
    grad, = torch.autograd.grad(loss, st["values"])
    return {"x": x.detach(), "logdet": logdet.detach(), "grad": grad}


# --------------------------------------------------------------------------
# what a pass cannot do without, and its exact outputs
# --------------------------------------------------------------------------

@lru_cache(maxsize=64)
def _counts(family, nx, ny, nz):
    """Of one matrix: stored entries of A and of L, and the real operations of
    the factorization and of the selected inversion (a multiply-add of complex
    numbers is 8)."""
    case = {"family": family, "nx": nx, "ny": ny, "nz": nz, "batch": 1}
    S = _context(case, adjoint=False, device="cpu")
    sym = S.symbolic()
    S.close()
    s = np.diff(sym["xsuper"]).astype(np.float64)
    c = np.diff(sym["rowptr"]).astype(np.float64)
    m = sym["colcount"].astype(np.float64) - 1.0
    mul = 4.0 if _scalar(case).is_complex else 1.0
    lu = 2.0 if DTYPE[family] == "lu64" else 1.0
    fac = mul * lu * float(np.sum(m * (m + 1.0)))
    # normalization: Lhat = L_C L_KK^{-1} and the inverse of the pivot block
    norm = mul * lu * float(np.sum(c * s * s + s * s * s))
    inv = mul * float(np.sum(lu * 2.0 * c * c * s + 2.0 * c * s * s))
    return int(_pattern(family, nx, ny, nz)[0][-1]), int(sym["nnzL"]), fac, norm, inv


def work(case):
    nnz, nnzl, fac, norm, inv = _counts(*_dims(case))
    B, size = case["batch"], _scalar(case).itemsize
    lu = 2 if DTYPE[case["family"]] == "lu64" else 1
    op = case["op"]
    if op == "solve":
        return {"bytes": B * size * 2 * nnz, "flops": B * (fac + norm + inv)}
    if op == "selinv":
        return {"bytes": B * size * 2 * nnzl * lu, "flops": B * (norm + inv)}
    # the reverse sweep: two products with X_{C,C}-sized operands, the rank-2s update and the s x s steps
    back = 2.0 * inv
    if op == "backward":
        return {"bytes": B * size * (2 * nnz + 3 * nnzl), "flops": B * back}
    return {"bytes": B * size * 3 * nnz, "flops": B * (fac + norm + inv + back)}


def exact(case, seed):
    """Dense 64-bit inverses (float64 or complex128), for matrices small enough."""
    colptr, rowind, perm = _pattern(*_dims(case))[:3]
    n, B, op = len(perm), case["batch"], case["op"]
    if op == "selinv" or n > 3000 or float(n) ** 3 * B * (4 if _scalar(case).is_complex else 1) > 2e11:
        return None
    host = _values(case, seed)
    cols = np.repeat(np.arange(n), np.diff(colptr))
    rng = np.random.default_rng(seed + 1)
    if op == "backward":
        g, wl = rng.standard_normal((2,) + host.shape), rng.standard_normal((2, B))
        cx = _scalar(case).is_complex
        g, wl = (g[0] + 1j * g[1], wl[0] + 1j * wl[1]) if cx else (g[0], wl[0])
    elif op == "train":
        g, wl = np.zeros(host.shape), np.ones(B)
        g[:, colptr[:-1]] = rng.uniform(0.0, 1.0, n)
    half = np.where(rowind == cols, 1.0, 0.5)
    xs, grads, logdets = [], [], []
    for l in range(B):
        A = np.zeros((n, n), dtype=host.dtype)
        A[cols, rowind] = np.conj(host[l]) if DTYPE[case["family"]] == "h128" else host[l]
        A[rowind, cols] = host[l]
        X = np.linalg.inv(A)
        xs.append(X[rowind, cols])
        if op != "solve":
            W = np.zeros((n, n), dtype=host.dtype)
            W[cols, rowind] = W[rowind, cols] = g[l] * half
            G = -X @ W @ X + wl[l] * X
            grads.append(G[rowind, cols] / half)
            logdets.append(np.linalg.slogdet(A)[1])
    if op == "solve":
        return np.stack(xs)
    if op == "backward":
        return np.stack(grads)
    return {"x": np.stack(xs), "logdet": np.array(logdets), "grad": np.stack(grads)}
