"""torch.autograd binding of the selected inversion and its adjoint (float64 and
complex128).

    S = SelInv(n, colptr, rowind, perm, batch=B)
    x, logdet = SelInvFunction.apply(values, S)   # values [B, nnz(A)], requires_grad
    loss = (c * x[:, diag]).sum() + logdet.sum()
    loss.backward()                               # values.grad = dloss/dvalues

The forward factors on the GPU, where siblings' updates meet in atomic adds: x
and logdet agree from run to run to rounding only, as with the host
factorization on several threads.  SelInvFunction.apply(values, S, False) factors
on the host; with SelInv(..., nthreads=1) both are then repeatable bit for bit
(the traversal has no atomics; the reverse sweep has, so gradients agree to
rounding either way).

x holds the selected entries of A^{-1} on A's stored lower pattern (original
indexing), logdet the log-determinants.  Gradients use the stored-value
convention: an off-diagonal value stands for both (i, j) and (j, i).  The
backward pass hands dloss/dx to the library's scatter (panel layout) and its
reverse sweep (selinv_backward), which also adds the log-det term
d log det A / dA = A^{-1}; no arithmetic happens here.  S holds the buffers of
the last forward call: a backward whose forward is no longer the latest
factorization of S raises instead of differentiating the wrong matrix.

For complex-symmetric A the library's adjoint is the holomorphic one (plain
transposes).  torch passes conjugate cotangents (dL/d conj(y) of a real loss L)
and expects them back for the input, so the binding conjugates gx and glogdet
on the way in and the result on the way out: for a holomorphic map with
Jacobian J that is exactly J^H g.
"""

from __future__ import annotations

import torch

from .capi import ESINGULAR, SelinvError
from .selinv import SelInv


def _selected(values, S, on_device):
    """Selected entries and log det of the values' matrices.  A bad pivot of the
    device factorization raises at S.logdet(), which waits for the device."""
    S.factor(values.detach(), want_dtilde=True, on_device=on_device)
    S.run()
    return S.extract(), S.logdet()


class SelInvFunction(torch.autograd.Function):
    @staticmethod
    def forward(ctx, values, S: SelInv, on_device=None):
        # On the GPU unless asked otherwise (the LU form has a host
        # factorization only): the host one is 30 of the 33 ms of a 200 x 200
        # GMRF's training step, most of it the panels' way through host memory.
        if on_device is None:
            on_device = not S.is_lu
        try:
            x, logdet = _selected(values, S, on_device)
        except SelinvError as e:
            if not on_device or e.status != ESINGULAR:
                raise
            # a zero or non-finite pivot is the host factorization's to report: it
            # leaves S unfactored (or finds a pivot that rounding made zero here)
            x, logdet = _selected(values, S, False)
        logdet = torch.as_tensor(logdet, dtype=S.scalar_dtype, device=x.device)
        ctx.S = S
        ctx.generation = S.generation
        ctx.in_device = values.device
        return x, logdet

    @staticmethod
    def backward(ctx, gx, glogdet):
        S = ctx.S
        if S.generation != ctx.generation:
            raise RuntimeError("SelInvFunction.backward: S was factored again after this forward call; "
                               "run each forward's backward before the next forward on the same SelInv")
        if gx is None:
            gx = torch.zeros((S.batch, S.nnzA), dtype=S.scalar_dtype, device=S.device)
        wl = glogdet
        if S.is_complex:
            gx = gx.conj().resolve_conj()
            wl = None if wl is None else wl.conj().resolve_conj()
        xbar = S.scatter(gx.contiguous())
        abar = S.backward(xbar, None if wl is None else wl.contiguous())
        if S.is_complex:
            abar = abar.conj().resolve_conj()
        return abar.to(ctx.in_device), None, None
