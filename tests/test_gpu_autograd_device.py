"""SelInvFunction's forward factors on the GPU: a singular matrix raises there,
and the context goes on with the next one."""

import numpy as np
import pytest
import torch

from tests._ref import workload


@pytest.mark.gpu
@pytest.mark.parametrize("bad", [0.0, float("nan"), float("inf")])
def test_forward_reports_a_bad_pivot(bad):
    from paper_1604_02528_amd import SelInv, SelInvFunction
    from paper_1604_02528_amd.capi import SelinvError

    w = workload("C4s")
    S = SelInv(w.n, w.colptr, w.rowind, w.perm, dtype="f64", batch=2)
    good = torch.from_numpy(np.repeat(w.values, 2, axis=0)).to("cuda").requires_grad_(True)
    vals = good.detach().clone()
    vals[1, int(w.colptr[int(w.perm[0])])] = bad
    with pytest.raises(SelinvError) as ei:
        SelInvFunction.apply(vals.requires_grad_(True), S)
    assert ei.value.status == 3 and ei.value.info == (0, 1)
    x, logdet = SelInvFunction.apply(good, S)
    logdet.sum().backward()
    # d log det A / da = A^{-1}: twice the stored entry off the diagonal
    cols = np.repeat(np.arange(w.n), np.diff(w.colptr))
    two = torch.from_numpy(np.where(w.rowind == cols, 1.0, 2.0)).to("cuda")
    err = (good.grad - two * x).abs().max() / x.abs().max()
    # W = 0: the reverse sweep contributes zeros, so only the doubling rounds
    assert float(err.detach()) <= 4 * np.finfo(float).eps
    S.close()
