"""SelInvFunction beside its default: the host factorization on request, on one
thread repeatable bit for bit, and the state that a forward with a bad pivot
leaves."""

import numpy as np
import pytest
import torch

from tests._ref import workload


@pytest.mark.gpu
@pytest.mark.parametrize("name,scale,dtype", [("C4", 60, "f64"), ("C3", 9, "c128")])
def test_host_factorization_is_repeatable(name, scale, dtype):
    from paper_1604_02528_amd import SelInv, SelInvFunction

    w = workload(name, scale)
    # (on several threads siblings reach an ancestor's panel in any order)
    S = SelInv(w.n, w.colptr, w.rowind, w.perm, dtype=dtype, batch=w.batch, nthreads=1)
    S.factor(w.values, want_dtilde=True)  # host factorization
    S.run()
    x0, ld0 = S.extract().cpu(), S.logdet()
    vals = torch.from_numpy(w.values).cuda().requires_grad_(True)
    for _ in range(3):
        x, logdet = SelInvFunction.apply(vals, S, False)
        assert torch.equal(x.detach().cpu(), x0) and np.array_equal(logdet.detach().cpu().numpy(), ld0)
    g, = torch.autograd.grad(logdet.real.sum(), vals)
    x, logdet = SelInvFunction.apply(vals, S)
    h, = torch.autograd.grad(logdet.real.sum(), vals)
    assert float((g - h).abs().max()) <= 1e-13 * float(g.abs().max()) * max(1.0, float(x.detach().abs().max()))
    S.close()


@pytest.mark.gpu
def test_a_bad_pivot_leaves_the_context_unfactored():
    from paper_1604_02528_amd import SelInv, SelInvFunction
    from paper_1604_02528_amd.capi import SelinvError

    w = workload("C4s")
    S = SelInv(w.n, w.colptr, w.rowind, w.perm, dtype="f64", batch=1)
    good = torch.from_numpy(w.values).cuda().requires_grad_(True)
    SelInvFunction.apply(good, S)
    bad = good.detach().clone()
    bad[0, int(w.colptr[int(w.perm[0])])] = 0.0
    with pytest.raises(SelinvError) as ei:
        SelInvFunction.apply(bad.requires_grad_(True), S)
    assert ei.value.status == 3
    for call in (S.run, S.logdet):
        with pytest.raises(SelinvError) as ei:
            call()
        assert ei.value.status == 6
    S.close()
