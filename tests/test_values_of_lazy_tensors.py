"""Values given as lazily conjugated or negated torch tensors: what reaches the
library's device factorization is the memory of the formed tensor."""

import numpy as np
import pytest
import torch

from tests._ref import workload


@pytest.mark.parametrize("view", ["conj", "neg", "conj of a slice", "transposed"])
def test_values_are_formed(view):
    from paper_1604_02528_amd import SelInv

    w = workload("C3", 6, 2)
    S = SelInv(w.n, w.colptr, w.rowind, w.perm, dtype="c128", batch=2, device="cpu", adjoint=False)
    z = torch.from_numpy(w.values)
    lazy = {"conj": lambda: z.conj(), "neg": lambda: torch._neg_view(z),
            "conj of a slice": lambda: torch.cat([z, z], dim=1)[:, :z.shape[1]].conj(),
            "transposed": lambda: z.t().contiguous().t()}[view]()
    v = S._values_device(lazy)
    buf = (2 * v.numel() * np.ctypeslib.ctypes.c_double).from_address(v.data_ptr())
    got = np.frombuffer(buf, dtype=np.complex128).reshape(2, -1)
    want = {"neg": -w.values, "transposed": w.values}.get(view, w.values.conj())
    assert np.array_equal(got, want)


@pytest.mark.gpu
def test_forward_of_conjugated_values():
    from paper_1604_02528_amd import SelInv, SelInvFunction

    w = workload("C3", 6, 2)
    S = SelInv(w.n, w.colptr, w.rowind, w.perm, dtype="c128", batch=2)
    z = torch.from_numpy(w.values).cuda()
    x, logdet = SelInvFunction.apply(z.conj(), S)
    y, ld = SelInvFunction.apply(z, S)
    # A conj -> A^{-1} conj; atomics may order the updates differently
    assert float((x - y.conj()).abs().max()) <= 1e-12 * float(y.abs().max())
    assert float((logdet - ld.conj()).abs().max()) <= 1e-12 * float(ld.abs().max())
    S.close()
