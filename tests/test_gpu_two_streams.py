"""Plans on either side of the work from which a traversal takes two streams
(halves of a batch, subtree groups of a single matrix): X is bit for bit that
of a traced run, which keeps one stream and a launch per depth."""

import numpy as np
import pytest
import torch

from tests._ref import workload
from tests.test_gpu_batch_halves import _run_three_ways


@pytest.mark.gpu
@pytest.mark.parametrize("name,scale,batch", [("C3", 24, 4), ("C3", 24, 5), ("H3", 24, 5), ("U3", 24, 2), ("U3", 24, 3),
                                              ("C2", 30, None), ("C2", 34, None)])
def test_either_side_of_the_rule(name, scale, batch):
    from paper_1604_02528_amd import SelInv

    w = workload(name, scale, batch)
    print(f"two streams case {name} scale={scale} batch={batch}", flush=True)
    S = SelInv(w.n, w.colptr, w.rowind, w.perm, dtype=w.dtype, batch=w.batch, cap=w.cap, relax=0.05, adjoint=False)
    S._alloc(False)
    ldlt = torch.from_numpy(S.factor_host(w.values)).cuda()
    xa, xb, xc = _run_three_ways(S, ldlt)
    assert np.array_equal(xa, xb) and np.array_equal(xa, xc)
    S.close()
