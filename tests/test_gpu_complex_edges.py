"""Complex panel sizes at the borders of its variants, against the oracle: the
last order that one workgroup holds and the first that needs two, for one, two
and four lanes per row; blocks narrower than a group of the g ring (2, 4, 8
steps), of one group and of one more; half and whole passes of the refresh.  Bars as
in the complex tests (normwise 1e-10 in complex128)."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import compare_factors, device_colmajor, host_packed

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nb", [(513, 32), (514, 32), (257, 64), (258, 64), (129, 128), (130, 128), (30, 1), (30, 2),
                                  (30, 3), (200, 36), (200, 37), (300, 72), (300, 73), (400, 100)])
def test_complex_panel_edges(n, nb):
    import paper_2005_06410_amd as lt
    X = synth.skew_gauss_complex(n, 7000 + n + nb)
    print(f"[complex edges] n={n} nb={nb}", flush=True)
    flat, A = device_colmajor(X)
    ipiv = lt.factor(A, nb=nb)
    torch.cuda.synchronize()
    lt.device_status()
    packed = host_packed(flat, n, n)
    info = compare_factors(X, packed, ipiv.cpu().numpy(), np.complex128)
    assert info["first_pivot_mismatch"] == n
    assert oracle.residual(X, packed, ipiv.cpu().numpy()) <= 10
