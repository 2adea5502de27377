"""The even-step panel where one workgroup holds every row (agreement in LDS) and
at the orders around it: 448, 224 and 112 rows for blocks of up to 64, 128 and
256 columns.  Pivots, alphas and log|Pf| against the oracle's even-step
Pfaffian; a zero column and ties between waves; non-finite input returns."""
from __future__ import annotations

import numpy as np
import pytest

import synth
from test_gpu_pfaffian_direct import check_direct, gpu_direct

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nb", [(2, 64), (112, 256), (114, 256), (224, 128), (226, 128), (448, 64), (450, 64),
                                  (448, 128)])
def test_one_workgroup_edges(n, nb):
    print(f"[pair] n={n} nb={nb}", flush=True)
    check_direct(synth.skew_gauss(n, 700 + n), nb)


@pytest.mark.parametrize("n", [8, 140, 224])
def test_one_workgroup_zero_columns_and_ties(n):
    """4 x 4 blocks: exact zeros and all-zero waves at every step."""
    check_direct(synth.skew_blockdiag4(n, 31), 128)


@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_one_workgroup_non_finite(value):
    X = synth.skew_gauss(96, 5)
    X[40, 3], X[3, 40] = value, -value
    ipiv, *_ = gpu_direct(X, 64)
    assert ((ipiv >= 0) & (ipiv < 96)).all()
