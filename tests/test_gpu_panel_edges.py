"""Panel sizes at the borders of its variants, against the oracle: the last
order that one workgroup holds (it agrees on its pivots without records) and
the first that needs two, for one, two and four lanes per row; blocks narrower
than one group of the g ring (4, 8, 16 steps), of one group and of one more.
Bars as in the factorization tests (normwise 1e-10 in fp64)."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import synth
from gpu_util import compare_factors, gpu_factor

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("n,nb", [(513, 64), (514, 64), (257, 128), (258, 128), (129, 256), (130, 256),
                                  (40, 3), (40, 4), (40, 5), (300, 72), (300, 73), (600, 136), (600, 145)])
def test_panel_edges(n, nb, dtype):
    X = synth.skew_gauss(n, 4000 + n + nb).astype(dtype)
    print(f"[edges] n={n} nb={nb} {np.dtype(dtype).name}", flush=True)
    packed, ipiv, logabs, sign, _ = gpu_factor(X, nb=nb)
    info = compare_factors(X, packed, ipiv, dtype)
    if dtype == np.float64:
        assert info["first_pivot_mismatch"] == n
    assert oracle.residual(X, packed, ipiv) <= 10


@pytest.mark.parametrize("n", [250, 500])
def test_one_workgroup_zero_columns_and_ties(n):
    """4 x 4 blocks on the diagonal: columns of zeros (every wave ties at zero)
    and steps without any nonzero pivot."""
    X = synth.skew_blockdiag4(n // 4 * 4, 4100 + n)
    packed, ipiv, logabs, sign, _ = gpu_factor(X, nb=64)
    compare_factors(X, packed, ipiv, np.float64)
    ref, ri = oracle.ltlt(X)
    rl, rs = oracle.pfaffian_packed(ref, ri)
    assert int(sign) == rs and abs(float(logabs) - rl) <= 1e-9 * abs(rl)
