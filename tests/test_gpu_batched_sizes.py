"""The batched path at the borders of its size instances (16, 32, 48, 64), with
half blocks (no step past the eighth), batches that do not fill a workgroup,
ties and columns of zeros, against the oracle member by member.  Bars as in
the factorization tests."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import compare_factors

pytestmark = pytest.mark.gpu


def run(Xs, dtype):
    import paper_2005_06410_amd as lt
    batch, n = Xs.shape[0], Xs.shape[1]
    d = torch.from_numpy(np.ascontiguousarray(np.transpose(Xs, (0, 2, 1)))).cuda()
    A = d.as_strided((batch, n, n), (n * n, 1, n))
    ipiv, logabs, sign = lt.factor_batched(A)
    torch.cuda.synchronize()
    got = np.tril(np.transpose(d.cpu().numpy(), (0, 2, 1)), -1)
    return got, ipiv.cpu().numpy(), logabs.cpu().numpy(), sign.cpu().numpy()


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("n", [2, 9, 10, 16, 17, 18, 25, 26, 32, 33, 34, 41, 42, 48, 49, 50, 57, 58, 64])
def test_sizes(n, dtype):
    Xs = synth.skew_batch(n, 7, 5000 + n).astype(dtype)
    print(f"[batched] n={n} {np.dtype(dtype).name}", flush=True)
    got, ipiv, logabs, sign = run(Xs, dtype)
    for b in range(7):
        compare_factors(Xs[b], got[b], ipiv[b], dtype)
        rl, rs = oracle.pfaffian_packed(*oracle.ltlt(Xs[b].astype(np.float64)))
        assert int(sign[b]) == rs
        if n % 2 == 0:
            assert abs(logabs[b] - rl) <= (1e-9 if dtype == np.float64 else 1e-4) * max(1.0, abs(rl))


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("n", [12, 16, 20, 32, 44])
def test_ties_and_zero_columns(n, dtype):
    """4 x 4 blocks on the diagonal (every column ties at zero in most lanes) and
    matrices of +1 and -1, whose first steps tie everywhere."""
    ones = synth.skew_batch(n, 2, 5100 + n)
    Xs = np.stack([synth.skew_blockdiag4(n, 5200 + n), np.sign(ones[0]), np.sign(ones[1])]).astype(dtype)
    got, ipiv, logabs, sign = run(Xs, dtype)
    for b in range(3):
        info = compare_factors(Xs[b], got[b], ipiv[b], dtype)
        assert info["first_pivot_mismatch"] >= 3
