"""The solve at the borders of its blocks (64 rows), of its instances (one, two
and up to four right-hand sides, passes of four) and of the tridiagonal scan (one
step per thread, fewer steps than threads), against the oracle on the same
factors; leading dimensions of A and B larger than n.  Bars as in the solve
tests (1e-9 in fp64, 1e-3 in fp32, backward error 10)."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import device_colmajor
from test_gpu_solve import check, gpu_factor_solve, lt

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nrhs", [(62, 1), (64, 2), (66, 3), (126, 4), (128, 5), (130, 6), (192, 7), (194, 9),
                                    (320, 1), (324, 2), (2046, 1), (2050, 3), (2052, 1)])
def test_block_borders(n, nrhs):
    X = synth.skew_gauss(n, 6000 + n)
    B = synth.rng_for(6001 + n).standard_normal((n, nrhs))
    print(f"[solve] n={n} nrhs={nrhs}", flush=True)
    packed, ipiv, x = gpu_factor_solve(X, B)
    check(X, B, x, packed, ipiv, 1e-9)


@pytest.mark.parametrize("n,nrhs", [(130, 1), (322, 2), (194, 4)])
def test_block_borders_fp32(n, nrhs):
    X = synth.skew_gauss(n, 6100 + n)
    B = synth.rng_for(6101 + n).standard_normal((n, nrhs)).astype(np.float32)
    packed, ipiv, x = gpu_factor_solve(X.astype(np.float32), B, dtype=np.float32)
    check(X.astype(np.float32), B, x, packed, ipiv, 1e-3)


def test_leading_dimensions():
    n, lda, ldb, nrhs = 190, 203, 197, 3
    X = synth.skew_gauss(n, 6200)
    B = synth.rng_for(6201).standard_normal((n, nrhs))
    flat, A = device_colmajor(X, lda=lda, fill=np.nan)
    ipiv = lt().factor(A)
    buf = torch.full((nrhs * ldb,), np.nan, dtype=torch.float64, device="cuda")
    Bd = buf.as_strided((n, nrhs), (1, ldb))
    Bd.copy_(torch.from_numpy(B))
    lt().solve(A, ipiv, Bd)
    torch.cuda.synchronize()
    lt().device_status()
    packed = np.tril(A.cpu().numpy(), -1)
    check(X, B, Bd.cpu().numpy(), packed, ipiv.cpu().numpy(), 1e-9)
    pad = buf.reshape(nrhs, ldb)[:, n:]
    assert bool(torch.isnan(pad).all())
