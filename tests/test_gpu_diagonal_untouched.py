"""The diagonal and the upper triangle are neither read nor written: NaN there
stays and does not spread, and a buffer that ends with the last entry of the
strict lower triangle, A(n-1, n-2), is enough.  With a large leading dimension
the last diagonal entry would lie beyond that buffer; the matrices are graded
towards the last row, so that it is a pivot at once (in one workgroup's panel and
in several)."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import synth
from gpu_util import compare_factors

pytestmark = pytest.mark.gpu


def lt():
    import paper_2005_06410_amd as m
    return m


def last_row_heavy(n, seed):
    X = synth.skew_gauss(n, seed)
    X[-1, :] *= 1e3
    X[:, -1] *= 1e3
    return X


@pytest.mark.parametrize("n,lda,dtype", [(70, 300000, np.float64), (300, 3000, np.float64), (700, 1500, np.float64),
                                         (70, 600000, np.float32), (700, 1500, np.float32)])
def test_buffer_of_the_strict_lower_triangle(n, lda, dtype):
    X = last_row_heavy(n, 7000 + n).astype(dtype)
    tdt = torch.float64 if dtype == np.float64 else torch.float32
    buf = torch.full(((n - 2) * lda + n,), float("nan"), dtype=tdt, device="cuda")
    cols = torch.from_numpy(np.ascontiguousarray(X.T)).cuda()      # row c: column c of X
    for c in range(n - 1):
        buf[c * lda + c + 1:c * lda + n] = cols[c, c + 1:]
    lower = torch.zeros_like(buf, dtype=torch.bool)
    for c in range(n - 1):
        lower[c * lda + c + 1:c * lda + n] = True
    ipiv = torch.empty(n, dtype=torch.int32, device="cuda")
    print(f"[diagonal] n={n} lda={lda} {np.dtype(dtype).name}", flush=True)
    lib = lt().load()
    code = lib.ltlt_factor(n, buf.data_ptr(), lda, 0 if dtype == np.float64 else 1, ipiv.data_ptr(),
                           torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert code == 0
    lt().device_status()
    assert bool(torch.isnan(buf[~lower]).all())
    packed = np.zeros((n, n), dtype=dtype)
    for c in range(n - 1):
        packed[c + 1:, c] = buf[c * lda + c + 1:c * lda + n].cpu().numpy()
    compare_factors(X, packed, ipiv.cpu().numpy(), dtype)
