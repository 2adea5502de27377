"""The trailing update at the borders of its two kernels (64 x 64 tiles up to
order 1984, 128 x 128 beyond) and of their tiles and steps, against the same
product in fp64: C(i, c) = S(perm i, perm c) + sum_u Lx(i, u) Bt(c, u) below the
diagonal, sources before the block, everything else untouched.  Operands with
odd leading dimensions take the 128 x 128 kernel's register-staged loads; rows
and columns held before the block fall into tiles inside the block, on its
diagonal and at its edge.  Bar:
gamma_{K+1} (|S| + |Lx| |Bt|^T) entrywise (any order of the sums)."""
from __future__ import annotations

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("m,K,odd", [(2, 1, 0), (63, 4, 1), (64, 5, 0), (65, 31, 0), (129, 33, 1), (200, 129, 0),
                                     (700, 130, 1), (1984, 36, 0), (1985, 36, 0), (1985, 37, 1), (2111, 129, 0), (2304, 20, 0),
                                     # one round of 128 x 128 tiles and two; either side of 32 columns
                                     (4864, 33, 0), (4866, 32, 0), (4866, 33, 0), (5000, 129, 0)])
def test_update_sizes(m, K, odd, dtype):
    import paper_2005_06410_amd as lt
    g = torch.Generator(device="cuda")
    g.manual_seed(m + K)
    off = 40
    n = m + off
    ldc, ld = n + 3, m + (m + odd) % 2
    print(f"[update] m={m} K={K} ld={ld} {dtype}", flush=True)
    buf = torch.randn((n, ldc), generator=g, device="cuda", dtype=dtype)
    C = buf.t()[:n]                                          # column-major, ldc > n
    L = torch.randn((K, ld), generator=g, device="cuda", dtype=dtype).t()[:m]
    B = torch.randn((K, ld), generator=g, device="cuda", dtype=dtype).t()[:m]
    perm = torch.arange(m, dtype=torch.int32)
    for z in range(min(off, m // 3)):
        perm[(z * 37 + 1) % m] = -1 - z                      # rows held before the block
    old = buf.clone()
    lt.skew_update(C, L, B, perm.cuda(), offset=off)
    torch.cuda.synchronize()
    low = torch.tril(old.t()[:n].double(), -1)
    S = low - low.t()
    src = (perm.long() + off).cuda()
    Sp = S[src][:, src]
    ref = Sp + L.double() @ B.double().t().contiguous()
    u = 2.0 ** (-53 if dtype == torch.float64 else -24)
    gam = (K + 1) * u / (1 - (K + 1) * u)
    bound = gam * (Sp.abs() + L.double().abs() @ B.double().abs().t().contiguous()) + (1e-30 if u < 1e-10 else 0)
    # the fp64 reference's own sums carry the same kind of error
    bound = bound * (2 if dtype == torch.float64 else 1.001)
    got = C[off:, off:].double()
    strict = torch.tril(torch.ones(m, m, dtype=torch.bool, device="cuda"), -1)
    assert bool((((got - ref).abs() <= bound) | ~strict).all())
    mask = torch.ones_like(buf, dtype=torch.bool)            # (column, row)
    mask[off:n, off:n] = ~strict.t()
    assert torch.equal(buf[mask], old[mask])
