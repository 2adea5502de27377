"""How many passes the solve makes over its right-hand sides: up to eight take
one (two groups of four side by side), counted as the kernels of a captured call,
and each column's result does not depend on the others beside it."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import device_colmajor
from test_gpu_solve import check, lt

pytestmark = pytest.mark.gpu


def factored(n, dtype, seed):
    X = synth.skew_gauss(n, seed).astype(dtype)
    flat, A = device_colmajor(X, dtype=dtype)
    return X, A, lt().factor(A)


def captured_kernels(call):
    """Kernels that one call enqueues (it is captured, not run)."""
    hip = lt().load()                                    # its dependencies hold the runtime's functions
    s = torch.cuda.Stream()
    graph = ctypes.c_void_p()
    nodes = ctypes.c_size_t(0)
    with torch.cuda.stream(s):
        assert hip.hipStreamBeginCapture(ctypes.c_void_p(s.cuda_stream), 2) == 0     # relaxed
        call()
        assert hip.hipStreamEndCapture(ctypes.c_void_p(s.cuda_stream), ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(nodes)) == 0
    assert hip.hipGraphDestroy(graph) == 0
    return nodes.value


def test_eight_right_hand_sides_take_one_pass():
    n = 130
    _, A, ipiv = factored(n, np.float64, 6300)
    B = torch.ones((16, n), dtype=torch.float64, device="cuda")
    for nrhs in (1, 16):                                 # workspace and kernel attributes in place
        lt().solve(A, ipiv, B[:nrhs].clone().t())
    torch.cuda.synchronize()
    count = {}
    for nrhs in (1, 4, 5, 8, 9, 16):
        x = B[:nrhs].clone().t()
        torch.cuda.synchronize()
        count[nrhs] = captured_kernels(lambda: lt().solve(A, ipiv, x))
    print(f"[solve] kernels by right-hand sides {count}", flush=True)
    assert count[1] == count[4] == count[5] == count[8]
    assert count[9] == count[16] and count[16] - count[8] < count[8]


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("n,nrhs", [(2, 8), (64, 5), (130, 7), (194, 8), (322, 13), (2050, 6)])
def test_columns_do_not_depend_on_each_other(n, nrhs, dtype):
    X, A, ipiv = factored(n, dtype, 6400 + n)
    B = synth.rng_for(6401 + n).standard_normal((n, nrhs)).astype(dtype)
    print(f"[solve] n={n} nrhs={nrhs} {np.dtype(dtype).name}", flush=True)
    Bd = torch.from_numpy(np.ascontiguousarray(B.T)).cuda()
    x = Bd.clone().t()
    lt().solve(A, ipiv, x)
    for q in range(0, nrhs, 4):                          # groups of four: the same instance
        m = min(4, nrhs - q)
        if m > 2:
            y = Bd[q:q + m].clone().t()
            lt().solve(A, ipiv, y)
            assert torch.equal(y, x[:, q:q + m])
    torch.cuda.synchronize()
    lt().device_status()
    packed = np.tril(A.cpu().numpy(), -1)
    check(X, B, x.cpu().numpy(), packed, ipiv.cpu().numpy(), 1e-9 if dtype == np.float64 else 1e-3)
