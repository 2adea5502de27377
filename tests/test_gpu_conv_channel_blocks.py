"""The channel-block convolution kernels against the oracle's direct loops, at
sizes that reach each of their tiles (64 x 32 with four and eight waves, 64 x 16
with four and eight, 32 x 32, 32 x 64, 16 x 16, and the short-contraction
64 x 128), with filter counts that do and do not allow wide loads, partial
channel blocks, padding and strides; the tile that the library takes for each
case is asserted (on 256 CUs; filters loaded one by one never get the 64 x 32 tile
nor 64 x 16 with four waves).  Integer-valued tensors, where every fp32 sum is
exact in any order: bit-equal.  Infinities outside a tap's window must not
reach the sum (a padded or clamped load times zero would give NaN)."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import synth
from oracle import conv as oc
from synth import conv as sc
from test_gpu_convgemm import dev, host, run

pytestmark = pytest.mark.gpu

# (kn, k, ci, hi, wi, b, stride, pad), (filters, positions, waves) of the tile
CASES = [
    ((40, 1, 16, 29, 18, 8, 1, 0), (64, 32, 4)),        # one group
    ((36, 3, 11, 72, 15, 4, 1, 1), (64, 32, 4)),        # smallest partial block (11 of 16)
    ((128, 3, 16, 61, 59, 4, 1, 1), (64, 32, 4)),
    ((64, 3, 128, 40, 40, 3, 1, 1), (64, 32, 8)),       # at least 64 groups, few tiles
    ((44, 5, 33, 23, 76, 3, 1, 0), (64, 32, 8)),        # partial block, no padding
    ((296, 1, 16, 62, 8, 7, 1, 0), (64, 16, 4)),
    ((36, 1, 11, 19, 45, 10, 1, 0), (64, 16, 4)),       # partial block
    ((236, 5, 64, 52, 60, 8, 2, 2), (64, 16, 4)),       # strided and padded
    ((92, 5, 16, 64, 52, 2, 2, 0), (64, 16, 8)),
    ((176, 7, 33, 44, 15, 2, 1, 3), (64, 16, 8)),       # partial block, padded
    ((191, 2, 32, 21, 30, 9, 2, 0), (64, 16, 8)),       # odd filter count: scalar filter loads
    ((166, 3, 16, 16, 17, 5, 1, 1), (64, 16, 8)),       # filters a multiple of 2 only, padded
    ((178, 3, 64, 44, 13, 42, 1, 0), (32, 32, 8)),
    ((66, 3, 40, 19, 23, 5, 1, 1), (32, 32, 8)),        # partial block, padded
    ((17, 1, 12, 76, 27, 2, 1, 0), (32, 32, 8)),        # odd filter count
    ((17, 2, 32, 15, 43, 6, 1, 1), (32, 32, 8)),
    ((22, 5, 16, 48, 43, 15, 1, 2), (32, 64, 8)),
    ((17, 3, 48, 41, 40, 6, 1, 1), (32, 64, 8)),        # odd filter count
    ((17, 1, 11, 40, 32, 7, 1, 0), (32, 64, 8)),
    ((18, 1, 16, 29, 38, 8, 1, 0), (32, 64, 8)),
    ((33, 3, 64, 20, 21, 3, 2, 1), (16, 16, 16)),
    ((30, 2, 33, 23, 19, 2, 1, 0), (16, 16, 16)),       # partial block
    ((128, 3, 16, 30, 29, 2, 2, 1), (16, 16, 16)),      # nine groups for sixteen waves
    ((256, 3, 80, 13, 13, 1, 1, 0), (16, 16, 16)),      # single image
    ((5, 5, 11, 12, 9, 1, 3, 2), (16, 16, 16)),         # one row of tiles
    ((64, 1, 16, 260, 260, 2, 1, 0), (64, 128, 1)),     # one group
    ((196, 2, 16, 82, 76, 9, 1, 1), (64, 128, 1)),      # padded, ragged filters
    ((141, 2, 32, 61, 92, 9, 1, 1), (64, 128, 1)),      # odd filter count, eight groups
]


@pytest.mark.parametrize("case,tile", CASES)
def test_channel_blocks_integer_exact(case, tile):
    import paper_2005_06410_amd as lt
    kn, k, ci, hi, wi, b, s, p = case
    assert lt.conv_choice(kn, k, k, ci, hi, wi, b, s, p) == (3, *tile)
    F = sc.int_tensor((kn, k, k, ci), 80, -3, 3, index=9)
    I = sc.int_tensor((hi, wi, ci, b), 80, 0, 3, index=10)
    print(f"[conv] channel blocks {case}", flush=True)
    got = host(run(F, I, s, p))
    assert np.array_equal(got.astype(np.float64), oc.conv_direct(F, I, s, p))


@pytest.mark.parametrize("case", [(64, 1, 32, 130, 130, 3, 1, 0), (68, 1, 128, 190, 180, 2, 1, 0),
                                  (263, 1, 128, 54, 12, 54, 1, 0), (33, 3, 16, 112, 112, 10, 1, 1)])
def test_neighbours_on_the_general_kernels_integer_exact(case):
    """Layers that the channel blocks would slow down: same results, other kernel."""
    import paper_2005_06410_amd as lt
    kn, k, ci, hi, wi, b, s, p = case
    assert lt.conv_choice(kn, k, k, ci, hi, wi, b, s, p)[0] == (1 if p else 2)
    F = sc.int_tensor((kn, k, k, ci), 80, -3, 3, index=9)
    I = sc.int_tensor((hi, wi, ci, b), 80, 0, 3, index=10)
    print(f"[conv] beside channel blocks {case}", flush=True)
    got = host(run(F, I, s, p))
    assert np.array_equal(got.astype(np.float64), oc.conv_direct(F, I, s, p))


def test_channel_blocks_accumulate_misaligned():
    """O += conv into an output that is not 16-byte aligned (scalar stores)."""
    import paper_2005_06410_amd as lt
    kn, k, ci, hi, wi, b = 36, 3, 32, 14, 15, 2
    F = sc.int_tensor((kn, k, k, ci), 81, -3, 3, index=9)
    I = sc.int_tensor((hi, wi, ci, b), 81, 0, 3, index=10)
    ref = oc.conv_direct(F, I, 1, 1)
    n = kn * hi * wi * b
    flat = torch.full((n + 2,), 7.0, dtype=torch.float32, device="cuda")
    out = flat[1:1 + n].as_strided((kn, hi, wi, b), (1, kn, kn * hi, kn * hi * wi), 1)
    lt.convgemm(dev(F), dev(I), stride=1, pad=1, out=out, accumulate=True)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy().astype(np.float64), ref + 7.0)
    assert float(flat[0]) == 7.0 and float(flat[n + 1]) == 7.0


@pytest.mark.parametrize("ci", [32, 24])
def test_infinities_stay_in_their_windows(ci):
    """One infinite input value: exactly the outputs whose window holds it are
    not finite (padding, clamped positions and partial channel blocks add none)."""
    kn, k, hi, wi, b = 20, 3, 12, 11, 2
    F = np.asfortranarray(np.abs(synth.rng_for(82).standard_normal((kn, k, k, ci))).astype(np.float32) + 0.1)
    I = sc.int_tensor((hi, wi, ci, b), 82, 1, 3, index=10)
    I[hi - 1, wi - 1, ci - 1, 0] = np.inf
    got = host(run(F, I, 1, 1))
    want = np.zeros(got.shape, bool)
    want[:, hi - 2:, wi - 2:, 0] = True
    assert np.array_equal(~np.isfinite(got), want) and not np.isnan(got).any()
