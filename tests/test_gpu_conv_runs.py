"""The runs-of-taps convolution kernel (strided, not padded, few channels) against
the oracle's direct loops: tap heights that are and are not multiples of four
(the last run of a column then overlaps the one before), two and four waves to a
tile, filter counts off the tile, one position and one filter block, accumulation
and unaligned outputs, and the shapes on either side of its rule (kh = 5, odd
filter counts, fewer than 16 runs, more than 2048).  Integer-valued tensors, where
every fp32 sum is exact in any order: bit-equal."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import synth
from oracle import conv as oc
from synth import conv as sc
from test_gpu_convgemm import dev, host, run

pytestmark = pytest.mark.gpu

# kn, k, ci, hi, wi, b, stride
CASES = [
    (64, 11, 3, 51, 47, 3, 4),      # first layer: 99 runs, four waves
    (64, 7, 3, 40, 41, 2, 2),       # 42 runs, two waves
    (68, 6, 3, 23, 20, 3, 2),       # two rows of tiles; last run overlaps by two
    (4, 4, 4, 4, 4, 1, 2),          # one position, 16 runs exactly
    (4, 4, 3, 18, 18, 2, 3),        # 12 runs: not taken
    (20, 5, 6, 19, 21, 2, 2),       # kh = 5: not taken
    (33, 7, 3, 30, 30, 2, 2),       # odd filter count: not taken
    (12, 8, 8, 31, 33, 2, 5),       # whole runs, 128 of them, stride past the run
    (8, 10, 6, 24, 27, 1, 3),       # 180 runs, last overlaps by two
    (8, 9, 7, 17, 20, 2, 2),        # 189 runs: a ragged group; overlaps by three
    (4, 32, 8, 40, 36, 1, 4),       # 2048 runs exactly
    (4, 33, 8, 41, 37, 1, 4),       # 2376 runs: not taken
    (36, 4, 4, 90, 88, 6, 2),       # many tiles, ragged positions
]


@pytest.mark.parametrize("case", CASES)
def test_runs_integer_exact(case):
    kn, k, ci, hi, wi, b, s = case
    F = sc.int_tensor((kn, k, k, ci), 83, -3, 3, index=9)
    I = sc.int_tensor((hi, wi, ci, b), 83, 0, 3, index=10)
    print(f"[conv] runs {case}", flush=True)
    got = host(run(F, I, s, 0))
    assert np.array_equal(got.astype(np.float64), oc.conv_direct(F, I, s, 0))


def test_runs_accumulate_misaligned():
    """O += conv into an output that is not 16-byte aligned, and from filters and
    an input that are not either (their loads are 16 bytes wide)."""
    import paper_2005_06410_amd as lt
    kn, k, ci, hi, wi, b, s = 36, 7, 3, 24, 25, 2, 2
    F = sc.int_tensor((kn, k, k, ci), 84, -3, 3, index=9)
    I = sc.int_tensor((hi, wi, ci, b), 84, 0, 3, index=10)
    ref = oc.conv_direct(F, I, s, 0)

    def shifted(t):
        flat = torch.zeros(t.size + 1, dtype=torch.float32, device="cuda")
        flat[1:] = torch.from_numpy(t.ravel(order="F").copy()).cuda()
        strides = [1]
        for d in t.shape[:-1]:
            strides.append(strides[-1] * d)
        return flat[1:].as_strided(t.shape, strides, 1)

    flat = torch.full((ref.size + 2,), 7.0, dtype=torch.float32, device="cuda")
    st = [1, kn, kn * ref.shape[1], kn * ref.shape[1] * ref.shape[2]]
    out = flat[1:1 + ref.size].as_strided(ref.shape, st, 1)
    lt.convgemm(shifted(F), shifted(I), stride=s, pad=0, out=out, accumulate=True)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy().astype(np.float64), ref + 7.0)
    assert float(flat[0]) == 7.0 and float(flat[-1]) == 7.0


@pytest.mark.parametrize("k", [6, 7, 9, 11])
def test_runs_infinities_stay_in_their_windows(k):
    """One infinite input value: exactly the outputs whose window holds it are not
    finite (rows that an overlapping run leaves out add none)."""
    kn, ci, hi, wi, b, s = 8, 4, 29, 27, 2, 3
    F = np.asfortranarray(np.abs(synth.rng_for(85).standard_normal((kn, k, k, ci))).astype(np.float32) + 0.1)
    I = sc.int_tensor((hi, wi, ci, b), 85, 1, 3, index=10)
    y, x = 13, 14
    I[y, x, ci - 1, 0] = np.inf
    got = host(run(F, I, s, 0))
    oh, ow = np.arange(got.shape[1])[:, None], np.arange(got.shape[2])[None, :]
    inside = (oh * s <= y) & (y < oh * s + k) & (ow * s <= x) & (x < ow * s + k)
    want = np.zeros(got.shape, bool)
    want[..., 0] = inside[None]
    assert np.array_equal(~np.isfinite(got), want) and not np.isnan(got).any()
