"""Both forms of the registration's window products by the rule that chooses
between them: folded ones in calls large enough for them (or where they need no
further pass over the pairs), plain ones in small calls, whose windows above 320
samples keep their maxima over the spectra.  Peaks equal the oracle's."""
import math

import numpy as np
import pytest
import torch

import oracle

from gpu_util import need_gpu
from test_gpu_register import gpu_register, pairs_shifted

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


def check(N, up, B, distinct, norm):
    """B pairs, `distinct` of them over and over."""
    rng = np.random.default_rng(1000 * N + up + B)
    d = min(B, distinct)
    ref, mov, _ = pairs_shifted(rng, d, N, max_shift=N / 6.0)
    reps = (B + d - 1) // d
    sh, pk = gpu_register(np.tile(ref, (reps, 1, 1))[:B], np.tile(mov, (reps, 1, 1))[:B], up, norm)
    for b in range(B):
        assert list(pk[b]) == list(pk[b % d]) and np.array_equal(sh[b], sh[b % d]), b
    for b in range(d):
        so, po = oracle.register64(ref[b].astype(np.complex128), mov[b].astype(np.complex128), up, norm)
        assert list(pk[b]) == list(po), (norm, b, pk[b], po)
        assert np.allclose(sh[b], so, atol=1e-5)


# the smallest folded window (32 samples), windows around whole tiles of 16 + 16
# samples, even and odd, with and without a full second column tile
@pytest.mark.parametrize("N", [32, 64, 128, 192, 256])
@pytest.mark.parametrize("up", [21, 22, 43, 63, 64, 85, 213])
def test_large_calls_take_folded_products(N, up):
    U = math.ceil(1.5 * up)
    B = math.ceil(3.6e8 / (U * N * (N + U)))
    check(N, up, B, 4, up % 2)


@pytest.mark.parametrize("N,up,B", [(32, 22, 10), (64, 100, 3), (64, 37, 67), (128, 100, 30), (256, 100, 3),
                                    (192, 150, 2),                                          # plain
                                    (32, 214, 3), (32, 333, 10), (64, 214, 10), (32, 700, 2), (128, 214, 2),  # ... wide
                                    (128, 75, 1), (256, 100, 1), (64, 333, 3), (32, 1000, 1), (32, 1000, 2)])
def test_small_calls(N, up, B):
    for norm in (0, 1):
        check(N, up, B, 4, norm)
