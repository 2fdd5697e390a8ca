"""GPU parity at the sizes where a choice of kernel, tile or hand-over changes: the edges that the general parity
tests do not visit.  Oracle, bar and helpers as there (lists and counts bit-exact, y within max-abs 1e-2, rel-L2 2e-3)."""
import numpy as np
import pytest
import torch

import workloads as wl
from workloads import BF16, F16, I8

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from gpu_util import Layer, check_against_oracle


def _layer(K, N, wdt, seed, B=16):
    if wdt == I8:
        q, sc = wl.quantize_i8(K, N, seed)
        return Layer(q, I8, col_scale_bits=sc, B=B), BF16
    return Layer(wl.weights(K, N, seed, wdt), wdt, B=B), wdt


# tokens' lists are dealt out over the column tiles: one tile, fewer tiles than tokens, as many as lists, more
@pytest.mark.parametrize("lanes", [0, 64, 16, 1])
@pytest.mark.parametrize("K,N", [(40, 128), (1000, 128), (1000, 256), (2000, 384), (1100, 2048), (1100, 2176), (600, 2312)])
def test_lists_of_a_batch_whatever_the_number_of_tiles(K, N, lanes):
    layer, xdt = _layer(K, N, BF16, 900 + N)
    for B in (2, 5, 16):
        X = wl.laplace(B, K, 901 + K, xdt, loc=0.1, scale=0.5)
        for tau in (0.3, 1.2):
            print(f"lists K={K} N={N} B={B} lanes={lanes} tau={tau}", flush=True)
            check_against_oracle(layer, X, xdt, 0.1, tau, None, cfg=(0, 0, 0, lanes) if lanes else None, what=f"{K} {N} {B} {lanes}")
