"""Sizes at which the kernels change their path or run out of a tile: edges of segments, tiles, digit widths and
candidate lists, against the CPU oracle."""
import numpy as np
import pytest
import torch

import dhsa_inputs
import oracle
import paper_2510_24606_amd as dhsa

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,W,levels", [(511, 3, 0), (512, 8, 0), (513, 8, 4), (1024, 31, 0), (1025, 32, 0),
                                        (5000, 33, 3), (4096, 512, 0), (4097, 600, 5), (131073, 8, 0), (140001, 40, 9)])
def test_boundary_windows_and_slabs(L, W, levels):
    """Windows of 512 positions, halos of 128 .. 512 (W of 512 and more decide nothing locally), compaction slabs of
    131072; `levels` distinct scores make runs of equal ones, which a window cannot always decide."""
    rng = np.random.default_rng(L + W)
    p = rng.random(L).astype(np.float32)
    if levels:
        p = (np.ceil(p * levels) / levels).astype(np.float32)
        p[L // 3:L // 2] = p[L // 3]              # one run across many windows
    for tau in (0.0, 0.7):
        got = dhsa.dhsa_finalize_boundaries(torch.from_numpy(p).cuda(), tau, W)
        np.testing.assert_array_equal(got, oracle.finalize_boundaries(p, tau, W))
