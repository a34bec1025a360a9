"""Which workgroup takes which head and row tile: every tile of every head has one, whatever the numbers of both."""
import numpy as np
import pytest
import torch

import paper_2510_24606_amd as dhsa

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H_kv,G", [(1, 1), (1, 7), (2, 3), (3, 1), (4, 7), (5, 2), (6, 1), (8, 1), (12, 3)])
@pytest.mark.parametrize("lens", [(100,), (20, 50, 90, 128, 3), (128, 128, 33)])
def test_every_tile_of_every_head_is_taken(H_kv, G, lens):
    B = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    L, D = int(B[-1]), 128
    gen = torch.Generator(device="cuda").manual_seed(H_kv * 16 + G)
    q, k, v = (torch.randn((H, L, D), dtype=torch.bfloat16, device="cuda", generator=gen) for H in (H_kv * G, H_kv, H_kv))

    def attend(q, k, v):
        O = torch.full_like(q, float("nan"))
        prob = dhsa.problem(q, k, B, 64)
        plan, ws = dhsa.alloc(prob, B)
        dhsa.dhsa_prefill(prob, q, k, v, B, O, plan, ws)
        return O

    every = attend(q, k, v)
    assert bool(torch.isfinite(every).all())
    for h in range(H_kv * G):       # one head at a time: the order of tiles alone
        assert torch.equal(every[h:h + 1], attend(q[h:h + 1], k[h // G:h // G + 1], v[h // G:h // G + 1])), h
