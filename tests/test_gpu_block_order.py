"""Which workgroup takes which head and row tile: every tile of every head has one, whatever the numbers of both."""
import numpy as np
import pytest
import torch

import paper_2510_24606_amd as dhsa

pytestmark = pytest.mark.gpu


def attend(q, k, v, B, N_b, B_r=0):
    """The output of routing and attention in launches of their own, and the kernels that take the height classes."""
    O = torch.full_like(q, float("nan"))
    prob = dhsa._with_vo(dhsa.problem(q, k, B, N_b, B_r=B_r), v, O)
    plan, ws = dhsa.alloc(prob, B)
    dhsa.dhsa_route(prob, q, k, B, plan, ws)
    dhsa.dhsa_sparse_prefill(prob, q, k, v, B, plan, O)
    return O, dhsa.dhsa_attention_kernels(prob, B)[0]


def tensors(H_kv, G, L, D):
    gen = torch.Generator(device="cuda").manual_seed(H_kv * 16 + G)
    return [torch.randn((H, L, D), dtype=torch.bfloat16, device="cuda", generator=gen) for H in (H_kv * G, H_kv, H_kv)]


@pytest.mark.parametrize("H_kv,G", [(1, 1), (1, 7), (2, 3), (3, 1), (4, 7), (5, 2), (6, 1), (8, 1), (12, 3)])
@pytest.mark.parametrize("lens", [(100,), (20, 50, 90, 128, 3), (128, 128, 33)])
def test_every_tile_of_every_head_is_taken(H_kv, G, lens):
    """Few tiles: by dhsa_prefill all in one launch, by dhsa_sparse_prefill in those of the four-wave kernels."""
    B = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    q, k, v = tensors(H_kv, G, int(B[-1]), 128)

    def joined(q, k, v):
        O = torch.full_like(q, float("nan"))
        prob = dhsa.problem(q, k, B, 64)
        plan, ws = dhsa.alloc(prob, B)
        dhsa.dhsa_prefill(prob, q, k, v, B, O, plan, ws)
        return O

    every, (apart, kernels) = joined(q, k, v), attend(q, k, v, B, 64)
    assert 1 not in kernels
    assert bool(torch.isfinite(every).all()) and torch.equal(every, apart)
    for h in range(H_kv * G):       # one head at a time: the order of tiles alone
        one = joined(q[h:h + 1], k[h // G:h // G + 1], v[h // G:h // G + 1])
        assert torch.equal(every[h:h + 1], one), h


@pytest.mark.parametrize("H_kv,G", [(1, 5), (2, 3), (3, 5), (4, 7), (5, 2), (6, 1), (7, 1), (12, 3), (20, 1)])
@pytest.mark.parametrize("D,step,n", [(64, 24, 181), (128, 13, 299), (64, 33, 301), (128, 140, 51)])
def test_many_rounds_of_the_four_wave_kernels(H_kv, G, D, step, n):
    """Odd numbers of tiles a head, by sequences on both sides of 4096 tokens and launches on both sides of 1536 workgroups, where
    all heads go side by side or some wait for others."""
    B = np.arange(0, n * step + 1, step, dtype=np.int32)
    q, k, v = tensors(H_kv, G, int(B[-1]), D)
    every, kernels = attend(q, k, v, B, 150)
    assert 1 not in kernels and bool(torch.isfinite(every).all())
    for g in range(H_kv):
        few, _ = attend(q[G * g:G * (g + 1)], k[g:g + 1], v[g:g + 1], B, 150)
        assert torch.equal(every[G * g:G * (g + 1)], few), g


@pytest.mark.parametrize("cls,B_r,step,n,N_b", [(0, 128, 50, 612, 1536), (1, 0, 80, 207, 1301), (2, 64, 40, 495, 1024)])
@pytest.mark.parametrize("H_kv,G", [(5, 3), (3, 5), (1, 15)])
def test_many_rounds_of_the_lone_wave_kernels(cls, B_r, step, n, N_b, H_kv, G):
    """Odd numbers of tiles a head; the same rows of a kv-head alone are too few for these kernels and have the same bits."""
    B = np.arange(0, n * step + 1, step, dtype=np.int32)
    L = int(B[-1]) // (B_r or 1) * (B_r or 1)
    B = np.r_[B[B < L], L].astype(np.int32)
    q, k, v = tensors(H_kv, G, L, 128)
    every, kernels = attend(q, k, v, B, N_b, B_r)
    assert kernels[cls] == 1 and (L // B_r if B_r else n) % 2 == 1 and bool(torch.isfinite(every).all())
    for h in range(0, H_kv * G, G if G < 15 else 4):
        one, kernels = attend(q[h:h + 1], k[h // G:h // G + 1], v[h // G:h // G + 1], B, N_b, B_r)
        assert 1 not in kernels and torch.equal(every[h:h + 1], one), h
