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


@pytest.mark.parametrize("L,D,dtype,n_rows,integers", [(300, 64, "f32", 1, False), (5000, 128, "bf16", 17, True),
                                                       (9000, 64, "bf16", 8, True), (9000, 128, "f32", 9, False),
                                                       (4097, 128, "f32", 513, False)])
def test_recall_row_groups_ties_and_candidate_list(L, D, dtype, n_rows, integers):
    """Row groups of 8, 512 rows per launch, key blocks of 512, regions above and below the 4096 keys the select
    finishes in LDS; small integers tie by the thousand, so the threshold falls into a tie."""
    w = dhsa_inputs.make("c1" if dtype == "f32" else "c3", L=L, H_q=2, H_kv=1, D=D, N_b=max(64, L // 8))
    Qh, Kh = w.Q, w.K
    if integers:
        Qh, Kh = (torch.sign(x.float()).mul(torch.arange(x.shape[2]) < 3).to(x.dtype) for x in (Qh, Kh))
    Q, K = Qh.cuda(), Kh.cuda()
    prob = dhsa.problem(Q, K, w.B, w.N_b)
    plan, ws = dhsa.alloc(prob, w.B)
    dhsa.dhsa_route(prob, Q, K, w.B, plan, ws)
    rows = np.unique(np.linspace(0, L - 1, n_rows).astype(np.int64))
    hits, size = dhsa.dhsa_recall_rows(prob, Q, K, w.B, plan, 1, rows)
    h_ref, s_ref = oracle.recall_rows(Qh.float().numpy(), Kh.float().numpy(), w.B, w.N_b, 1, rows)
    np.testing.assert_array_equal(hits.cpu().numpy(), h_ref)
    np.testing.assert_array_equal(size.cpu().numpy(), s_ref)
