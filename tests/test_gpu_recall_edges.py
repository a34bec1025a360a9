"""Recall counts where the logits' tiles (16 rows, 16 keys a wave) and the digits of the ranking begin and end: few rows and keys,
rows in any order, logits that are equal."""
import numpy as np
import pytest
import torch

import oracle
import paper_2510_24606_amd as dhsa

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,n_rows,D,dtype,values", [
    (1, 1, 128, "bf16", "normal"), (15, 16, 64, "f32", "normal"), (16, 15, 128, "bf16", "few"), (17, 17, 64, "bf16", "normal"),
    (63, 33, 128, "f32", "few"), (65, 1, 64, "bf16", "few"), (700, 31, 128, "bf16", "wide"), (700, 64, 64, "f32", "wide"),
    (5000, 20, 128, "bf16", "equal"), (9000, 18, 128, "bf16", "normal"), (9000, 18, 64, "f32", "few")])
@pytest.mark.parametrize("B_r", [0, 48])
def test_recall_at_the_edges(L, n_rows, D, dtype, values, B_r):
    rng = np.random.default_rng(L + n_rows)
    B = np.unique(np.r_[0, np.arange(7, L, 7), np.arange(50, L, 50), L]).astype(np.int32)
    draw = {"normal": lambda s: rng.standard_normal(s), "few": lambda s: rng.integers(-1, 2, s), "equal": lambda s: np.ones(s),
            "wide": lambda s: rng.standard_normal(s) * 2.0 ** rng.integers(-20, 20, s)}[values]
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    Q, K = (torch.from_numpy(draw((H, L, D)).astype(np.float32)).to(t) for H in (2, 1))
    rows = rng.integers(0, L, n_rows).astype(np.int64)
    rows[0] = L - 1
    N_b = max(1, L // 9)
    q, k = Q.cuda(), K.cuda()
    prob = dhsa.problem(q, k, B, N_b, B_r=B_r)
    plan, ws = dhsa.alloc(prob, B)
    dhsa.dhsa_route(prob, q, k, B, plan, ws)
    hits, size = dhsa.dhsa_recall_rows(prob, q, k, B, plan, 1, rows)
    # the rows' own lists (equal values make chunk scores that are equal but for their rounding: another ranking would be as good)
    idx, cnt = (x.cpu().numpy() for x in dhsa.dhsa_plan_expand_rows(prob, plan, 1, rows))
    for r, i in enumerate(rows):
        listed = idx[r, :cnt[r]]
        want = oracle.recall_row(Q[1, i].float().numpy(), K[0].float().numpy(), int(i), listed[listed <= i], min(N_b, int(i) + 1))
        assert (int(hits[r]), int(size[r])) == want, (r, i)
