"""Sizes at which the kernels change their path or run out of a tile: edges of segments, tiles, digit widths and
candidate lists, against the CPU oracle."""
import os
import re

import numpy as np
import pytest
import torch

import dhsa_inputs
import oracle
import paper_2510_24606_amd as dhsa

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,W,levels", [(511, 3, 0), (512, 8, 0), (513, 8, 4), (1024, 31, 0), (1025, 32, 0),
                                        (5000, 33, 3), (4096, 512, 0), (4097, 600, 5), (131073, 8, 0), (140001, 40, 9),
                                        (20000, 300, 2), (20001, 511, 40), (6000, 2000, 0), (1400, 900, 50)])
def test_boundary_windows_and_slabs(L, W, levels):
    """Windows of 512 positions, halos of 128 .. 512 (W of 512 and more decide nothing locally), compaction slabs of
    131072; `levels` distinct scores make runs of equal ones, which a window cannot always decide, next to kept positions
    of the segment beside it."""
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
                                                       (20000, 64, "bf16", 5, True), (700, 64, "f32", 9, True),
                                                       (4097, 128, "f32", 513, False)])
def test_recall_row_groups_ties_and_candidate_list(L, D, dtype, n_rows, integers):
    """512 rows per launch, regions above and below the 4096 keys the select finishes in LDS; small integers tie by the
    thousand, so the threshold falls into a tie.  (The edges of the 16 rows and 64 keys of a workgroup of the logits are
    test_gpu_recall_edges.py's.)"""
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


@pytest.mark.parametrize("L,H_q,D,N_b,lens,B_r", [(700, 2, 64, 90, ("uniform", 1, 20), 0),          # 16-row pieces
                                                  (1500, 1, 128, 1400, ("uniform", 100, 300), 0),   # > 1024 listed keys
                                                  (4100, 8, 64, 500, ("uniform", 90, 160), 0),      # 32-row pieces
                                                  (4100, 8, 128, 300, ("fixed", 1), 0),             # > 256 plan entries
                                                  (4100, 8, 128, 1100, ("uniform", 16, 64), 97),
                                                  (900, 2, 64, 3, ("uniform", 16, 64), 128),        # rows without a key
                                                  (901, 2, 64, 90, ("uniform", 16, 64), 1),         # a wave per row
                                                  (1100, 3, 128, 700, ("uniform", 100, 300), 1),
                                                  (901, 2, 128, 100, ("uniform", 16, 64), 2),
                                                  (901, 2, 128, 101, ("uniform", 16, 64), 2),       # ... and no more
                                                  (903, 2, 64, 25, ("uniform", 1, 9), 4),
                                                  (903, 2, 64, 26, ("uniform", 1, 9), 4),
                                                  (903, 2, 64, 1, ("uniform", 16, 64), 20)])
def test_f32_pieces_lists_and_batches(L, H_q, D, N_b, lens, B_r):
    w = dhsa_inputs.make("c1", L=L, H_q=H_q, H_kv=1, D=D, N_b=N_b, lens=lens)
    Q, K, V = (t.cuda() for t in (w.Q, w.K, w.V))
    O = torch.full_like(Q, float("nan"))
    prob = dhsa.problem(Q, K, w.B, w.N_b, B_r=B_r)
    plan, ws = dhsa.alloc(prob, w.B)
    dhsa.dhsa_prefill(prob, Q, K, V, w.B, O, plan, ws)
    rows = np.arange(0, L, 1 if L < 2000 else 5, dtype=np.int64)
    f32 = [w.f32(x) for x in "QKV"]
    if B_r:
        ref = oracle.prefill_rows_blocks(*f32, w.B, B_r, w.N_b, rows)[0]
    else:
        ref = oracle.prefill_rows(*f32, w.B, w.N_b, rows)[0]
    assert torch.isfinite(O).all()
    err = np.abs(O[:, torch.from_numpy(rows).cuda()].cpu().numpy().astype(np.float64) - ref).max()
    assert err <= 1e-5, err


@pytest.mark.parametrize("B_r", [0, 96])
@pytest.mark.parametrize("L,lens,N_b,keys", [(6100, ("fixed", 2), 300, "iid"),              # > 2048 chunks
                                             (2300, ("fixed", 1), 1500, "iid"),             # > 1024 listed chunks
                                             (3001, ("fixed", 4), 400, "equal"),            # all scores of a group tie
                                             (3000, ("uniform", 1, 9), 333, "two_values"),
                                             (9001, ("fixed", 2), 150, "equal"),            # ids of two digits
                                             (3000, ("fixed", 2), 260, "near"),             # equal in 32 bits only
                                             (3000, ("fixed", 2), 260, "near_and_equal"),
                                             (3000, ("uniform", 2, 6), 200, "outliers"),    # one bin holds nearly all
                                             (700, ("uniform", 3, 60), 2000, "iid"),        # everything fits
                                             (1000, ("fixed", 2), 900, "equal"),            # crowded bins, one wave a row
                                             (1000, ("fixed", 2), 900, "outliers"),
                                             (1000, ("uniform", 1, 4), 600, "two_values"),
                                             (1800, ("fixed", 2), 1700, "outliers"),        # two waves a row
                                             (900, ("fixed", 4), 800, "outliers")])         # four waves: few rows
def test_ranking_bins_cuts_and_ties(L, lens, N_b, keys, B_r):
    w = dhsa_inputs.make("c1", L=L, H_q=2, H_kv=1, D=64, N_b=N_b, lens=lens)
    K = w.K.clone()
    k_of = torch.repeat_interleave(torch.arange(w.N_c), torch.from_numpy(np.diff(w.B).astype(np.int64)))
    if keys == "equal":
        K[:] = K[:, :1]
    elif keys == "two_values":
        K[0] = torch.where((k_of % 3 == 0)[:, None], K[0, :1], K[0, 1:2])
    elif keys.startswith("near"):
        K[0, :, 1:] = 1e-10 * K[0, :, 1:]
        K[0, :, 0] = 1.0
        if keys == "near_and_equal":
            K[0] = torch.where((k_of % 5 < 3)[:, None], K[0, :1], K[0])
    elif keys == "outliers":
        K[0] *= torch.where(k_of % 97 == 5, 1e4, 1.0)[:, None]
        K[0] *= torch.where(k_of % 193 == 7, -1e8, 1.0)[:, None]
    Q, Kg = w.Q.cuda(), K.cuda()
    prob = dhsa.problem(Q, Kg, w.B, w.N_b, B_r=B_r)
    plan, ws = dhsa.alloc(prob, w.B)
    plan.fill_(255)
    dhsa.dhsa_route(prob, Q, Kg, w.B, plan, ws)
    rows = np.arange(0, L, 3, dtype=np.int64)
    args = (w.f32("Q"), K.numpy(), w.f32("V"), w.B)
    ref = oracle.prefill_rows_blocks(*args, B_r, N_b, rows) if B_r else oracle.prefill_rows(*args, N_b, rows)
    for h in range(2):
        idx, cnt = dhsa.dhsa_plan_expand_rows(prob, plan, h, rows)
        np.testing.assert_array_equal(cnt.cpu().numpy(), ref[2][h])
        np.testing.assert_array_equal(idx.cpu().numpy(), ref[1][h][:, :idx.shape[1]])


@pytest.mark.parametrize("L,chunk,N_b", [(500, 1, 1000), (4000, 4, 3600), (32768, 40, 2048)])   # one, two, two waves a row
def test_ranking_time_hangs_little_on_the_scores(L, chunk, N_b):
    """Scores that crowd one bin are sorted.  Compared one with another they took 14, 23 and 7 times as long as ordinary
    ones here, sorted 1.0 to 2.6 times: the bound lies between."""
    B = np.r_[np.arange(0, L, chunk), L].astype(np.int32)
    gen = torch.Generator(device="cuda").manual_seed(3)
    Q = torch.randn(12, L, 64, dtype=torch.bfloat16, device="cuda", generator=gen)
    K = torch.randn(1, L, 64, dtype=torch.bfloat16, device="cuda", generator=gen)
    loud = torch.where(torch.arange(L, device="cuda") // chunk % 97 == 5, 1e4, 1.0).to(K.dtype)
    prob = dhsa.problem(Q, K, B, N_b)
    plan, ws = dhsa.alloc(prob, B)
    times = []
    for keys in (K, torch.zeros_like(K), K * loud[None, :, None]):
        best = float("inf")
        for _ in range(12):
            t0, t1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            t0.record()
            for _ in range(4):
                dhsa.dhsa_route(prob, Q, keys, B, plan, ws)
            t1.record()
            torch.cuda.synchronize()
            best = min(best, t0.elapsed_time(t1))
        times.append(best)
    print(f"L={L}: equal scores {times[1] / times[0]:.2f} x, outliers {times[2] / times[0]:.2f} x ordinary ones")
    assert max(times[1:]) < 4.5 * times[0]


@pytest.mark.parametrize("L,H_q,H_kv,D,dtype,N_b,B_r", [(900, 20, 1, 128, "bf16", 31, 0),      # > 16 heads of one kv-head
                                                        (2000, 17, 1, 64, "f32", 1700, 0),
                                                        (5000, 8, 8, 128, "bf16", 4095, 0),    # slices of 128 keys
                                                        (9000, 8, 2, 64, "bf16", 4097, 0),     # one more than 32 of them
                                                        (5000, 8, 2, 128, "bf16", 512, 0),     # the most of 32 keys
                                                        (5000, 8, 2, 64, "f32", 513, 0),       # ... of 64
                                                        (5000, 8, 2, 128, "bf16", 2048, 0),    # the most of 64 keys
                                                        (5000, 8, 2, 64, "bf16", 2049, 0),     # ... of 128
                                                        (17000, 1, 1, 64, "bf16", 16384, 0),   # 256 slices of one head
                                                        (3000, 129, 1, 64, "bf16", 30, 0),     # a slice of 64 keys per head
                                                        (3000, 257, 1, 64, "bf16", 30, 0),     # ... of 128
                                                        (9000, 4, 1, 128, "f32", 8300, 0),
                                                        (3000, 2, 1, 128, "bf16", 1, 64)])
def test_decode_heads_slices_and_merge(L, H_q, H_kv, D, dtype, N_b, B_r):
    w = dhsa_inputs.make("c1" if dtype == "f32" else "c3", L=L, H_q=H_q, H_kv=H_kv, D=D, N_b=N_b)
    Q, K, V = (t.cuda() for t in (w.Q, w.K, w.V))
    prob = dhsa.problem(Q, K, w.B, w.N_b, B_r=B_r)
    ws = dhsa.alloc_decode(prob, w.N_c + 3, L + 100)
    ws.fill_(255)
    O_ref, I_ref, c_ref = oracle.decode_row(w.f32("Q"), w.f32("K"), w.f32("V"), w.B, w.N_b, B_r=B_r)
    first = None
    for valid in (0, w.N_c - 1, w.N_c - 1):            # the workspace serves step after step
        O, idx, cnt = dhsa.dhsa_decode_step(prob, Q, K, V, w.B, ws, w.N_c + 3, L + 100, valid, want_idx=True)
        np.testing.assert_array_equal(cnt.cpu().numpy(), c_ref)
        np.testing.assert_array_equal(idx.cpu().numpy(), I_ref[:, :idx.shape[1]])
        err = np.abs(O.float().cpu().numpy().astype(np.float64) - O_ref).max()
        assert err <= (1e-5 if dtype == "f32" else 2e-2), err
        first = O if first is None else first
        assert torch.equal(first, O)                   # whichever workgroup merges, the order of the sum is the same


@pytest.mark.parametrize("L,N_b,chunk", [(400, 40, 4), (2400, 100, 4), (4800, 400, 4)])      # one, two and four waves a row
def test_ranking_of_infinite_and_nan_scores(L, N_b, chunk):
    """Scores far below the rest leave all others in one bin, which is cut again; NaN rank beyond the infinities, on the
    side of their sign, as the 64-bit images of the scores do."""
    rng = np.random.default_rng(L)
    B = np.arange(0, L + 1, chunk, dtype=np.int32)
    N_c = len(B) - 1
    Q = torch.from_numpy(rng.standard_normal((16, L, 64)).astype(np.float32))
    K = torch.from_numpy(rng.standard_normal((1, L, 64)).astype(np.float32))
    Q[:, :, 0] = 1.0 + 0.1 * Q[:, :, 0]
    K[0, B[3], 0] = -1e7                                                     # the outlier
    for k in range(5, N_c, 9):
        K[0, B[k], 1] = float(np.copysign(np.nan, 1 if k % 2 else -1))
    for k in range(7, N_c, 40):
        K[0, B[k], 0] = float("inf") if k % 80 < 40 else float("-inf")
    Q, K = Q.cuda(), K.cuda()
    prob = dhsa.problem(Q, K, B, N_b)
    plan, ws = dhsa.alloc(prob, B)
    dhsa.dhsa_route(prob, Q, K, B, plan, ws)
    S = dhsa.dhsa_debug_scores(prob, B, ws).cpu().numpy()
    assert np.isnan(S[:, -1]).any() and np.isinf(S[:, -1]).any()
    rows = np.array([0, L // 2 + 1, L - 3, L - 1], dtype=np.int64)
    for h in (0, 15):
        idx, cnt = dhsa.dhsa_plan_expand_rows(prob, plan, h, rows)
        for t, i in enumerate(rows):
            l = i // chunk
            u = (S[h, l, :l + 1] + 0.0).view(np.uint64)
            key = np.where(u >> np.uint64(63), ~u, u | np.uint64(1 << 63))
            left, want = N_b, []
            for k in np.lexsort((np.arange(l + 1), np.uint64(2**64 - 1) - key)):
                n = min(left, i + 1 - B[k] if k == l else chunk)
                want += range(B[k], B[k] + n)
                left -= n
            assert cnt[t].item() == len(want)
            np.testing.assert_array_equal(idx[t, :len(want)].cpu().numpy(), np.sort(want))


@pytest.mark.parametrize("L,D,B_r", [(300, 64, 0), (300, 128, 96), (4100, 64, 0), (4100, 128, 0)])
def test_f32_infinite_values_reach_only_the_rows_that_take_them(L, D, B_r):
    """Rows of a workgroup share blocks of keys that not all of them take (16- and 32-row pieces, both forms)."""
    w = dhsa_inputs.make("c1", L=L, H_q=8, H_kv=2, D=D, N_b=60, lens=("uniform", 16, 64))
    for j, (d, x) in enumerate([(3, float("inf")), (5, float("-inf")), (D - 1, float("nan")), (3, float("-inf"))]):
        w.V[:, (2 * j + 1) * L // 9, d] = x
    Q, K, V = (t.cuda() for t in (w.Q, w.K, w.V))
    O = torch.empty_like(Q)
    prob = dhsa.problem(Q, K, w.B, w.N_b, B_r=B_r)
    plan, ws = dhsa.alloc(prob, w.B)
    dhsa.dhsa_prefill(prob, Q, K, V, w.B, O, plan, ws)
    rows = np.arange(0, L, 1 if L < 2000 else 7, dtype=np.int64)
    Vh = w.f32("V")
    odd = np.where(np.isfinite(Vh), 0.0, Vh)
    args = (w.f32("Q"), w.f32("K"), np.where(np.isfinite(Vh), Vh, 0.0).astype(np.float32), w.B)
    ref, I, cnt = oracle.prefill_rows_blocks(*args, B_r, w.N_b, rows) if B_r else oracle.prefill_rows(*args, w.N_b, rows)
    for h in range(8):
        for t, i in enumerate(rows):
            sel = I[h, t, :cnt[h, t]]
            with np.errstate(invalid="ignore"):
                ref[h, t] += odd[h // 4][sel[sel <= i]].sum(0)               # a row block's list reaches past the row
    got = O[:, torch.from_numpy(rows).cuda()].cpu().numpy().astype(np.float64)
    assert not np.isfinite(ref).all() and np.isfinite(ref).any()
    np.testing.assert_allclose(got, ref, rtol=0, atol=1e-4)


@pytest.mark.parametrize("B_r", [0, 96, 1])
@pytest.mark.parametrize("L,D", [(300, 64), (300, 128), (4100, 64)])
def test_f32_rows_of_nothing_but_minus_infinity(L, D, B_r):
    """The softmax of scores that are all -inf is NaN; beside a finite one they weigh nothing; a row without a key is zero."""
    w = dhsa_inputs.make("c1", L=L, H_q=8, H_kv=2, D=D, N_b=60, lens=("uniform", 16, 64))
    w.Q[:, :, 1] = 1.0
    w.K[:, :80, 1] = float("-inf")
    Q, K, V = (t.cuda() for t in (w.Q, w.K, w.V))
    O = torch.empty_like(Q)
    prob = dhsa.problem(Q, K, w.B, w.N_b, B_r=B_r)
    plan, ws = dhsa.alloc(prob, w.B)
    dhsa.dhsa_prefill(prob, Q, K, V, w.B, O, plan, ws)
    rows = np.arange(0, L, 1 if L < 2000 else 7, dtype=np.int64)
    Qh, Kh, Vh = (w.f32(x).astype(np.float64) for x in "QKV")
    want = np.zeros((8, len(rows), D))
    for h in range(8):
        idx, cnt = (x.cpu().numpy() for x in dhsa.dhsa_plan_expand_rows(prob, plan, h, rows))
        for t, i in enumerate(rows):
            j = idx[t, :cnt[t]]
            j = j[j <= i]
            if len(j):
                s = Kh[h // 4, j] @ Qh[h, i] / np.sqrt(D)
                with np.errstate(invalid="ignore"):
                    p = np.exp(s - s.max())
                want[h, t] = p @ Vh[h // 4, j] / p.sum()
    got = O[:, torch.from_numpy(rows).cuda()].cpu().numpy().astype(np.float64)
    assert np.isnan(want).any() and np.isfinite(want).any()
    np.testing.assert_allclose(got, want, rtol=0, atol=1e-5)


@pytest.mark.parametrize("L,H_q,D", [(2048, 4, 64), (6001, 16, 64), (2048, 4, 128), (6001, 16, 128)])
def test_f32_error_against_64_bits(L, H_q, D):
    """16- and 32-row workgroups.  A score of D unit normals summed in four chains of D / 4 leaves O 1.8e-7 to 2.1e-7
    (relative) from its 64-bit value here; along one chain of D it was 2.7e-7 to 3.3e-7 at such sizes, so the bound lies between."""
    w = dhsa_inputs.make("c1", L=L, H_q=H_q, H_kv=H_q // 4, D=D, N_b=L // 8)
    Q, K, V = (t.cuda() for t in (w.Q, w.K, w.V))
    O = torch.empty_like(Q)
    prob = dhsa.problem(Q, K, w.B, w.N_b)
    plan, ws = dhsa.alloc(prob, w.B)
    dhsa.dhsa_prefill(prob, Q, K, V, w.B, O, plan, ws)
    rows = np.arange(5, L, L // 60, dtype=np.int64)
    ref = oracle.prefill_rows(w.f32("Q"), w.f32("K"), w.f32("V"), w.B, w.N_b, rows)[0]
    got = O[:, torch.from_numpy(rows).cuda()].cpu().numpy().astype(np.float64)
    rel = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    print(f"L={L} D={D}: relative error {rel:.3e}")
    assert rel < 2.4e-7


@pytest.mark.parametrize("dtype,H_q,B_r,N_b", [(torch.float32, 16, 1, 16), (torch.float32, 16, 2, 128),
                                               (torch.bfloat16, 40, 1, 16)])
def test_more_workgroups_than_one_launch_holds(dtype, H_q, B_r, N_b):
    """2^20 row blocks a head: a workgroup of the attention each (fp32: of two rows), and a quarter of one in the ranking
    (40 heads: five launches of the attention, two of the ranking).  Heads are independent and every row's sums have one
    order, so calls of eight heads (2^23 workgroups) give the same bits."""
    L, D = B_r << 20, 64
    gen = torch.Generator(device="cuda").manual_seed(5)
    Q = torch.randn(H_q, L, D, dtype=dtype, device="cuda", generator=gen)
    K, V = (torch.randn(1, L, D, dtype=dtype, device="cuda", generator=gen) for _ in range(2))
    B = np.array([0, 700, 300000, 300050, L], dtype=np.int32)

    def prefill(q):
        prob = dhsa.problem(q, K, B, N_b, B_r=B_r)
        plan, ws = dhsa.alloc(prob, B)
        O = torch.full_like(q, float("nan"))
        dhsa.dhsa_prefill(prob, q, K, V, B, O, plan, ws)
        return O

    whole = prefill(Q)
    assert torch.isfinite(whole[:, -1]).all()
    for h in (0, 8, H_q - 8):
        assert torch.equal(whole[h:h + 8].view(torch.uint8), prefill(Q[h:h + 8]).view(torch.uint8))


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("rows", [64, 49, 32])
def test_rows_of_other_16_row_blocks_keep_their_bits(rows, D):
    """Row tiles of at most 64 rows, two 16-row blocks per wave (at most 32 rows: one).  Logits of one block that grow
    far past its exponent reference late in the key list move that block's reference, and nobody else's."""
    L, H_q, H_kv = 40 * rows, 8, 2
    w = dhsa_inputs.make("c3", L=L, H_q=H_q, H_kv=H_kv, D=D, N_b=300, lens=("fixed", rows))
    Q, K, V = (t.cuda() for t in (w.Q, w.K, w.V))
    prob = dhsa.problem(Q, K, w.B, w.N_b)
    plan, ws = dhsa.alloc(prob, w.B)
    dhsa.dhsa_route(prob, Q, K, w.B, plan, ws)

    def attend(q):
        O = torch.full_like(q, float("nan"))
        dhsa.dhsa_sparse_prefill(prob, q, K, V, w.B, plan, O)
        return O

    before = attend(Q)
    at = torch.arange(L, device="cuda") % rows
    for block in range((rows + 15) // 16):
        mine = at // 16 == block
        loud = torch.where(mine[:, None], 40.0 * Q.float(), Q.float()).to(Q.dtype)    # logits of about 40 (one rms)
        after = attend(loud)
        assert torch.isfinite(after).all()
        assert torch.equal(after[:, ~mine], before[:, ~mine])
        assert not torch.equal(after[:, mine], before[:, mine])


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("tall,middle,short", [((65, 96, 97, 127, 128, 129, 160, 200), (33, 48, 49, 63, 64, 64), (1, 16, 17, 31, 32)),
                                               ((80, 128, 100, 90, 70, 110), (), (1, 15, 32)),
                                               ((), (33, 47, 64, 40, 50, 60), (2, 16, 17, 32)),
                                               ((256, 96), (), ())])
def test_a_tile_has_one_result_in_every_launch(tall, middle, short, D):
    """A class of few row tiles joins the launch of the next taller one.  The more heads, the fewer classes are that
    small: with 4 heads all join, with 512 (1536 workgroups and more of each) none, with 128 of them the shortest may.
    The rows of the first heads keep their bits, so the parity tests of joined launches hold for separate ones too.
    dhsa_prefill does the routing of few tiles in the same launch (k_route_attend), so attention is called apart, too."""
    # the launcher's rule, so that another line in it cannot empty this test
    src = open(os.path.join(os.path.dirname(dhsa.__file__), "csrc", "attn_mfma.hip")).read()
    (most,) = re.findall(r"p\.H_q \* all\[c\] <= (\d+)\)", src)
    classes = [2 * len(c) for c in (tall, middle, short) if c]              # tiles, at least
    assert all(512 * n > int(most) for n in classes) and all(4 * n <= int(most) for n in classes)
    rng = np.random.default_rng(D + len(tall))
    lens = rng.permutation(np.array((tall + middle + short) * 2))
    B = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    L = int(B[-1])
    gen = torch.Generator(device="cuda").manual_seed(3)
    Q, K, V = (torch.randn(H, L, D, dtype=torch.bfloat16, device="cuda", generator=gen) for H in (512, 128, 128))

    def prefill(H_q, B_r):
        q, k, v = Q[:H_q], K[:H_q // 4], V[:H_q // 4]
        prob = dhsa.problem(q, k, B, 300, B_r=B_r)
        plan, ws = dhsa.alloc(prob, B)
        O, apart = torch.full_like(q, float("nan")), torch.full_like(q, float("nan"))
        dhsa.dhsa_prefill(prob, q, k, v, B, O, plan, ws)
        dhsa.dhsa_sparse_prefill(prob, q, k, v, B, plan, apart)
        assert torch.equal(O, apart), (H_q, B_r)
        return O[:4]

    for B_r in (0, 72):                            # row blocks: tiles of 72 rows and one of the rest
        few = prefill(4, B_r)
        assert torch.isfinite(few).all()
        for H_q in (32, 128, 512):
            assert torch.equal(few, prefill(H_q, B_r)), (H_q, B_r)
