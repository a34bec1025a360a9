"""Routing whose launches are joined because a problem is small (k_score_select, k_decode_few, k_route_attend), against the same routing by
the launches of larger problems: scores, plans and outputs are the same bits."""
import numpy as np
import pytest
import torch

import paper_2510_24606_amd as dhsa

pytestmark = pytest.mark.gpu
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def tensors(H_q, H_kv, L, D, dtype, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return [torch.randn((H, L, D), dtype=DTYPES[dtype], device="cuda", generator=gen) for H in (H_q, H_kv, H_kv)]


def boundaries(N_c, longest, seed):
    return np.concatenate([[0], np.cumsum(np.random.default_rng(seed).integers(1, longest + 1, N_c))]).astype(np.int32)


@pytest.mark.parametrize("N_c,D,dtype,B_r,pooling", [
    (1, 128, "bf16", 0, 0), (2, 64, "f32", 0, 0), (15, 128, "f32", 0, 1), (16, 64, "bf16", 0, 0), (17, 128, "bf16", 7, 0),
    (33, 128, "bf16", 0, 0), (48, 64, "f32", 32, 1), (63, 128, "bf16", 100, 0), (64, 128, "f32", 0, 0), (64, 64, "bf16", 0, 0),
    (65, 128, "bf16", 0, 0), (100, 64, "f32", 0, 0), (128, 128, "bf16", 0, 1), (128, 64, "bf16", 33, 0), (129, 128, "bf16", 0, 0)])
def test_few_groups_get_the_scores_and_plans_of_many(N_c, D, dtype, B_r, pooling):
    B = boundaries(N_c, 20, N_c)
    L = int(B[-1])
    q, k, _ = tensors(2, 1, L, D, dtype, N_c)
    N_b = max(1, L // 5)

    def route(q, k):
        prob = dhsa.problem(q, k, B, N_b, B_r=B_r, pooling=pooling)
        plan, ws = dhsa.alloc(prob, B)
        ws.fill_(255)
        dhsa.dhsa_route(prob, q, k, B, plan, ws)
        return dhsa.parse_plan(plan.cpu().numpy()), dhsa.dhsa_debug_scores(prob, B, ws)

    few, s_few = route(q, k)
    N_q = s_few.shape[1]
    times = -(-512 // (2 * N_q))                      # as many heads as 512 groups take
    many, s_many = route(q.repeat(times, 1, 1), k.repeat(times, 1, 1))
    ends = np.minimum((np.arange(N_q) + 1) * B_r, L) if B_r else B[1:]
    seen = torch.from_numpy(B[None, :-1] < ends[:, None]).cuda()
    for h in range(2):
        assert torch.equal(s_few[h][seen], s_many[h][seen]) and bool(torch.isfinite(s_few[h][seen]).all())
        assert np.array_equal(few["count"][h], many["count"][h])
        for l in range(N_q):
            n = few["count"][h][l]
            assert np.array_equal(few["entries"][h][l][:n], many["entries"][h][l][:n]), (h, l)


@pytest.mark.parametrize("N_c,n_new,D,dtype,B_r,pooling", [
    (2, 1, 128, "bf16", 0, 0), (5, 3, 64, "f32", 0, 1), (16, 2, 128, "bf16", 0, 0), (17, 1, 128, "f32", 0, 0), (40, 3, 64, "bf16", 50, 0),
    (64, 2, 128, "bf16", 128, 1), (100, 1, 128, "bf16", 0, 0), (128, 1, 64, "f32", 0, 0), (128, 3, 128, "bf16", 0, 0), (129, 1, 128, "bf16", 0, 0)])
def test_joined_decoding_steps_give_what_separate_ones_give(N_c, n_new, D, dtype, B_r, pooling):
    B = boundaries(N_c, 60, N_c)
    L = int(B[-1])
    q, k, v = tensors(6, 2, L, D, dtype, N_c)
    prob = dhsa.problem(q, k, B, max(1, L // 3), B_r=B_r, pooling=pooling, V=v)
    caps = (N_c + 4, L + 100)
    ws = dhsa.alloc_decode(prob, *caps)
    want = dhsa.dhsa_decode_step(prob, q, k, v, B, ws, *caps, 0, want_idx=True)      # pools all keys: never joined
    ws2 = dhsa.alloc_decode(prob, *caps)
    old = B[:N_c - n_new + 1].copy()                                                 # the sequence before its newest chunks
    Lo = int(old[-1])
    qo, ko, vo = (x[:, :Lo].contiguous() for x in (q, k, v))
    dhsa.dhsa_decode_step(dhsa.problem(qo, ko, old, max(1, L // 3), B_r=B_r, pooling=pooling, V=vo), qo, ko, vo, old, ws2, *caps, 0)
    for valid in (N_c - n_new, N_c - 1):      # the second step takes what the first one has pooled
        got = dhsa.dhsa_decode_step(prob, q, k, v, B, ws2, *caps, valid, want_idx=True)
        for x, y in zip(got, want):
            assert torch.equal(x, y), valid


@pytest.mark.parametrize("N_c,dtype,B_r", [(513, "bf16", 0), (1030, "f32", 0), (2049, "bf16", 0), (2600, "bf16", 40), (8192, "bf16", 0)])
@pytest.mark.parametrize("values", ["normal", "equal"])
def test_long_lists_of_few_rows(N_c, dtype, B_r, values):
    """A step's ranking by eight waves gives the keys that the prefill's routing, of many rows, gives the last row.  (8192 chunks:
    the list may hold more than 1024 of them, which the kernel that sorts the whole row ranks in both.)"""
    long_lists(N_c, dtype, B_r, values, None)


@pytest.mark.parametrize("N_c,dtype,B_r", [(4097, "f32", 0), (5000, "bf16", 33), (8192, "bf16", 0)])
@pytest.mark.parametrize("values", ["normal", "equal", "two"])
def test_rows_of_more_chunks_than_eight_waves_hold(N_c, dtype, B_r, values):
    """More than 4096 scores are read again in every pass; the list is short enough for the ranking by eight waves."""
    long_lists(N_c, dtype, B_r, values, 700)


def long_lists(N_c, dtype, B_r, values, N_b):
    B = boundaries(N_c, 3, N_c)
    L = int(B[-1])
    q, k, v = tensors(2, 1, L, 64, dtype, N_c)
    if values == "equal":
        k = torch.ones_like(k)
    elif values == "two":                                 # scores that tie by the thousand
        k = torch.where(k[..., :1] > 0.5, 2.0, 1.0).to(k.dtype).expand_as(k).contiguous()
    prob = dhsa.problem(q, k, B, N_b or L // 6, B_r=B_r, V=v)
    plan, ws = dhsa.alloc(prob, B)
    dhsa.dhsa_route(prob, q, k, B, plan, ws)
    assert (dhsa.parse_plan(plan.cpu().numpy())["stride"] <= 1024) == (N_b is not None or N_c <= 2600)
    caps = (N_c, L)
    _, idx, cnt = dhsa.dhsa_decode_step(prob, q, k, v, B, dhsa.alloc_decode(prob, *caps), *caps, 0, want_idx=True)
    for h in range(2):
        want, n = (x.cpu().numpy()[0] for x in dhsa.dhsa_plan_expand_rows(prob, plan, h, np.array([L - 1], dtype=np.int64)))
        want = want[:n][want[:n] <= L - 1]
        assert np.array_equal(idx[h].cpu().numpy()[:len(want)], want) and int(cnt[h]) == len(want)


@pytest.mark.parametrize("N_c,longest,H_q,D,dtype,B_r", [
    (1, 300, 2, 128, "bf16", 0), (3, 1, 2, 64, "f32", 0), (16, 40, 6, 128, "bf16", 0), (17, 150, 4, 64, "bf16", 0), (33, 60, 2, 128, "f32", 0),
    (64, 130, 8, 128, "bf16", 0), (64, 20, 2, 64, "f32", 0), (40, 60, 4, 128, "bf16", 96), (50, 30, 2, 64, "f32", 17), (64, 9, 2, 128, "bf16", 300),
    (65, 40, 2, 128, "bf16", 0)])
def test_prefill_in_one_launch_gives_what_routing_and_attention_give(N_c, longest, H_q, D, dtype, B_r):
    B = boundaries(N_c, longest, N_c + H_q)
    L = int(B[-1])
    q, k, v = tensors(H_q, 2, L, D, dtype, L)
    prob = dhsa._with_vo(dhsa.problem(q, k, B, max(1, L // 3), B_r=B_r), v, q)

    def plan_ws():
        plan, ws = dhsa.alloc(prob, B)
        plan.fill_(0x55)
        ws.fill_(255)
        return plan, ws

    (p1, w1), (p2, w2) = plan_ws(), plan_ws()
    O1, O2 = torch.full_like(q, float("nan")), torch.full_like(q, float("nan"))
    dhsa.dhsa_prefill(prob, q, k, v, B, O1, p1, w1)
    dhsa.dhsa_route(prob, q, k, B, p2, w2)
    dhsa.dhsa_sparse_prefill(prob, q, k, v, B, p2, O2)
    assert torch.equal(O1, O2) and torch.equal(p1, p2) and bool(torch.isfinite(O1).all())
    s1, s2 = dhsa.dhsa_debug_scores(prob, B, w1), dhsa.dhsa_debug_scores(prob, B, w2)
    ends = np.minimum((np.arange(s1.shape[1]) + 1) * B_r, L) if B_r else B[1:]
    seen = torch.from_numpy(B[None, :-1] < ends[:, None]).cuda().expand(H_q, -1, -1)
    assert torch.equal(s1[seen], s2[seen]) and bool(torch.isfinite(s1[seen]).all())
