"""Row tiles that go to the lone-wave kernels (csrc/attn_wave.hip) because there are many of them, against the same rows of
few heads alone (csrc/attn_mfma.hip takes few tiles), whose bits they have, and against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2510_24606_amd as dhsa

pytestmark = pytest.mark.gpu
H_Q, H_KV, FEW, D = 64, 8, 8, 128


def tensors(L, layout, seed=5):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    out = []
    for H in (H_Q, H_KV, H_KV):
        x = torch.randn((L, H, D) if layout == "lhd" else (H, L, D), dtype=torch.bfloat16, device="cuda", generator=gen)
        out.append(x.transpose(0, 1) if layout == "lhd" else x)
    return out


def run(q, k, v, B, N_b, B_r):
    """The output, the kernels that take the height classes, and the most entries of a list."""
    O = torch.full_like(q, float("nan"))
    prob = dhsa._with_vo(dhsa.problem(q, k, B, N_b, B_r=B_r), v, O)
    plan, ws = dhsa.alloc(prob, B)
    dhsa.dhsa_prefill(prob, q, k, v, B, O, plan, ws)
    return O, dhsa.dhsa_attention_kernels(prob, B)[0], int(dhsa.parse_plan(plan.cpu().numpy())["count"].max())


def check_route(few, every, classes):
    """`every` has the height classes `classes` taken by lone waves, `few` none."""
    assert [c for c in range(3) if every[c] == 1] == list(classes) and 1 not in few, (few, every)


TALL, MIDDLE, SHORT = (97, 128, 110), (65, 96, 80), (33, 64, 50)


@pytest.mark.parametrize("lens,B_r,N_b,layout,classes", [
    ((TALL + MIDDLE) * 19 + SHORT * 25 + (1, 32), 0, 1536, "hld", (0, 1, 2)),
    (TALL * 100 + (1, 16, 63) * 4, 0, 2048, "lhd", (0,)),               # beside classes that keep their launch
    (MIDDLE * 19 + SHORT * 2, 0, 1301, "lhd", (1,)),
    (SHORT * 25 + (129, 97, 65, 3), 0, 4100, "hld", (2,)),
    ((16, 64, 48, 2, 33) * 45, 128, 4101, "hld", (0,)),
    ((30, 64, 2, 50, 20) * 35, 97, 1600, "lhd", (0, 1)),            # the last block has 87 rows
    ((1, 2, 60, 3, 30, 1, 4, 40) * 40, 96, 2047, "hld", (1,)),          # more than four chunks begin among 64 keys
    ((200, 7, 18) * 20, 65, 1100, "lhd", (1,)),
    ((17, 40, 1) * 90, 64, 1999, "hld", (2,)),
    ((100, 3, 33) * 20, 33, 1024, "lhd", (2,))])
def test_many_tiles_give_what_few_give(lens, B_r, N_b, layout, classes):
    many_and_few(lens, B_r, N_b, layout, classes)


@pytest.mark.parametrize("lens,B_r,N_b,layout,classes", [
    ((20, 30, 40, 45) * 160, 128, 10007, "hld", (0, 1)),
    ((17, 20, 15, 18) * 260, 96, 6007, "lhd", (1,)),
    ((17, 20, 15, 18) * 260, 64, 7001, "hld", (2,)),
    ((17, 20, 15, 18) * 260, 40, 7001, "lhd", (2,))])
def test_lists_of_several_parts(lens, B_r, N_b, layout, classes):
    """The lone-wave kernels take a list's entries 64 at a time; after 256, where attn_mfma.hip starts a new segment table,
    both go on with a new tile."""
    assert many_and_few(lens, B_r, N_b, layout, classes) > 300


def many_and_few(lens, B_r, N_b, layout, classes):
    """Checks the output of all heads; returns the most entries of a list."""
    B = np.concatenate([[0], np.cumsum(np.random.default_rng(len(lens)).permutation(lens))]).astype(np.int32)
    L = int(B[-1])
    q, k, v = tensors(L, layout)
    every, kernels, entries = run(q, k, v, B, N_b, B_r)
    for g in (0, 3, H_KV - 1):      # the query heads of a kv-head alone: a row gets the same bits
        few, kernels_few, _ = run(q[FEW * g:FEW * (g + 1)], k[g:g + 1], v[g:g + 1], B, N_b, B_r)
        check_route(kernels_few, kernels, classes)
        assert torch.equal(every[FEW * g:FEW * (g + 1)], few), g
    # the weights, which sum to 1, and the result are rounded to 8 bits, each by at most 2^-8 of the largest value of V (sums
    # in 32 bits add less than 2^-14 of it).  In the norm each rounding is a uniform error of at most 2^-8 of its value, and the
    # two are independent: sqrt(2 / 3) 2^-8 = 3.2e-3 of the result at most (values are not all just above a power of two: 2.3e-3)
    tol = (2.0 ** -7 + 2.0 ** -14) * float(v[0].float().abs().max())

    assert bool(torch.isfinite(every).all())
    rows = np.unique(np.r_[np.linspace(0, L - 1, 40).astype(np.int64), B[1:6] - 1, L - 2])
    f32 = [x.float().cpu().numpy() for x in (q[:2], k[:1], v[:1])]
    ref = oracle.prefill_rows_blocks(*f32, B, B_r, N_b, rows)[0] if B_r else oracle.prefill_rows(*f32, B, N_b, rows)[0]
    got = every[:2, torch.from_numpy(rows).cuda()].float().cpu().numpy()
    assert np.abs(got - ref).max() <= tol and np.linalg.norm(got - ref) <= 3.2e-3 * np.linalg.norm(ref)
    return entries


@pytest.mark.parametrize("rows", [128, 96, 64])
def test_references_that_move_and_values_that_are_not_finite(rows):
    """Logits that outgrow their exponent reference late in the list; NaN, infinite and lowest keys and values: what the
    four-wave kernels make of them, and nothing in chunks before the first."""
    B = np.arange(0, 73 * rows + 1, rows, dtype=np.int32)
    L = int(B[-1])
    q, k, v = tensors(L, "hld", rows)
    q *= torch.linspace(1, 8, L, device="cuda")[None, :, None]     # (a weight that vanishes would make NaN of an infinite value)
    k, v = k.clone(), v.clone()
    for j, (x, val) in enumerate([(v, float("inf")), (v, float("-inf")), (v, float("nan")), (k, torch.finfo(torch.bfloat16).min),
                                  (k, float("inf")), (k, float("nan"))]):
        x[:, (10 + 10 * j) * rows + j, j] = val
    B_r = rows if rows == 128 else 0      # (few tiles of 128 rows of a chunk each stay with four waves)
    every, kernels, _ = run(q, k, v, B, 1536, B_r)
    few, kernels_few, _ = run(q[:FEW], k[:1], v[:1], B, 1536, B_r)
    check_route(kernels_few, kernels, [{128: 0, 96: 1, 64: 2}[rows]])
    got, want = every[:FEW].float(), few.float()
    assert bool(torch.isnan(want).any()) and bool(torch.isinf(want).any())
    assert bool(torch.isfinite(want[:, :10 * rows]).all())
    torch.testing.assert_close(got, want, rtol=0, atol=0, equal_nan=True)
