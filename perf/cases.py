"""What a user of this framework has it do, as cases that can be timed and compared.

Each case names one public entry point and a problem:

  prefill      one attention layer of a prompt, routing and attention (dhsa_prefill)
  static       the same without a workspace argument (dhsa_prefill_static)
  attend       attention alone over a plan that is kept (dhsa_sparse_prefill; the paper caches routing results)
  decode       one step of a generation loop for the newest token (dhsa_decode_step)
  boundaries   boundary scores of a prompt -> chunk boundaries on the host (dhsa_finalize_boundaries)
  recall       how well the routed sets of sampled rows cover exact top-k attention (dhsa_recall_rows)

The five prefill problems c1..c5 are the configurations of dhsa_inputs (shapes, budgets, chunk-length
laws and the structure of the keys); the inputs here follow the same distributions but are made on the
GPU, since they are made often.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import dhsa_inputs
import paper_2510_24606_amd as dhsa

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}


def _problem(op, L, H_q, H_kv, D, dtype, N_b, law, structure, **options):
    """A case of an entry point that works on Q, K (and V).  law: (name, a, b, c) as in dhsa_inputs."""
    law = tuple(law) + (0,) * (4 - len(law))
    c = dict(op=op, L=L, H_q=H_q, H_kv=H_kv, D=D, dtype=dtype, N_b=N_b, law=law[0], law_a=law[1], law_b=law[2],
             law_c=law[3], structure=structure, B_r=0, pooling="robust", layout="hld")
    c.update(options)
    return c


def _config(name, op="prefill", **options):
    """A case on the shapes of configuration `name` of dhsa_inputs."""
    s = dhsa_inputs.SPECS[name]
    return _problem(op, s["L"], s["H_q"], s["H_kv"], s["D"], s["dtype"], s["N_b"], s["lens"], s["structure"], **options)


def listed():
    cases = {
        # a small fp32 problem: a prompt of 2K tokens, where launches and latency count
        "prefill_c1_f32": _config("c1"),
        # the smallest call of a serving loop that cannot allocate: a short prompt of odd length
        "prefill_short_static": _problem("static", 1021, 8, 2, 128, "bf16", 128, ("uniform", 16, 64), "mixture"),
        # an ordinary prompt, 32K tokens at the LLaMA shape
        "prefill_c2": _config("c2"),
        # the headline: 128K tokens at 6.25 % density
        "prefill_c3": _config("c3"),
        # chunk lengths spread widely around 64: many short row tiles, a small budget
        "prefill_c4": _config("c4"),
        # groups of seven query heads, dense budget, chunks up to 256
        "prefill_c5": _config("c5"),
        # Alg. 1 as printed, fixed row blocks of 128 rows, on the headline problem
        "prefill_c3_row_blocks": _config("c3", B_r=128),
        # attention over a kept plan, on projections as a model has them ([L, H, D] rows), heads of 64,
        # fixed chunks with plain averages (the ablation, conventional block-sparse attention)
        "attend_kept_plan_d64": _problem("attend", 16384, 16, 4, 64, "bf16", 2048, ("fixed", 64), "iid",
                                         pooling="mean", layout="lhd"),
        # a generation loop at full context: pooled keys of the closed chunks are there from the step before
        "decode_c3": _config("c3", op="decode"),
        # ... and early in a conversation
        "decode_short": _problem("decode", 3001, 8, 2, 128, "bf16", 512, ("uniform", 32, 128), "mixture"),
        # boundaries of a 128K prompt from a detector's scores: once per prompt
        "boundaries_128k": dict(op="boundaries", L=131072, window=8, threshold=0.4, peak_lo=20, peak_hi=80),
        # quality diagnostic on sampled rows of one head of an ordinary prompt
        "recall_c2": _config("c2", op="recall", n_rows=48),
    }
    return [dict(c, name=n) for n, c in cases.items()]


def _log(rng, lo, hi):
    """A whole number between lo and hi, spread over the logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _mean_length(case):
    if case["law"] == "uniform":
        return 0.5 * (case["law_a"] + case["law_b"])
    return float(case["law_a"])


def _attention_cost(case):
    """Rows of K and V that the row tiles of an attention pass have to see, all heads (a tile is at
    most 128 rows of one query group)."""
    group = case["B_r"] or _mean_length(case)
    tiles = case["L"] / group * math.ceil(group / 128)
    return case["H_q"] * tiles * min(case["N_b"], case["L"]) * case["D"]


def draw(rng):
    op = rng.choice(["prefill"] * 5 + ["static", "attend", "decode", "decode", "boundaries", "recall"])
    if op == "boundaries":
        lo = rng.randint(10, 40)
        return dict(op=op, L=_log(rng, 1024, 131072), window=_log(rng, 4, 64), threshold=round(rng.uniform(0.25, 0.6), 3),
                    peak_lo=lo, peak_hi=lo + rng.randint(20, 100))
    dtype = "f32" if rng.random() < 0.2 else "bf16"
    D = rng.choice([64, 128, 128])
    small = dtype == "f32" or op == "static"
    H_kv = rng.choice([1, 2, 4]) if small else rng.choice([2, 4, 8])
    H_q = H_kv * (rng.choice([1, 2, 4]) if small else rng.choice([2, 4, 4, 7] if H_kv <= 4 else [2, 4]))
    L = _log(rng, 512, 8192 if small else 131072)
    if L >= 1024 and rng.random() < 0.4:
        L = L // 1024 * 1024                    # a round context length; the others are odd ones
    kind = rng.random()
    if kind < 0.6:
        lo = rng.choice([8, 16, 32] if L <= 65536 else [16, 32])       # at most 8192 chunks
        law = ("uniform", lo, lo * rng.choice([3, 4, 8]))
    elif kind < 0.85:
        law = ("geometric", rng.choice([48, 64, 96]), 8, 512)
    else:
        law = ("fixed", rng.choice([32, 64, 128]))
    case = _problem(op, L, H_q, H_kv, D, dtype, max(16, int(L * rng.choice([1 / 32, 1 / 16, 1 / 16, 1 / 8]))), law,
                    rng.choice(["iid", "needles", "mixture", "loud_chunks", "lowrank"]),
                    B_r=rng.choice([64, 128, 128, 256]) if rng.random() < 0.3 else 0,
                    pooling="mean" if rng.random() < 0.2 else "robust", layout="lhd" if rng.random() < 0.3 else "hld")
    if op == "recall":
        case["n_rows"] = rng.randint(16, 64)
    # no drawn case is heavier than the headline: the budget gives way
    case["N_b"] = max(16, int(case["N_b"] * min(1.0, 0.9 * _attention_cost(_config("c3")) / _attention_cost(case))))
    return case


def _boundaries(case, seed):
    law = tuple(x for x in (case["law"], case["law_a"], case["law_b"], case["law_c"]) if x)
    return dhsa_inputs.draw_boundaries(np.random.default_rng([seed, 1]), case["L"], law)


def _normal(gen, H, L, D, dtype, layout):
    """Standard normals [H, L, D], contiguous or as a view of [L, H, D] (a projection's output)."""
    shape = (H, L, D) if layout == "hld" else (L, H, D)
    x = torch.randn(shape, dtype=dtype, device="cuda", generator=gen)
    return x if layout == "hld" else x.transpose(0, 1)


def _structured_keys(case, seed, B, Q, K):
    """Gives K the structure that the configurations of dhsa_inputs have, head by head."""
    L, D, G, N_c = case["L"], case["D"], case["H_q"] // case["H_kv"], len(B) - 1
    gen = torch.Generator(device="cuda").manual_seed(seed * 4 + 3)
    rx = np.random.default_rng([seed, 2])
    lens = torch.from_numpy(np.diff(B).astype(np.int64)).cuda()
    kind = case["structure"]

    def per_token(per_chunk):
        return torch.repeat_interleave(per_chunk, lens, dim=0, output_size=L)

    if kind == "lowrank":
        Z = torch.randn(L, 8, device="cuda", generator=gen)
    for g in range(case["H_kv"]):
        if kind == "needles":     # key chunks shifted along the direction of a later query
            n, hi = min(64, max(1, N_c // 4)), max(1, int(N_c * 0.9))
            ids = rx.choice(hi, size=min(n, hi), replace=False)
            at = np.minimum(B[ids + 1] + (rx.random(len(ids)) * (L - B[ids + 1])).astype(np.int64), L - 1)
            heads = g * G + rx.integers(0, G, size=len(ids))
            q = Q[torch.from_numpy(heads).cuda(), torch.from_numpy(at).cuda()].float()
            shift = torch.zeros(N_c, D, device="cuda")
            shift[torch.from_numpy(ids).cuda()] = q * (3.0 * math.sqrt(D) / q.square().sum(1, keepdim=True))
            K[g] += per_token(shift).to(K.dtype)
        elif kind == "mixture":   # the keys of a chunk share one of 256 centres
            centres = torch.randn(256, D, device="cuda", generator=gen)
            of_chunk = centres[torch.from_numpy(rx.integers(0, 256, size=N_c)).cuda()]
            K[g] = (0.3 * K[g].float() + per_token(of_chunk)).to(K.dtype)
        elif kind == "loud_chunks":
            loud = torch.from_numpy(np.where(rx.random(N_c) < 0.01, 4.0, 1.0)).cuda()
            K[g] *= per_token(loud)[:, None].to(K.dtype)
        elif kind == "lowrank":   # a component of rank 8 that all keys share
            W = torch.randn(8, D, device="cuda", generator=gen)
            K[g] += ((0.5 / math.sqrt(8.0)) * (Z @ W)).to(K.dtype)


def _detector_scores(case, seed):
    """A low noise floor with a sharp peak and its shoulders at every chunk end."""
    rng = np.random.default_rng([seed, 3])
    L = case["L"]
    p = 0.2 * rng.random(L)
    at = np.cumsum(rng.integers(case["peak_lo"], case["peak_hi"], size=L // case["peak_lo"] + 2))
    at = at[at < L]
    p[at] += 0.5 + 0.3 * rng.random(len(at))
    for d in (-1, 1):
        ok = (at + d >= 0) & (at + d < L)
        p[at[ok] + d] += 0.3
    return torch.from_numpy(p.astype(np.float32)).cuda()


def prepare(case, seed):
    if case["op"] == "boundaries":
        # the caller keeps its boundaries in an array with room for any number of chunks (zeros behind them)
        return dict(case=case, scores=_detector_scores(case, seed), B=np.zeros(case["L"] + 1, dtype=np.int32))
    op, L, dtype, layout = case["op"], case["L"], DTYPES[case["dtype"]], case["layout"]
    B = _boundaries(case, seed)
    gen = torch.Generator(device="cuda").manual_seed(seed * 4 + 1)
    Q = _normal(gen, case["H_q"], L, case["D"], dtype, layout)
    K = _normal(gen, case["H_kv"], L, case["D"], dtype, layout)
    _structured_keys(case, seed, B, Q, K)
    pooling = dhsa.DHSA_POOL_MEAN if case["pooling"] == "mean" else dhsa.DHSA_POOL_ROBUST
    s = dict(case=case, Q=Q, K=K, B=B, pooling=pooling)
    if op != "recall":
        s["V"] = _normal(gen, case["H_kv"], L, case["D"], dtype, layout)
    prob = dhsa.problem(Q, K, B, case["N_b"], B_r=case["B_r"], pooling=pooling, V=s.get("V"))
    s["prob"] = prob
    if op == "decode":
        # the loop has run up to the token before: its workspace holds the pooled keys of the closed chunks
        s["caps"] = (min(len(B) - 1 + 64, 8192), L + 4096)
        s["ws"] = dhsa.alloc_decode(prob, *s["caps"])
        dhsa.dhsa_decode_step(prob, Q, K, s["V"], B, s["ws"], *s["caps"], 0)
        return s
    if op == "recall":
        rng = np.random.default_rng([seed, 4])
        s["head"] = int(rng.integers(case["H_q"]))
        s["rows"] = np.sort(rng.choice(L, size=case["n_rows"], replace=False)).astype(np.int64)
    else:
        s["O"] = torch.empty_like(Q)            # keeps the strides of Q
    s["plan"], s["ws"] = dhsa.alloc(prob, B)
    if op in ("attend", "recall"):
        dhsa.dhsa_route(prob, Q, K, B, s["plan"], s["ws"])
        del s["ws"]
    elif op == "static":
        del s["ws"]
    return s


def run(s):
    c = s["case"]
    op = c["op"]
    if op == "boundaries":
        B = dhsa.dhsa_finalize_boundaries(s["scores"], c["threshold"], c["window"])
        s["B"][:len(B)] = B
        return {"B": s["B"], "N_c": len(B) - 1}
    if op == "prefill":
        dhsa.dhsa_prefill(s["prob"], s["Q"], s["K"], s["V"], s["B"], s["O"], s["plan"], s["ws"])
        return s["O"]
    if op == "static":
        dhsa.dhsa_prefill_static(s["prob"], s["Q"], s["K"], s["V"], s["B"], s["O"], s["plan"])
        return s["O"]
    if op == "attend":
        dhsa.dhsa_sparse_prefill(s["prob"], s["Q"], s["K"], s["V"], s["B"], s["plan"], s["O"])
        return s["O"]
    if op == "decode":
        # the sequence grows with every step of a generation loop, so the step describes its problem anew
        prob = dhsa.problem(s["Q"], s["K"], s["B"], c["N_b"], B_r=c["B_r"], pooling=s["pooling"], V=s["V"])
        return dhsa.dhsa_decode_step(prob, s["Q"], s["K"], s["V"], s["B"], s["ws"], *s["caps"], len(s["B"]) - 2)
    return dhsa.dhsa_recall_rows(s["prob"], s["Q"], s["K"], s["B"], s["plan"], s["head"], s["rows"])


def work(case):
    L = case["L"]
    if case["op"] == "boundaries":
        return {"bytes": 4.0 * L + 4.0 * L / (0.5 * (case["peak_lo"] + case["peak_hi"])), "flops": float(L)}
    H_q, H_kv, D, nb = case["H_q"], case["H_kv"], case["D"], min(case["N_b"], L)
    esz = 4.0 if case["dtype"] == "f32" else 2.0
    N_c = max(1.0, L / _mean_length(case))
    if case["op"] == "decode":
        # the selected K and V rows (the heads of a group select their own), the pooled keys, the open group's queries
        rows = min(H_q * nb, H_kv * L)
        return {"bytes": 2.0 * rows * D * esz + 8.0 * H_kv * N_c * D + 2.0 * H_q * D * esz,
                "flops": 4.0 * H_q * nb * D + 2.0 * H_q * N_c * D}
    if case["op"] == "recall":
        return {"bytes": (L + case["n_rows"]) * D * esz, "flops": case["n_rows"] * (L / 2.0) * 2.0 * D}
    pairs = H_q * (L * nb - nb * (nb - 1) / 2.0)            # selected (row, key) pairs
    N_q = math.ceil(L / case["B_r"]) if case["B_r"] else N_c
    route = H_q * N_q * N_c * D + (H_q + H_kv) * L * D      # scores of the visible chunk pairs, pooled sums
    if case["op"] == "attend":
        route = 0.0
    return {"bytes": (2.0 * H_q + 2.0 * H_kv) * L * D * esz, "flops": 4.0 * D * pairs + route}


def tolerance(case):
    if case["op"] in ("boundaries", "recall"):
        return "exact"
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-4}
    # outputs and probabilities are rounded to bf16 (2^-9 relative each)
    return {"rel": 1e-2, "max": 6e-2}
