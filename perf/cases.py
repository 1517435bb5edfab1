"""What the speed of this library is measured on: its decode steps and prefix expansions as a
serving program calls them, with seeded synthetic inputs.

A case is one call of `typhoon_mla_decode`, `typhoon_mla_decode_tree` or
`typhoon_mla_expand_prefix` at the sizes a serving program meets: the benchmark configurations of
`workloads.py`, rows of the batch sweep in `bench.py`, the tree shape measured there, and ragged
sizes between them.  `naive_only` is left out: it is the baseline formulation of the paper's
Table 1, which nobody serves with.
"""
import math
import random

import torch

from paper_2509_21081_amd import binding as T

D_LATENT, D_NOPE, D_ROPE, D_V = 512, 128, 64, 128
D_QK, D_ROW = D_NOPE + D_ROPE, D_LATENT + D_ROPE
SM_SCALE = 1.0 / math.sqrt(D_QK)


def _decode(name, mode, batch, heads, prefix, suffix, q_len=1, block=64, dtype="bf16"):
    return dict(name=name, kind="decode", mode=mode, dtype=dtype, batch=batch, heads=heads,
                q_len=q_len, prefix=prefix, suffix_min=suffix[0], suffix_max=suffix[1],
                block=block)


def _expand(name, prefix, heads, dtype="bf16"):
    return dict(name=name, kind="expand", dtype=dtype, prefix=prefix, heads=heads)


def listed():
    return [
        # the fp32 mode, at the size of the repository's fp32 configuration: checking a model's
        # outputs against a higher-precision run
        _decode("fp32_tiny", "mixed", 4, 16, 256, (64, 64), dtype="fp32"),
        # one user behind a long system prompt: the smallest batch, where auto mode takes the
        # absorb form of both parts
        _decode("one_user_long_prompt", "auto", 1, 128, 16384, (512, 512)),
        # a tensor-parallel rank's 16 heads at an ordinary small batch with ragged answers
        _decode("rank_small_batch", "auto", 8, 16, 4096, (100, 1200)),
        # a mid-size batch of a 64-head model drafting three tokens, nothing a multiple of a tile
        _decode("drafting_ragged", "mixed", 37, 64, 5003, (1, 1500), q_len=3, block=128),
        # DeepSeek-v3 shape, batch 64: just above the batch where the mixed form starts to pay
        _decode("batch64", "mixed", 64, 128, 4096, (512, 512)),
        # the headline: a 32768-token system prompt shared by 256 requests of ragged length
        _decode("long_prompt", "mixed", 256, 128, 32768, (256, 2048)),
        # multi-token decode (two query positions per request)
        _decode("two_tokens", "mixed", 128, 128, 8192, (1024, 1024), q_len=2),
        # a tensor-parallel rank's 16 heads at a large batch with long answers
        _decode("rank_large_batch", "mixed", 512, 16, 16384, (512, 4096)),
        # a server that does not keep the expanded prefix (memory): Kimi-K2's 64 heads, batch 256
        _decode("latent_only", "absorb_only", 256, 64, 4096, (512, 512)),
        # a system prompt behind which a tenant's prompt is shared by half of the requests each
        dict(name="two_tenants", kind="tree", dtype="bf16", batch=256, heads=128, q_len=1,
             prefix=4096, groups=2, group_prefix=4096, suffix_min=512, suffix_max=512, block=64),
        # expansion of a new shared prompt: a short odd one for a rank's 16 heads, and the
        # headline's for all 128
        _expand("expand_short", 1003, 16),
        _expand("expand_long", 32768, 128),
    ]


def _log_int(rng, lo, hi):
    """A whole number spread over the logarithm of lo ... hi; odd sizes as likely as even ones."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    while True:
        kind = rng.choices(("decode", "tree", "expand", "fp32"), (12, 2, 4, 1))[0]
        heads = rng.choice((16, 32, 64, 128, rng.choice((48, 80, 96))))
        block = rng.choice((64, 64, 128))
        if kind == "expand":
            case = _expand("", _log_int(rng, 200, 32768), heads)
        elif kind == "fp32":
            case = _decode("", rng.choice(("mixed", "absorb_only")), _log_int(rng, 1, 8),
                           rng.choice((16, 32)), _log_int(rng, 32, 600),
                           (_log_int(rng, 1, 40), _log_int(rng, 41, 200)), rng.choice((1, 1, 2)),
                           block, "fp32")
        else:
            q_len = rng.choice((1, 1, 1, 2, 3, 4))
            hi = _log_int(rng, 64, 4096)
            lo = rng.choice((hi, max(1, hi // 8), 1))
            prefix = _log_int(rng, 256, 32768)
            batch = _log_int(rng, 1, 1024)
            if kind == "tree":
                case = dict(name="", kind="tree", dtype="bf16", batch=max(batch, 16), heads=heads,
                            q_len=min(q_len, 2), prefix=prefix, groups=rng.choice((2, 3, 4)),
                            group_prefix=_log_int(rng, 256, 8192), suffix_min=lo, suffix_max=hi,
                            block=block)
            else:
                # the absorb form of a long prefix is served to small batches (or by choice, for
                # memory), the mixed form to large ones; auto covers both
                mode = rng.choice(("auto", "auto", "mixed", "absorb_only"))
                case = _decode("", mode, batch, heads, prefix, (lo, hi), q_len, block)
        w = work(case)
        if w["flops"] <= 4e11 and w["bytes"] <= 1.5e9:
            del case["name"]
            return case


def _randn(gen, shape, dtype, std=1.0):
    x = torch.empty(shape, dtype=dtype, device="cuda")
    x.normal_(0.0, std, generator=gen)
    return x


def _suffix(case, gen, rng, dtype):
    """A paged pool, its shuffled block table and the requests' lengths, known to the host too."""
    B, bs = case["batch"], case["block"]
    lens = [rng.randint(case["suffix_min"], case["suffix_max"]) for _ in range(B)]
    blocks = [-(-n // bs) for n in lens]
    ids = list(range(sum(blocks)))
    rng.shuffle(ids)
    table = torch.zeros((B, max(blocks)), dtype=torch.int32)
    at = 0
    for b, n in enumerate(blocks):
        table[b, :n] = torch.tensor(ids[at:at + n], dtype=torch.int32)
        at += n
    return dict(suffix_pool=_randn(gen, (len(ids), bs, D_ROW), dtype), block_table=table.cuda(),
                suffix_lens=torch.tensor(lens, dtype=torch.int32, device="cuda"),
                max_suffix_len=max(lens))


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    rng = random.Random(seed)
    dtype = {"bf16": torch.bfloat16, "fp32": torch.float32}[case["dtype"]]
    H = case["heads"]
    dims = T.make_dims(H, SM_SCALE, dtype)
    weights = dict(w_uk=_randn(gen, (H, D_NOPE, D_LATENT), dtype, 0.02),
                   w_uv=_randn(gen, (H, D_V, D_LATENT), dtype, 0.02))

    def latent(n):
        return (_randn(gen, (n, D_LATENT), dtype), _randn(gen, (n, D_ROPE), dtype))

    if case["kind"] == "expand":
        c, r = latent(case["prefix"])
        k = torch.empty(T.typhoon_mla_expanded_k_bytes(dims, case["prefix"]), dtype=torch.uint8,
                        device="cuda")
        v = torch.empty(T.typhoon_mla_expanded_v_bytes(dims, case["prefix"]), dtype=torch.uint8,
                        device="cuda")
        return dict(kind="expand", dtype=dtype,
                    args=dict(dims=dims, prefix_ckv=c, prefix_krope=r, prefix_k=k, prefix_v=v,
                              **weights))

    B, S = case["batch"], case["q_len"]
    args = dict(dims=dims, q=_randn(gen, (B, S, H, D_QK), dtype), **weights,
                **_suffix(case, gen, rng, dtype))
    args["out"] = torch.empty((B, S, H, D_V), dtype=dtype, device="cuda")
    args["lse_out"] = torch.empty((B, S, H), dtype=torch.float32, device="cuda")

    def expanded(n):
        c, r = latent(n)
        return T.typhoon_mla_expand_prefix(dims, c, r, weights["w_uk"], weights["w_uv"])

    if case["kind"] == "tree":
        nodes = [(*expanded(case["prefix"]), case["prefix"], 0, 0, B)]
        edges = [B * g // case["groups"] for g in range(case["groups"] + 1)]
        for lo, hi in zip(edges, edges[1:]):
            nodes.append((*expanded(case["group_prefix"]), case["group_prefix"], 1, lo, hi - lo))
        need = T.typhoon_mla_decode_tree_workspace_bytes(dims, B, S, nodes, args["max_suffix_len"])
        args["nodes"] = nodes
    else:
        n, mode = case["prefix"], case["mode"]
        args.update(mode=mode, prefix_len=n)
        if mode != "mixed":
            args["prefix_ckv"], args["prefix_krope"] = latent(n)
        if mode == "mixed":
            args["prefix_k"], args["prefix_v"] = expanded(n)
        elif mode == "auto":
            args["prefix_k"], args["prefix_v"] = T.typhoon_mla_expand_prefix(
                dims, args["prefix_ckv"], args["prefix_krope"], weights["w_uk"], weights["w_uv"])
        need = T.typhoon_mla_decode_workspace_bytes(dims, T.MODES[mode], B, S, n,
                                                    args["max_suffix_len"])
    args["workspace"] = torch.empty(max(need, 256), dtype=torch.uint8, device="cuda")
    return dict(kind=case["kind"], dtype=dtype, args=args)


def run(state):
    if state["kind"] == "expand":
        k, v = T.typhoon_mla_expand_prefix(**state["args"])
        return k.view(state["dtype"]), v.view(state["dtype"])
    if state["kind"] == "tree":
        return T.typhoon_mla_decode_tree(**state["args"])
    return T.typhoon_mla_decode(**state["args"])


def work(case):
    H = case["heads"]
    esz = {"bf16": 2, "fp32": 4}[case["dtype"]]
    weights = 2 * H * D_NOPE * D_LATENT
    if case["kind"] == "expand":
        L = case["prefix"]
        return {"bytes": esz * (L * D_ROW + weights + L * H * (D_QK + D_V)),
                "flops": 2 * L * H * (D_NOPE + D_V) * D_LATENT}
    rows = case["batch"] * case["q_len"] * H
    tokens = case["batch"] * (case["suffix_min"] + case["suffix_max"]) / 2
    base_b = esz * (rows * (D_QK + D_V) + weights + tokens * D_ROW) + 4 * rows
    base_f = 2 * case["q_len"] * H * tokens * (D_ROW + D_LATENT) + \
        2 * rows * (D_NOPE + D_V) * D_LATENT

    def naive(n, sharers):   # the RoPE part of a key is the same for every head
        return (esz * n * (H * (D_NOPE + D_V) + D_ROPE),
                2 * sharers * case["q_len"] * H * n * (D_QK + D_V))

    def absorb(n, sharers):
        return esz * n * D_ROW, 2 * sharers * case["q_len"] * H * n * (D_ROW + D_LATENT)

    if case["kind"] == "tree":
        b, f = naive(case["prefix"], case["batch"])
        gb, gf = naive(case["group_prefix"], case["batch"])
        return {"bytes": base_b + b + case["groups"] * gb, "flops": base_f + f + gf}
    forms = {"mixed": [naive], "absorb_only": [absorb], "auto": [naive, absorb]}[case["mode"]]
    # auto may take either form of the prefix: the one a full-speed GPU would be done with first
    b, f = min((form(case["prefix"], case["batch"]) for form in forms),
               key=lambda bf: max(bf[0] / 8e12, bf[1] / 2.5e15))
    return {"bytes": base_b + b, "flops": base_f + f}


def tolerance(case):
    # about four times what the path differs by from itself in 64 bits (measured 2-norms: decode
    # 2.0e-3 ... 3.2e-3, expansion 1.7e-3, fp32 decode 3.7e-7; largest single differences 1.6e-2,
    # 3.9e-3 and 1.7e-6)
    if case["dtype"] == "fp32":
        return {"rel": 1.5e-6, "max": 7e-6}
    if case["kind"] == "expand":
        return {"rel": 6.8e-3, "max": 1.6e-2}
    return {"rel": 1.2e-2, "max": 6.4e-2}
