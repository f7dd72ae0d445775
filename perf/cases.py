"""Cases of the dynamic-sparse GEMM hot path: what a program built on this library has it do, through the
public entry points of ``paper_2301_10936_amd.pit``, over the range of sizes it is used at.

Kinds of case (``case["kind"]``) and what each stands for in real use:

ffn         down-projection of a ReLU feed-forward block: the activation arrives channel-major, its sparsity
            index is rebuilt on every call (a new activation every step), the product runs over the listed
            micro-tiles.  Independent zeros ("live" = 1) or whole micro-tiles silenced in runs of tokens.
select      the same product when the caller lets the cost model choose the kernel (tile height or dense).
preact      the same layer entered one step earlier: the token-major pre-activation; ReLU, layout change and
            index in one call, then the product.
microtile   a row-major operand with 1 x 32, 1 x 64 or 1 x 128 micro-tiles along k (pruned weights, block sparsity).
moe         top-1 mixture-of-experts feed-forward: a prefill batch of thousands of tokens, or a decode step of a few.
padded      linear layer over a padded batch of sequences of different lengths, valid rows only (forward; the
            gradient with respect to the input is the same call with the transposed weights).
wgrad       gradient of that layer's weights over the valid tokens only (the tokens are the reduction axis).
attn        attention under a dynamic mask: local window plus key columns chosen per block of 32 queries.

Buffers that a training or serving loop allocates once (index, workspace, output) are made in ``prepare``.  Index
lists are allocated zeroed, so that the entries past the end of a list are the same everywhere.
"""
from __future__ import annotations

import json
import math
import os

import torch

from paper_2301_10936_amd import pit

_PROFILE = os.path.join(os.path.dirname(os.path.abspath(pit.__file__)), "tile_cost_mi355x.json")


# ------------------------------------------------------------------------------------------------ the cases
def listed():
    return [
        # the smallest layer call: a handful of launches, nothing fills the chip
        {"name": "ffn_small", "kind": "ffn", "M": 256, "K": 512, "N": 256, "mt": 128, "live": 1.0, "run": 128,
         "dtype": "bf16", "out": "f32"},
        # OPT-size down-projection, independent zeros: every k-list is (almost) full
        {"name": "ffn_2048x8192x2048", "kind": "ffn", "M": 2048, "K": 8192, "N": 2048, "mt": 128, "live": 1.0, "run": 128,
         "dtype": "bf16", "out": "f32"},
        # zeros correlated over runs of 64 tokens, followed at that height; odd sizes, half precision out
        {"name": "ffn_ragged_runs64", "kind": "ffn", "M": 1856, "K": 5003, "N": 1408, "mt": 64, "live": 0.25, "run": 64,
         "dtype": "f16", "out": "f16"},
        # the 4096^3 micro-benchmark at 90 % zeros in runs of 32 tokens, kernel chosen by cost
        {"name": "select_4096_runs32", "kind": "select", "M": 4096, "K": 4096, "N": 4096, "live": 0.1, "run": 32,
         "dtype": "bf16", "out": "f32"},
        # the layer from the token-major pre-activation, three quarters of the channels dead per 128 tokens
        {"name": "preact_2048x8192x2048", "kind": "preact", "M": 2048, "K": 8192, "N": 2048, "live": 0.25,
         "dtype": "bf16", "out": "f32"},
        # 1 x 32 micro-tiles, 10 % kept, at a size where launches and latency decide
        {"name": "microtile_1x32_1024", "kind": "microtile", "M": 1024, "K": 1024, "N": 1024, "mt": 32, "keep": 0.1,
         "dtype": "f16"},
        # 1 x 64 micro-tiles, 10 % kept, at the size of the micro-benchmark sweep
        {"name": "microtile_1x64_4096", "kind": "microtile", "M": 4096, "K": 4096, "N": 4096, "mt": 64, "keep": 0.1,
         "dtype": "bf16"},
        # Switch-style layer, prefill: every expert's weights are read once per call
        {"name": "moe_prefill_4096x64", "kind": "moe", "T": 4096, "d_model": 768, "d_ff": 3072, "E": 64, "gate": True,
         "dtype": "bf16", "out": "f32"},
        # the same layer, one decode step of a batch of 48 sequences (48 rows are all that it gives back)
        {"name": "moe_decode_48x64", "kind": "moe", "T": 48, "d_model": 768, "d_ff": 3072, "E": 64, "gate": True,
         "dtype": "bf16", "out": "bf16"},
        # linear layer over a padded batch, lengths 16 .. 512
        {"name": "padded_32x512", "kind": "padded", "batch": 32, "max_len": 512, "min_len": 16, "hidden": 1024, "N": 4096,
         "dtype": "bf16", "out": "bf16"},
        # its weight gradient: valid tokens as the reduction axis, fp32 result
        {"name": "wgrad_32x512", "kind": "wgrad", "batch": 32, "max_len": 512, "min_len": 16, "hidden": 1024, "N": 4096,
         "dtype": "bf16", "out": "f32"},
        # Longformer-style attention, 12 heads
        {"name": "attn_12x4096", "kind": "attn", "H": 12, "S": 4096, "D": 64, "window": 256, "density": 0.05,
         "dtype": "bf16", "out": "f32"},
    ]


def _spread(rng, lo, hi, step=1):
    """A multiple of `step` in [lo, hi], spread evenly over the logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return int(min(hi, max(lo, step * max(1, round(v / step)))))


def _draw_one(rng):
    kind = rng.choice(["ffn", "ffn", "select", "preact", "microtile", "microtile", "moe", "moe", "padded", "padded", "wgrad", "attn"])
    dtype = rng.choice(["bf16", "bf16", "f16"])
    out = rng.choice(["f32", dtype])
    if kind == "ffn":
        mt = rng.choice([128, 128, 64, 32])
        live = rng.choice([1.0, rng.uniform(0.05, 0.9)])
        return {"kind": kind, "M": _spread(rng, 128, 4096, mt), "K": _spread(rng, 257, 8192), "N": _spread(rng, 128, 4096, 128),
                "mt": mt, "live": live, "run": rng.choice([32, 64, 128]), "dtype": dtype, "out": out}
    if kind == "select":
        return {"kind": kind, "M": _spread(rng, 512, 4096, 128), "K": _spread(rng, 512, 4096), "N": _spread(rng, 512, 4096, 128),
                "live": rng.uniform(0.02, 0.9), "run": rng.choice([32, 64, 128]), "dtype": dtype, "out": out}
    if kind == "preact":
        return {"kind": kind, "M": _spread(rng, 128, 4096, 128), "K": _spread(rng, 512, 8192, 8), "N": _spread(rng, 128, 2048, 128),
                "live": rng.choice([1.0, rng.uniform(0.1, 0.6)]), "dtype": dtype, "out": out}
    if kind == "microtile":
        mt = rng.choice([32, 64, 128])
        return {"kind": kind, "M": _spread(rng, 300, 4096), "K": _spread(rng, 512, 4096, mt), "N": _spread(rng, 256, 4096, 128),
                "mt": mt, "keep": math.exp(rng.uniform(math.log(0.01), math.log(0.5))), "dtype": dtype}
    if kind == "moe":
        d_model = _spread(rng, 256, 1024, 128)
        return {"kind": kind, "T": _spread(rng, 1, 8192), "d_model": d_model, "d_ff": d_model * rng.choice([2, 3, 4]),
                "E": rng.choice([8, 16, 32, 64, 128]), "gate": rng.choice([True, False]), "dtype": dtype, "out": out}
    if kind in ("padded", "wgrad"):
        max_len = _spread(rng, 48, 512)
        return {"kind": kind, "batch": _spread(rng, 1, 48), "max_len": max_len, "min_len": min(16, max_len),
                "hidden": _spread(rng, 256, 2048, 128), "N": _spread(rng, 256, 4096, 128), "dtype": dtype, "out": out}
    return {"kind": "attn", "H": rng.randint(1, 16), "S": _spread(rng, 256, 4096, 32), "D": 64,
            "window": rng.choice([64, 128, 256, 512]), "density": rng.uniform(0.0, 0.1), "dtype": dtype,
            "out": rng.choice(["f32", "bf16", "f16"])}


def draw(rng):
    most = [work(c) for c in listed()]
    max_b, max_f = max(w["bytes"] for w in most), max(w["flops"] for w in most)
    while True:
        c = _draw_one(rng)
        w = work(c)
        if w["bytes"] <= max_b and w["flops"] <= max_f:
            return c


# ------------------------------------------------------------------------------------------------ inputs
_T = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _normal(g, shape, dtype, std=1.0, mean=0.0):
    x = torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)
    return x.mul_(std).add_(mean).to(dtype)


def _live(g, k, m, run, p):
    """bool [k, m]: channel k is live for a whole run of `run` tokens with probability p."""
    if p >= 1.0:
        return torch.ones((k, m), dtype=torch.bool, device="cuda")
    nb = -(-m // run)
    return (torch.rand((k, nb), generator=g, device="cuda") < p).repeat_interleave(run, dim=1)[:, :m]


def _activation_km(g, k, m, run, p, dtype):
    """ReLU(N(-1.2, 1)) as [channels, tokens], silenced in runs: about 88 % zeros where a channel is live."""
    x = torch.randn((k, m), generator=g, device="cuda").sub_(1.2).relu_()
    return x.mul_(_live(g, k, m, run, p)).to(dtype)


def _index(nseg, cap, want_bits=False):
    z = lambda n: torch.zeros(max(n, 1), dtype=torch.int32, device="cuda")
    return pit.PitIndex(z(nseg + 1), z(cap), z(cap) if want_bits else None, nseg, cap)


def _bytes(n):
    return torch.empty(max(int(n), 256), dtype=torch.uint8, device="cuda")


def _row_mask(g, case):
    """Lengths uniform in [min_len, max_len]; uint8 [batch * max_len, 1], 1 for valid, left-aligned token rows."""
    b, n = case["batch"], case["max_len"]
    length = torch.randint(case["min_len"], n + 1, (b, 1), generator=g, device="cuda")
    return (torch.arange(n, device="cuda")[None, :] < length).to(torch.uint8).reshape(-1, 1)


def _candidates():
    """The kernels the cost model chooses from, with the costs of the committed profile of this GPU type."""
    prof = json.load(open(_PROFILE))["candidates"]
    return [{"mt_rows": 1, "mt_cols": mt, "tile_cost": prof[name]["step_ns_per_tile"],
             "fixed_cost": prof[name]["step_fixed_ns"], "dense": dense}
            for name, mt, dense in (("gather_k", 128, False), ("gather_k_64", 64, False), ("gather_k_32", 32, False),
                                    ("dense_k", 128, True))]


def prepare(case, seed):
    g = _gen(seed)
    kind, dt = case["kind"], _T[case["dtype"]]
    s = dict(case)
    if kind in ("ffn", "select", "preact"):
        M, K, N = case["M"], case["K"], case["N"]
        s["W"] = _normal(g, (K, N), dt, 0.02)
        s["C"] = torch.empty((M, N), dtype=_T[case["out"]], device="cuda")
        if kind == "preact":
            h = torch.randn((M, K), generator=g, device="cuda").sub_(1.2)
            dead = ~_live(g, K, M, 128, case["live"]).t()
            s["H"] = torch.where(dead, -h.abs() - 0.5, h).to(dt).contiguous()
            s["Xt"] = torch.empty((K, M), dtype=dt, device="cuda")
            s["ix"] = _index(M // 128, (M // 128) * K)
            s["ws"] = _bytes(pit.pit_relu_channel_major_index_workspace(M, K))
            return s
        s["Xt"] = _activation_km(g, K, M, case["run"], case["live"], dt)
        if kind == "ffn":
            mt = case["mt"]
            s["ix"] = _index(M // mt, (M // mt) * K)
            s["ws"] = _bytes(pit.pit_build_index_workspace(K, M, 1, mt, 0))
        else:
            # the caller's sparsity sample: an activation of an earlier step with the same statistics
            sample = _activation_km(g, K, M, case["run"], case["live"], dt)
            s["cands"] = _candidates()
            s["num"] = [[int(pit.pit_cover_count(sample, 1, c["mt_cols"]).item()) for c in s["cands"]]]
            s["grid"] = [[K * (M // c["mt_cols"]) for c in s["cands"]]]
            s["ws"] = _bytes(pit.pit_select_and_run_gemm_workspace(M, K))
    elif kind == "microtile":
        M, K, N, mt = case["M"], case["K"], case["N"], case["mt"]
        keep = torch.rand((M, K // mt), generator=g, device="cuda") < case["keep"]
        s["A"] = (torch.randn((M, K), generator=g, device="cuda") * keep.repeat_interleave(mt, dim=1)).to(dt)
        s["B"] = _normal(g, (K, N), dt)
        s["C"] = torch.empty((M, N), dtype=torch.float32, device="cuda")
        s["ix"] = _index(K // mt, (K // mt) * M)
        s["ws"] = _bytes(pit.pit_build_index_workspace(M, K, 1, mt, 0))
    elif kind == "moe":
        T, d, f, E = case["T"], case["d_model"], case["d_ff"], case["E"]
        p = torch.arange(1, E + 1, device="cuda", dtype=torch.float32).pow(-1.1)       # Zipf popularity of the experts
        rank = torch.multinomial(p / p.sum(), T, replacement=True, generator=g)
        s["eid"] = torch.randperm(E, generator=g, device="cuda")[rank].to(torch.int32)
        s["gate_w"] = 0.5 + 0.5 * torch.rand(T, generator=g, device="cuda") if case["gate"] else None
        s["X"] = _normal(g, (T, d), dt)
        s["W1"], s["W2"] = _normal(g, (E, d, f), dt, 0.02), _normal(g, (E, f, d), dt, 0.02)
        s["status"] = torch.zeros(1, dtype=torch.int32, device="cuda")
        s["Y"] = torch.empty((T, d), dtype=_T[case["out"]], device="cuda")
        s["ws"] = _bytes(pit.pit_moe_workspace(T, d, f, E))
    elif kind in ("padded", "wgrad"):
        rows, h, N = case["batch"] * case["max_len"], case["hidden"], case["N"]
        s["mask"] = _row_mask(g, case)
        if kind == "padded":
            s["X"] = _normal(g, (rows, h), dt)                    # padding rows hold whatever was there
            s["W"] = _normal(g, (h, N), dt, 0.02)
            s["Y"] = torch.empty((rows, N), dtype=_T[case["out"]], device="cuda")
            s["ix"] = _index(1, rows)
            s["ws"] = _bytes(pit.pit_build_index_workspace(rows, 1, 1, 1, 0))
        else:
            s["X"] = _normal(g, (rows, h), dt) * s["mask"].to(dt)  # saved activations, zero in the padding
            s["dY"] = _normal(g, (rows, N), dt, 0.02) * s["mask"].to(dt)
            s["dW"] = torch.empty((h, N), dtype=_T[case["out"]], device="cuda")
            s["ix"] = _index(h // 128, (h // 128) * rows)
            s["ws"] = _bytes(pit.pit_build_index_workspace(rows, h, 1, 128, 0))
    else:
        H, S, D = case["H"], case["S"], case["D"]
        s["Q"], s["Kt"], s["V"] = (_normal(g, (H, S, D), dt) for _ in range(3))
        i = torch.arange(S, device="cuda")
        band = (i[:, None] - i[None, :]).abs() <= case["window"] // 2
        cols = torch.rand((S // 32, S), generator=g, device="cuda") < case["density"]
        s["mask"] = (band | cols.repeat_interleave(32, dim=0)).to(torch.uint8)
        s["O"] = torch.empty((H, S, D), dtype=_T[case["out"]], device="cuda")
        s["ws"] = _bytes(pit.pit_sparse_attn_workspace(H, S, D))
    return s


# ------------------------------------------------------------------------------------------------ one pass
def run(s):
    kind = s["kind"]
    if kind == "ffn":
        pit.pit_build_index(s["Xt"], 1, s["mt"], 0, out=s["ix"], ws=s["ws"])
        pit.pit_sread_gemm(pit.PIT_GEMM_GATHER_K, s["Xt"], s["W"], s["ix"], s["mt"], s["M"], s["N"], s["K"], out=s["C"])
        return s["C"], s["ix"].seg_ptr, s["ix"].idx
    if kind == "select":
        # (which kernel the costs pick is a matter of the profile, not a result)
        pit.pit_select_and_run_gemm(s["cands"], s["num"], s["grid"], s["Xt"], s["W"], s["M"], s["N"], s["K"], out=s["C"], ws=s["ws"])
        return s["C"]
    if kind == "preact":
        pit.pit_relu_channel_major_index(s["H"], out_xt=s["Xt"], out=s["ix"], ws=s["ws"])
        pit.pit_sread_gemm(pit.PIT_GEMM_GATHER_K, s["Xt"], s["W"], s["ix"], 128, s["M"], s["N"], s["K"], out=s["C"])
        return s["C"], s["Xt"], s["ix"].seg_ptr, s["ix"].idx
    if kind == "microtile":
        pit.pit_build_index(s["A"], 1, s["mt"], 0, out=s["ix"], ws=s["ws"])
        pit.pit_sread_gemm(pit.PIT_GEMM_GATHER_M, s["A"], s["B"], s["ix"], s["mt"], s["M"], s["N"], s["K"], out=s["C"])
        return s["C"], s["ix"].seg_ptr, s["ix"].idx
    if kind == "moe":
        pit.pit_moe_dispatch_gemm(s["X"], s["eid"], s["gate_w"], s["W1"], s["W2"], out=s["Y"], status=s["status"], ws=s["ws"])
        return s["Y"], s["status"]
    if kind == "padded":
        rows = s["batch"] * s["max_len"]
        pit.pit_build_index(s["mask"], 1, 1, 0, out=s["ix"], ws=s["ws"])
        pit.pit_sread_gemm(pit.PIT_GEMM_GATHER_M, s["X"], s["W"], s["ix"], s["hidden"], rows, s["N"], s["hidden"], out=s["Y"])
        return s["Y"], s["ix"].seg_ptr, s["ix"].idx
    if kind == "wgrad":
        rows = s["batch"] * s["max_len"]
        pit.pit_build_index(s["X"], 1, 128, 0, out=s["ix"], ws=s["ws"])
        pit.pit_sread_gemm(pit.PIT_GEMM_GATHER_K, s["X"], s["dY"], s["ix"], 128, s["hidden"], s["N"], rows, out=s["dW"])
        return s["dW"], s["ix"].seg_ptr, s["ix"].idx
    return pit.pit_sparse_attn(s["Q"], s["Kt"], s["V"], s["mask"], 1.0 / math.sqrt(s["D"]), out=s["O"], ws=s["ws"])


# ------------------------------------------------------------------------------------------------ work
def _cover(live, run, mt):
    """Expected share of 1 x mt micro-tiles with a live token (a run or more of tokens is live as a whole)."""
    return 1.0 - (1.0 - live) ** max(1.0, mt / run)


def _experts_hit(T, E):
    w = [r ** -1.1 for r in range(1, E + 1)]
    t = sum(w)
    return sum(1.0 - (1.0 - x / t) ** T for x in w)


def work(case):
    """Expected bytes (each input read once, each output written once) and operations of one pass: the operands of
    micro-tiles that are all zero need not be multiplied, and rows of B that no list names need not be read."""
    kind = case["kind"]
    ob = 4 if case.get("out", "f32") == "f32" else 2
    if kind in ("ffn", "select", "preact"):
        M, K, N = case["M"], case["K"], case["N"]
        c = _cover(case["live"], case.get("run", 128), 32)        # non-zero 32 x 1 micro-tiles (the finest the kernels take)
        used = 1.0 - (1.0 - case["live"]) ** max(1.0, M / case.get("run", 128))
        b = 2.0 * M * K + 2.0 * used * K * N + ob * M * N + (2.0 * M * K if kind == "preact" else 0.0)
        b += 4.0 * _cover(case["live"], case.get("run", 128), 128) * K * M / case.get("mt", 128)
        return {"bytes": b, "flops": 2.0 * M * K * N * c}
    if kind == "microtile":
        M, K, N = case["M"], case["K"], case["N"]
        return {"bytes": 2.0 * M * K + 2.0 * K * N + 4.0 * M * N + 4.0 * case["keep"] * M * K / case["mt"],
                "flops": 2.0 * M * K * N * case["keep"]}
    if kind == "moe":
        T, d, f, E = case["T"], case["d_model"], case["d_ff"], case["E"]
        return {"bytes": 4.0 * _experts_hit(T, E) * d * f + 2.0 * T * d + ob * T * d + 8.0 * T, "flops": 4.0 * T * d * f}
    if kind in ("padded", "wgrad"):
        rows, h, N = case["batch"] * case["max_len"], case["hidden"], case["N"]
        valid = case["batch"] * (case["min_len"] + case["max_len"]) / 2.0
        if kind == "padded":
            return {"bytes": rows + 4.0 * valid + 2.0 * valid * h + 2.0 * h * N + ob * rows * N, "flops": 2.0 * valid * h * N}
        return {"bytes": 2.0 * rows * h + 2.0 * valid * N + ob * h * N + 4.0 * valid * h / 128, "flops": 2.0 * valid * h * N}
    H, S, D = case["H"], case["S"], case["D"]
    keys = min(S, case["window"] + 32) + case["density"] * max(0, S - case["window"] - 32)   # per block of 32 queries
    return {"bytes": S * S + 6.0 * H * S * D + ob * H * S * D, "flops": 4.0 * H * S * keys * D}


# ------------------------------------------------------------------------------------------------ tolerance
def tolerance(case):
    """About four times the difference measured between a pass and the same pass in 64 bits (rounded to the output
    type where that is 16 bits wide, so that what is left there are roundings that fall to the other side: one unit
    in the last place at most, 2^-7 of a value in bf16 and 2^-10 in fp16)."""
    kind, dtype, out = case["kind"], case["dtype"], case.get("out", "f32")
    if kind == "attn":       # probabilities enter the second product with 17 bits (bf16 inputs) or 11 bits (fp16 inputs)
        return {("bf16", "f32"): {"rel": 8e-6, "max": 6e-5}, ("bf16", "bf16"): {"rel": 3e-4, "max": 8e-3},
                ("bf16", "f16"): {"rel": 1.2e-4, "max": 1e-3}, ("f16", "f32"): {"rel": 6e-4, "max": 4e-3},
                ("f16", "bf16"): {"rel": 3e-3, "max": 1.6e-2}, ("f16", "f16"): {"rel": 1.1e-3, "max": 5e-3}}[dtype, out]
    if kind == "moe":        # the hidden row is rounded to the input type between the two products
        if out == "f32":
            return {"rel": 1.5e-4, "max": 7e-3} if dtype == "bf16" else {"rel": 8e-5, "max": 8e-4}
        return {"rel": 9e-4, "max": 1.6e-2} if out == "bf16" else {"rel": 2.6e-4, "max": 2e-3}
    if out == "bf16":
        return {"rel": 1.2e-4, "max": 8e-3}
    if out == "f16":
        return {"rel": 3e-5, "max": 1e-3}
    return {"rel": 1.2e-6, "max": 1.2e-5}
