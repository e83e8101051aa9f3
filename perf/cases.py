"""What a program that runs a table-lookup model through this package does, as cases to be timed.

Five kinds of work, each through the public entry points:

* ``call``     one linear layer for 1..16 tokens, called eagerly (``lcd_lut_gemv`` / ``lcd_lut_gemv_q8``);
* ``step``     one decode step of a stack of decoder blocks, 1..16 tokens: the layers that read one input
               go out as one grouped call (q, k, v | o | gate, up | down), the calls of the step captured
               once in a HIP graph and replayed, as a serving loop does;
* ``prefill``  the linear layers of one decoder block, 17 tokens and more, four grouped calls in the
               order of the block, launched eagerly (the token count changes from prompt to prompt);
* ``gemm``     one linear layer for 17 tokens and more (``lcd_lut_gemm`` / ``lcd_lut_gemm_q8``);
* ``offline``  one round of the clustering side on one layer: nearest centroids of the weights, cluster
               sizes, merge of the two closest centroids, packing of the new indices.

Weights are made as a model's would be: fp16 weights N(0, 0.02 * row factor), a codebook per row at the
mid-percentiles of that distribution, indices from ``lcd_assign_indices``.  Activations are N(0, 1) with
1 % of the channels times 50, the smoothing factor is the root of a calibration batch's channel maxima,
and the INT8 step puts the 99th percentile of |x / s| at code 127.
"""
from __future__ import annotations

import math
from statistics import NormalDist

import torch

import paper_2506_12038_amd as lcd
from paper_2506_12038_amd.binding import GemmGroup, GemvGroup

# index widths of a block whose layers have centroid counts of their own: q, k, v, o, gate, up, down
MIXED_BITS = (3, 3, 2, 4, 2, 3, 4)
SIGMA = 0.02


def listed():
    return [
        # the smallest call: one 4096 x 4096 layer, one token (launch latency)
        {"name": "call_4096x4096_2b_m1", "kind": "call", "bits": 2, "M": 1, "N": 4096, "K": 4096, "q8": False},
        # a long-K layer called on its own for an odd number of sequences
        {"name": "call_4096x11008_3b_m3", "kind": "call", "bits": 3, "M": 3, "N": 4096, "K": 11008, "q8": False},
        # single-stream decoding of a LLaMA-7B-shaped model, 3 bits (8 of its blocks)
        {"name": "step_7b_3b_m1", "kind": "step", "bits": 3, "M": 1, "H": 4096, "F": 11008, "attn": True, "blocks": 8, "q8": False},
        # single-stream decoding through the MLP of a LLaMA-70B-shaped model, 2 bits (3 blocks)
        {"name": "step_70b_mlp_2b_m1", "kind": "step", "bits": 2, "M": 1, "H": 8192, "F": 28672, "attn": False, "blocks": 3, "q8": False},
        # the same decoder for a full batch of 16 sequences
        {"name": "step_7b_2b_m16", "kind": "step", "bits": 2, "M": 16, "H": 4096, "F": 11008, "attn": True, "blocks": 8, "q8": False},
        # a few sequences with INT8 activations (the paper's own input transformation)
        {"name": "step_7b_2b_q8_m4", "kind": "step", "bits": 2, "M": 4, "H": 4096, "F": 11008, "attn": True, "blocks": 8, "q8": True},
        # layers of different index widths (2, 3 and 4 bits), a handful of sequences
        {"name": "step_5120_mixed_m6", "kind": "step", "bits": "mixed", "M": 6, "H": 5120, "F": 13824, "attn": True, "blocks": 4, "q8": False},
        # a short prompt, or a batch just too large for the decode entry points
        {"name": "prefill_7b_3b_m40", "kind": "prefill", "bits": 3, "M": 40, "H": 4096, "F": 11008, "q8": False},
        # one wide layer with 16 centroids, about a hundred tokens
        {"name": "gemm_11008x4096_4b_m100", "kind": "gemm", "bits": 4, "M": 100, "N": 11008, "K": 4096, "q8": False},
        # a prompt of ordinary, ragged length with INT8 activations
        {"name": "prefill_7b_2b_q8_m333", "kind": "prefill", "bits": 2, "M": 333, "H": 4096, "F": 11008, "q8": True},
        # a long prompt
        {"name": "prefill_7b_3b_m2048", "kind": "prefill", "bits": 3, "M": 2048, "H": 4096, "F": 11008, "q8": False},
        # making a layer: one round of clustering and packing
        {"name": "offline_11008x4096_3b", "kind": "offline", "bits": 3, "N": 11008, "K": 4096, "ncent": 8},
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _size(rng, lo, hi, step):
    return max(lo, min(hi, int(round(_log_uniform(rng, lo, hi) / step)) * step))


def draw(rng):
    kind = rng.choice(["call", "step", "step", "step", "prefill", "prefill", "prefill", "gemm", "offline"])
    bits = rng.choice([2, 3, 3, 4])
    q8 = rng.random() < 0.3
    if kind == "offline":
        ncent = rng.randint(3 if bits == 2 else (1 << (bits - 1)) + 1, 1 << bits)
        return {"kind": kind, "bits": bits, "N": _size(rng, 1024, 16384, 16), "K": _size(rng, 1024, 8192, 256), "ncent": ncent}
    if kind == "call":
        return {"kind": kind, "bits": bits, "M": rng.randint(1, 16), "N": _size(rng, 1024, 28672, 16),
                "K": _size(rng, 1024, 16384, 256), "q8": q8}
    if kind == "gemm":
        return {"kind": kind, "bits": bits, "M": int(_log_uniform(rng, 17, 1024)), "N": _size(rng, 1024, 16384, 16),
                "K": _size(rng, 1024, 11008, 256), "q8": q8}
    H = _size(rng, 2048, 8192, 256)
    F = max(H, int(H * rng.uniform(2.0, 4.0)) // 256 * 256)
    if kind == "step":
        attn = rng.random() < 0.7
        if attn and not q8 and rng.random() < 0.2:
            bits = "mixed"
        M = rng.choice([1, 1, 1, 2, 3, 4, rng.randint(5, 16), rng.randint(5, 16), 16])
        block = (4 * H * H if attn else 0) + 3 * H * F
        blocks = max(1, min(8, int(6e8 / (block * (3 if bits == "mixed" else bits) / 8))))
        return {"kind": kind, "bits": bits, "M": M, "H": H, "F": F, "attn": attn, "blocks": blocks, "q8": q8}
    most = 2048 * (4 * 4096 * 4096 + 3 * 4096 * 11008)             # the listed long prompt's products
    M = int(_log_uniform(rng, 17, 2048))
    M = max(17, min(M, most // (4 * H * H + 3 * H * F)))
    return {"kind": kind, "bits": bits, "M": M, "H": H, "F": F, "q8": q8}


def _stages(case):
    """(K, [N of every layer that reads this input]) in the order of a decoder block."""
    H, F = case["H"], case["F"]
    mlp = [(H, [F, F]), (F, [H])]
    return ([(H, [H, H, H]), (H, [H])] if case.get("attn", True) else []) + mlp


def _stage_bits(case):
    """Index width of every layer, stage by stage."""
    out, at = [], 0
    for _, ns in _stages(case):
        out.append([MIXED_BITS[(at + i) % 7] if case["bits"] == "mixed" else case["bits"] for i in range(len(ns))])
        at += len(ns)
    return out


def _layers(case):
    """(N, K, bits) of every layer of one pass."""
    if "N" in case:
        return [(case["N"], case["K"], case["bits"])]
    return [(N, K, b) for (K, ns), bs in zip(_stages(case), _stage_bits(case)) for N, b in zip(ns, bs)] * case.get("blocks", 1)


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _weights(N, K, bits, ncent, g):
    """fp16 weights and the ascending codebook of every row (unused entries zero)."""
    row = 1.0 + 0.25 * (2.0 * torch.rand((N, 1), device="cuda", generator=g) - 1.0)
    w = torch.randn((N, K), device="cuda", generator=g, dtype=torch.float16).mul_((SIGMA * row).half())
    z = torch.tensor([NormalDist().inv_cdf((2 * i + 1) / (2 * ncent)) for i in range(ncent)], device="cuda")
    codebook = torch.zeros((N, 1 << bits), dtype=torch.float16, device="cuda")
    codebook[:, :ncent] = (SIGMA * row * z).half()
    return w, codebook


def _layer(N, K, bits, g):
    """What a program keeps of a layer: packed indices and the table."""
    w, codebook = _weights(N, K, bits, 1 << bits, g)
    idx = lcd.lcd_assign_indices(w, codebook, 1 << bits, bits)
    return lcd.lcd_pack_indices(idx, bits), lcd.lcd_build_lut(codebook, bits)


def _input(M, K, g):
    """Activations, the smoothing factor of their channels and the INT8 step."""
    scale = torch.where(torch.rand((K,), device="cuda", generator=g) < 0.01, 50.0, 1.0)
    x = (torch.randn((M, K), device="cuda", generator=g) * scale).half()
    calibration = torch.randn((64, K), device="cuda", generator=g) * scale
    s = calibration.abs().amax(dim=0).sqrt().clamp_(min=1e-5)
    s_q = float(torch.quantile((calibration / s).abs().flatten(), 0.99)) / 127.0
    return x, s, s_q


def prepare(case, seed):
    g = _generator(seed)
    kind = case["kind"]
    if kind == "offline":
        w, codebook = _weights(case["N"], case["K"], case["bits"], case["ncent"], g)
        return {"case": case, "w": w, "codebook": codebook}
    M = case["M"]
    if kind in ("call", "gemm"):
        N, K, bits = case["N"], case["K"], case["bits"]
        packed, lut = _layer(N, K, bits, g)
        x, s, s_q = _input(M, K, g)
        return {"case": case, "packed": packed, "lut": lut, "x": x, "s": s, "s_q": s_q,
                "y": torch.empty((M, N), dtype=torch.float16, device="cuda"),
                "workspace": torch.empty(lcd.lcd_workspace_bytes(M, N, K, bits), dtype=torch.uint8, device="cuda")}
    groups, outputs = [], []
    for _ in range(case.get("blocks", 1)):
        for (K, ns), bs in zip(_stages(case), _stage_bits(case)):
            x, s, s_q = _input(M, K, g)
            problems = []
            for N, b in zip(ns, bs):
                y = torch.empty((M, N), dtype=torch.float16, device="cuda")
                problems.append((*_layer(N, K, b, g), x, s, y, N))
                outputs.append(y)
            steps = [s_q] * len(ns) if case["q8"] else None
            if kind == "step":
                groups.append(GemvGroup(problems, bs if len(set(bs)) > 1 else bs[0], s_q=steps))
            else:
                groups.append(GemmGroup(problems, bs[0], s_q=steps))
    # the calls follow one another on one stream: they share the largest call's workspace
    workspace = max((p.workspace for p in groups), key=lambda t: t.numel())
    for p in groups:
        p.workspace = workspace
    state = {"case": case, "groups": groups, "outputs": outputs}
    if kind == "step":
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            for p in groups:                # once outside the capture
                p()
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            for p in groups:
                p()
        state["graph"] = graph
    return state


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "step":
        state["graph"].replay()
        return state["outputs"]
    if kind == "prefill":
        for p in state["groups"]:
            p()
        return state["outputs"]
    if kind == "offline":
        bits, ncent = case["bits"], case["ncent"]
        idx = lcd.lcd_assign_indices(state["w"], state["codebook"], ncent, bits)
        counts = lcd.lcd_cluster_counts(idx, bits)
        codebook, merged_idx, merged = lcd.lcd_merge_closest(state["codebook"], counts, idx, ncent, bits)
        packed = lcd.lcd_pack_indices(merged_idx, bits)
        return {"idx": idx, "counts": counts, "codebook": codebook, "merged_idx": merged_idx, "merged": merged, "packed": packed}
    entry = {("call", False): lcd.lcd_lut_gemv, ("gemm", False): lcd.lcd_lut_gemm,
             ("call", True): lcd.lcd_lut_gemv_q8, ("gemm", True): lcd.lcd_lut_gemm_q8}[kind, case["q8"]]
    step = (state["s_q"],) if case["q8"] else ()
    return entry(state["packed"], state["lut"], state["x"], state["s"], *step, case["N"], case["bits"],
                 y=state["y"], workspace=state["workspace"])


def work(case):
    if case["kind"] == "offline":
        N, K, slots = case["N"], case["K"], 1 << case["bits"]
        # read: weights, codebook; written: both index matrices, sizes, new codebook, merged pair, packed indices
        return {"bytes": N * K * (2 + 1 + 1) + N * K * case["bits"] // 8 + N * slots * (2 + 4 + 2) + N, "flops": 0}
    M, total, flops = case["M"], 0, 0
    for N, K, bits in _layers(case):
        total += N * K * bits // 8 + N * (1 << bits) * 2 + M * N * 2      # indices, centroids, outputs
        flops += 2 * M * N * K
    inputs = [case["K"]] if "N" in case else [K for K, _ in _stages(case)] * case.get("blocks", 1)
    return {"bytes": total + sum(K * (2 * M + 4) for K in inputs), "flops": flops}


def tolerance(case):
    if case["kind"] == "offline":
        return "exact"
    # measured against the same product in 64 bits: rel 3.0e-4, max 1.35e-3 (fp16 activations: x / s and the
    # output are each rounded to fp16), rel 2.1e-4, max 4.9e-4 (INT8 codes: only the output is rounded)
    return {"rel": 8e-4, "max": 2e-3} if case["q8"] else {"rel": 1.2e-3, "max": 5e-3}
