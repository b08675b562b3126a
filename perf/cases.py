"""The work that a program built on this library has it do, as timed cases.

A case is one pass of one of three programs, all through the public entry points:

``layer``
    one GPU's MoE layer: gating, address resolution, expert FFN, combine.  With ``gather`` the gate/up
    projection fetches its rows from ``x`` itself (a device that computes every expert needs no send buffer),
    without it the rows are moved into expert order first.
``ep_dispatch``
    the token side of one expert-parallel rank: gating, the per-destination send layout and send buffer, and
    the combine of the rows that come back from the other ranks.
``ep_experts``
    the expert side of such a rank: the FFN of its local experts over a received buffer.

Sizes are those of the workload table in ``moe_inputs`` and of the token sweep of ``bench.py``; drawn cases
spread over the token counts between the smallest and the largest call and over generic shapes.
"""
import math

import numpy as np
import torch

import paper_2605_05888_amd as hub

# hidden size, experts, top-K, expert FFN size, score mode, Zipf exponent of the experts' popularity (0: uniform)
SHAPES = {
    "tiny": (128, 8, 2, 256, "softmax", 0.0),
    "mixtral": (4096, 8, 2, 14336, "softmax", 0.0),
    "gptoss": (2880, 128, 4, 2880, "softmax", 1.0),
    "dsv3": (7168, 256, 8, 2048, "sigmoid", 0.0),
    "dsv3_ep": (7168, 256, 8, 2048, "sigmoid", 1.2),
    "qwen2moe": (2048, 64, 4, 1408, "softmax", 0.0),
    "phi35moe": (4096, 16, 2, 6400, "softmax", 0.0),
}
EP_RANKS = 32


def _layer(shape, N, gather, dtype="bf16"):
    H, E, K, F, score, zipf = SHAPES[shape]
    return {"kind": "layer", "N": N, "H": H, "E": E, "K": K, "F": F, "score": score, "zipf": zipf,
            "gather": gather, "dtype": dtype}


def _ep_dispatch(N):
    H, E, K, F, score, zipf = SHAPES["dsv3_ep"]
    return {"kind": "ep_dispatch", "N": N, "H": H, "E": E, "K": K, "G": EP_RANKS, "score": score, "zipf": zipf,
            "dtype": "bf16"}


def _ep_experts(M):
    H, E, K, F, score, zipf = SHAPES["dsv3_ep"]
    return {"kind": "ep_experts", "M": M, "H": H, "E": E // EP_RANKS, "F": F, "zipf": zipf, "dtype": "bf16"}


def listed():
    return [
        # one sequence being decoded: a single token, launches and latency
        dict(_layer("qwen2moe", 1, True), name="decode_one_token"),
        # a small decoding batch: most experts see one row or none, the weights stream once
        dict(_layer("gptoss", 37, True), name="decode_batch_37"),
        # a larger decoding batch on few large experts (smallest point of the token sweep)
        dict(_layer("mixtral", 128, False), name="decode_batch_128"),
        # an odd-sized chunk of a chunked prefill
        dict(_layer("phi35moe", 1155, False), name="prefill_chunk_1155"),
        # ordinary prefills: many small experts, few large ones, skewed popularity
        dict(_layer("qwen2moe", 8192, False), name="prefill_small_experts"),
        dict(_layer("mixtral", 4096, False), name="prefill_large_experts"),
        dict(_layer("gptoss", 8192, True), name="prefill_skewed"),
        # the largest call: 16384 tokens over 256 experts on one GPU
        dict(_layer("dsv3", 16384, False), name="prefill_256_experts"),
        # an expert-parallel rank: what it does for its own tokens, and for the rows it receives
        dict(_ep_dispatch(8192), name="ep_dispatch_combine"),
        dict(_ep_experts(65536), name="ep_expert_ffn"),
        # single precision: the smallest model, and an odd-sized one
        dict(_layer("tiny", 256, False, "fp32"), name="fp32_tiny"),
        {"kind": "layer", "N": 1001, "H": 516, "E": 12, "K": 3, "F": 1028, "score": "softmax", "zipf": 0.0,
         "gather": False, "dtype": "fp32", "name": "fp32_odd"},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["layer", "layer", "layer", "generic", "generic", "ep_dispatch", "ep_experts", "fp32"])
    if kind == "ep_dispatch":
        return _ep_dispatch(_log_int(rng, 8, 8192))
    if kind == "ep_experts":
        return _ep_experts(_log_int(rng, 16, 65536))
    if kind == "fp32":
        E = rng.randint(2, 32)
        return {"kind": "layer", "N": _log_int(rng, 16, 1024), "H": 4 * _log_int(rng, 16, 160), "E": E,
                "K": rng.randint(1, min(E, 4)), "F": 4 * _log_int(rng, 16, 260), "score": rng.choice(["softmax", "sigmoid"]),
                "zipf": rng.choice([0.0, 1.0]), "gather": rng.random() < 0.5, "dtype": "fp32"}
    if kind == "generic":
        E = _log_int(rng, 4, 128)
        return {"kind": "layer", "N": _log_int(rng, 1, 8192), "H": 64 * _log_int(rng, 8, 64), "E": E,
                "K": rng.randint(1, min(E, 8)), "F": 64 * _log_int(rng, 4, 100), "score": rng.choice(["softmax", "sigmoid"]),
                "zipf": rng.choice([0.0, 0.0, 1.0]), "gather": rng.random() < 0.5, "dtype": "bf16"}
    shape = rng.choice(["mixtral", "gptoss", "dsv3", "qwen2moe", "phi35moe"])
    return _layer(shape, _log_int(rng, 1, 16384), rng.random() < 0.5)


def _popularity(E, zipf):
    p = np.arange(1, E + 1, dtype=np.float64) ** -zipf
    return p / p.sum()


def _bias(E, zipf):
    """Router bias whose logits make the experts' popularity follow Zipf's law: log-popularity at Gumbel scale."""
    p = _popularity(E, zipf)
    return math.sqrt(6.0) / math.pi * np.log(p / p.max())


def _touched(case):
    """Expected number of experts that get at least one row."""
    E = case["E"]
    if case["kind"] == "ep_experts":
        return float(np.sum(1.0 - (1.0 - _popularity(E, case["zipf"])) ** case["M"]))
    share = np.full(E, case["K"] / E)
    if case["zipf"]:
        tokens = 4096
        z = np.random.default_rng(0).standard_normal((tokens, E)) + _bias(E, case["zipf"])
        top = np.argpartition(-z, case["K"] - 1, axis=1)[:, :case["K"]]
        share = np.bincount(top.ravel(), minlength=E) / tokens
    return float(np.sum(1.0 - (1.0 - share) ** case["N"]))


def _normal(g, shape, std, dtype):
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, std, generator=g)


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    rng = np.random.default_rng(seed)
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    code = hub.BF16 if case["dtype"] == "bf16" else hub.F32
    H, E = case["H"], case["E"]
    i32 = lambda n: torch.empty(n, dtype=torch.int32, device="cuda")
    raw = lambda n: torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")
    s = {"case": case, "code": code}
    if case["kind"] != "ep_dispatch":
        F = case["F"]
        s["W_gate"] = _normal(g, (E, F, H), H ** -0.5, dt)
        s["W_up"] = _normal(g, (E, F, H), H ** -0.5, dt)
        s["W_down"] = _normal(g, (E, H, F), F ** -0.5, dt)
    if case["kind"] == "ep_experts":
        M = case["M"]
        counts = rng.multinomial(M, rng.permutation(_popularity(E, case["zipf"])))
        s["seg"] = torch.tensor(np.concatenate([[0], np.cumsum(counts)]), dtype=torch.int32, device="cuda")
        s["xp"] = _normal(g, (M, H), 1.0, dt)
        s["y"] = torch.empty((M, H), dtype=dt, device="cuda")
        s["ws"] = raw(hub.workspace_bytes(hub.OP_GROUPED_FFN, N=M, H=H, E=E, F=case["F"], dtype=code))
        return s
    N, K, G = case["N"], case["K"], case.get("G", 1)
    R = N * K
    s["x"] = _normal(g, (N, H), 1.0, dt)
    s["W_r"] = _normal(g, (H, E), H ** -0.5, torch.float32)
    s["bias"] = None
    if case["zipf"] > 0.0:
        s["bias"] = torch.tensor(rng.permutation(_bias(E, case["zipf"])), dtype=torch.float32, device="cuda")
    s["score"] = hub.SCORE_SIGMOID_TOPK if case["score"] == "sigmoid" else hub.SCORE_SOFTMAX_TOPK
    s["topk_idx"] = i32(R).view(N, K)
    s["topk_w"] = torch.empty((N, K), dtype=torch.float32, device="cuda")
    s["layout"] = (i32(E), i32(E + 1), i32(G), i32(G + 1), i32(R), i32(R))
    s["ws_route"] = raw(hub.workspace_bytes(hub.OP_ROUTE, N=N, E=E))
    s["ws_layout"] = raw(hub.workspace_bytes(hub.OP_DISPATCH_LAYOUT, N=N, E=E, K=K, G=G))
    s["out"] = torch.empty((N, H), dtype=dt, device="cuda")
    if not case.get("gather"):
        s["xp"] = torch.empty((R, H), dtype=dt, device="cuda")
    if case["kind"] == "ep_dispatch":
        s["y"] = _normal(g, (R, H), 1.0, dt) # the rows that the other ranks send back
    else:
        s["y"] = torch.empty((R, H), dtype=dt, device="cuda")
        s["ws"] = raw(hub.workspace_bytes(hub.OP_GROUPED_FFN, N=R, H=H, E=E, F=case["F"], dtype=code))
    return s


def run(s):
    case = s["case"]
    if case["kind"] == "ep_experts":
        hub.moe_grouped_ffn(s["xp"], s["seg"], s["W_gate"], s["W_up"], s["W_down"], s["y"], s["ws"])
        return s["y"]
    K, E, G = case["K"], case["E"], case.get("G", 1)
    hub.moe_route(s["x"], s["W_r"], s["bias"], K, s["score"], s["topk_idx"], s["topk_w"], ws=s["ws_route"])
    hub.moe_dispatch_layout(s["topk_idx"], E, G, *s["layout"], s["ws_layout"])
    counts, offsets, dest_counts, dest_offsets, slot_of_row, row_of_slot = s["layout"]
    if case.get("gather"):
        R, H, F = case["N"] * K, case["H"], case["F"]
        hub.moe_ffn_schedule(s["code"], R, H, F, offsets, s["ws"])
        hub.moe_ffn_gate_up_gather(s["x"], K, offsets, row_of_slot, s["W_gate"], s["W_up"], s["ws"])
        hub.moe_ffn_down(offsets, s["W_down"], s["y"], s["ws"])
    else:
        hub.moe_permute(s["x"], K, slot_of_row, row_of_slot, s["xp"])
        if case["kind"] == "layer":
            hub.moe_grouped_ffn(s["xp"], offsets, s["W_gate"], s["W_up"], s["W_down"], s["y"], s["ws"])
    hub.moe_combine(s["y"], K, slot_of_row, s["topk_w"], s["out"])
    result = {"out": s["out"], "topk_idx": s["topk_idx"], "topk_w": s["topk_w"]}
    if case["kind"] == "ep_dispatch":
        result.update(send=s["xp"], expert_counts=counts, expert_offsets=offsets, dest_counts=dest_counts,
                      dest_offsets=dest_offsets, slot_of_row=slot_of_row, row_of_slot=row_of_slot)
    return result


def work(case):
    b = 2 if case["dtype"] == "bf16" else 4
    H, E = case["H"], case["E"]
    nbytes = flops = 0
    if case["kind"] == "ep_experts":
        rows = case["M"]
        nbytes += 2 * rows * H * b
    else:
        N, K = case["N"], case["K"]
        rows = N * K
        nbytes += 2 * N * H * b + 4 * H * E + 8 * N * K # x, out, router weights, top-K
        flops += 2 * N * H * E
    if case["kind"] == "ep_dispatch":
        nbytes += 2 * rows * H * b + 8 * rows # send buffer, returned rows, the two slot maps
        flops += 2 * rows * H
    else:
        # the weights of the experts that get a row, once
        nbytes += _touched(case) * 3 * H * case["F"] * b
        flops += 6 * rows * H * case["F"]
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # bf16: a and y are rounded on the way, against the same path in 64 bits the output is off by 3e-3;
    # fp32: sums of up to some thousand products
    return {"rel": 1e-2} if case["dtype"] == "bf16" else {"rel": 5e-6}
