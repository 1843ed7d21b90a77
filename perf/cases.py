"""The work that users of this library have one GPU do, as measurable cases.

A case is a plain dict that describes one MoE-layer share and one batch.
`prepare` puts on the GPU what a serving program has in hand before a step (the
layer with its weights and buffers, the token rows), `run` takes one step
through the public entry points and returns what the step computes.  Two paths
are covered: the whole layer share (`MoELayerShare.forward`: route, dispatch,
expert FFN, combine) and the two sides of the fused TP-EP schedules
(`moe_dispatch_shard` before the exchange, `moe_combine_stage` after it).

The shapes are those of `workloads/gen.py`: the tiny fp32 layer, the
Qwen3-30B-A3B layer, the Qwen3-235B-A22B EP share and the DeepSeek-R1 TP x EP
share, each over the token counts between one decoded token and the largest
prefill step, with the TP degrees, weight types and gate options they are
served with.
"""
import math

import torch

import paper_2601_08800_amd as moe
from paper_2601_08800_amd.layer import MoELayerShare, config_from_workload
from workloads.gen import Workload

FP8_BLOCK = 128
E4M3_MAX = 448.0

# One layer of each model: sizes, gate, and how the share is cut (ep = number of
# expert ranges, tp = slices of the intermediate size).
TINY = dict(hidden=256, experts=8, top_k=2, inter=512, score="softmax", groups=1, kept_groups=1,
            scale=1.0, bias="none", ep=1, ep_rank=0, tp=1, act="f32", weights="f32",
            fp8_acts=False, shared=False, zipf=0.0)
QWEN30 = dict(hidden=2048, experts=128, top_k=8, inter=768, score="softmax", groups=1, kept_groups=1,
              scale=1.0, bias="none", ep=1, ep_rank=0, tp=1, act="bf16", weights="bf16",
              fp8_acts=False, shared=False, zipf=0.0)
QWEN235 = dict(hidden=4096, experts=128, top_k=8, inter=1536, score="softmax", groups=1, kept_groups=1,
               scale=1.0, bias="logit", ep=8, ep_rank=0, tp=1, act="bf16", weights="bf16",
               fp8_acts=False, shared=False, zipf=0.0)
DEEPSEEK = dict(hidden=7168, experts=256, top_k=8, inter=2048, score="sigmoid", groups=8, kept_groups=4,
                scale=2.5, bias="select", ep=8, ep_rank=0, tp=2, act="bf16", weights="bf16",
                fp8_acts=False, shared=True, zipf=0.0)


def _layer(model, tokens, **changes):
    c = dict(model, path="layer", tokens=tokens, nodes=1)
    c.update(changes)
    return c


def _staged(model, tokens, nodes, tp, **changes):
    c = dict(model, path="staged", tokens=tokens, nodes=nodes, tp=tp, shared=False, ep=1)
    c.update(changes)
    return c


def listed():
    named = [
        # fp32 layer of a debugging or conformance run: launches and latency only
        ("f32_tiny_64", _layer(TINY, 64)),
        # one sequence decoding alone: every kernel of the step is a latency chain
        ("decode_1", _layer(QWEN30, 1)),
        # a decode batch: nearly every expert's weights are read once for a few rows
        ("decode_64", _layer(QWEN30, 64)),
        # an EP rank of the larger model at an odd decode batch
        ("decode_ep_173", _layer(QWEN235, 173)),
        # e4m3 weights, a decode batch whose routing is skewed (hot experts)
        ("decode_fp8_skewed_256", _layer(DEEPSEEK, 256, weights="fp8", zipf=1.2)),
        # a prefill chunk mixed into serving, e4m3 weights, ragged token count
        ("chunk_fp8_1531", _layer(DEEPSEEK, 1531, weights="fp8")),
        # a prompt of the context length
        ("prefill_4096", _layer(QWEN30, 4096)),
        # the same layer cut over an eight-GPU TP group (96 columns per GPU), ragged
        ("prefill_tp8_3001", _layer(QWEN30, 3001, tp=8)),
        # 8-bit weights and activations, ragged token count
        ("prefill_fp8act_6007", _layer(DEEPSEEK, 6007, weights="fp8", fp8_acts=True)),
        # the default workload of bench.py
        ("prefill_ep_tp_16384", _layer(DEEPSEEK, 16384)),
        # the largest step: sixteen sequences of 4096 tokens
        ("prefill_65536", _layer(QWEN30, 65536)),
        # both ends of the fused schedules: a TP rank of eight builds the send buffers
        # of two nodes and adds up what the nodes return
        ("staged_tp8_8192", _staged(QWEN235, 8192, nodes=2, tp=8)),
    ]
    return [dict(c, name=n) for n, c in named]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("f32", "qwen30", "qwen30", "qwen30", "qwen235", "qwen235", "deepseek",
                       "deepseek", "deepseek", "staged"))
    if kind == "f32":
        experts = rng.choice((4, 8, 16, 32))
        return _layer(TINY, _log_int(rng, 16, 512), hidden=64 * rng.randint(2, 8), experts=experts,
                      top_k=rng.randint(1, 4), inter=64 * rng.randint(2, 8))
    if kind == "qwen30":
        weights = rng.choice(("bf16", "bf16", "bf16", "fp8"))
        tp = rng.choice((1, 1, 2, 4, 8)) if weights == "bf16" else rng.choice((1, 2))
        return _layer(QWEN30, _log_int(rng, 1, 65536 if weights == "bf16" else 49152), tp=tp, weights=weights)
    if kind == "qwen235":
        weights = rng.choice(("bf16", "bf16", "fp8"))
        return _layer(QWEN235, _log_int(rng, 1, 32768), ep_rank=rng.randint(0, 7), weights=weights,
                      tp=rng.choice((1, 1, 2, 4)))
    if kind == "deepseek":
        weights = rng.choice(("bf16", "fp8", "fp8"))
        fp8_acts = weights == "fp8" and rng.random() < 0.4
        tokens = _log_int(rng, 256 if fp8_acts else 1, 24576)
        zipf = rng.choice((0.0, 0.0, 0.0, 1.2)) if tokens <= 1024 else 0.0
        return _layer(DEEPSEEK, tokens, weights=weights, fp8_acts=fp8_acts, zipf=zipf,
                      ep_rank=rng.randint(0, 7), tp=rng.choice((1, 2, 2, 4)))
    model = rng.choice((QWEN30, QWEN235, DEEPSEEK))
    return _staged(model, _log_int(rng, 64, 16384), nodes=rng.choice((2, 4)), tp=rng.choice((2, 4, 8)))


# ---------------------------------------------------------------------------
def _workload(case, lo, hi):
    return Workload(name=case["path"], seed=0, T=case["tokens"], H=case["hidden"], E=case["experts"],
                    k=case["top_k"], I=case["inter"], score_fn=case["score"],
                    routed_scale=case["scale"], n_groups=case["groups"],
                    topk_groups=case["kept_groups"], group_score_n=2 if case["groups"] > 1 else 0,
                    expert_lo=lo, expert_hi=hi, tp=case["tp"], act_dtype=case["act"],
                    weight_dtype=case["weights"], shared_expert=case["shared"],
                    fp8_activations=case["fp8_acts"])


def _act_dtype(case):
    return torch.float32 if case["act"] == "f32" else torch.bfloat16


def _normal(g, shape, std, dtype):
    t = torch.empty(shape, dtype=dtype, device="cuda")
    return t.normal_(0.0, std, generator=g)


def _quantise(w):
    """e4m3 codes and one fp32 scale per 128 x 128 block of w [n, rows, cols]."""
    n, r, c = w.shape
    blocks = w.view(n, r // FP8_BLOCK, FP8_BLOCK, c // FP8_BLOCK, FP8_BLOCK)
    scale = blocks.abs().amax(dim=(2, 4)) / E4M3_MAX
    codes = (blocks / scale[:, :, None, :, None]).to(torch.float8_e4m3fn).view(torch.uint8)
    return codes.view(n, r, c), scale


def _expert_weights(g, case, n):
    """SwiGLU weights of n experts, N(0, 0.02), in their stored form."""
    inter, hidden = case["inter"] // case["tp"], case["hidden"]
    out = {}
    for name, shape in (("gate", (inter, hidden)), ("up", (inter, hidden)), ("down", (hidden, inter))):
        if case["weights"] != "fp8":
            dtype = torch.float32 if case["weights"] == "f32" else torch.bfloat16
            out["w_" + name] = _normal(g, (n,) + shape, 0.02, dtype)
            continue
        codes = torch.empty((n,) + shape, dtype=torch.uint8, device="cuda")
        scales = torch.empty(n, shape[0] // FP8_BLOCK, shape[1] // FP8_BLOCK, device="cuda")
        for e in range(0, n, 16):      # a few experts at a time: the fp32 values are four times the codes
            m = min(16, n - e)
            codes[e:e + m], scales[e:e + m] = _quantise(_normal(g, (m,) + shape, 0.02, torch.float32))
        out["w_" + name], out["s_" + name] = codes, scales
    return out


def _gate(g, case):
    E, H = case["experts"], case["hidden"]
    gate = {"gate_w": _normal(g, (E, H), 1.0 / math.sqrt(H), _act_dtype(case))}
    if case["bias"] == "logit":
        gate["logit_bias"] = _normal(g, (E,), 0.5, torch.float32)
    if case["bias"] == "select":
        gate["select_bias"] = _normal(g, (E,), 0.05, torch.float32)
    return gate


def _forced_routing(g, case):
    """Zipf-skewed expert choices: k distinct experts per token, probability
    proportional to rank^-s, ranks dealt round-robin to the expert ranges (every
    EP rank gets its share of the hot ones), normalised positive weights."""
    T, E, k, ep = case["tokens"], case["experts"], case["top_k"], case["ep"]
    ranks = torch.arange(1, E + 1, dtype=torch.float32, device="cuda")
    u = torch.rand(T, E, generator=g, device="cuda").clamp_(1e-7, 1 - 1e-7)
    top = (-case["zipf"] * ranks.log() - (-u.log()).log()).topk(k, dim=1).indices
    ids = (top % ep) * (E // ep) + top // ep
    w = torch.sigmoid(torch.randn(T, k, generator=g, device="cuda"))
    return ids.to(torch.int32).contiguous(), (w / w.sum(dim=1, keepdim=True) * case["scale"]).contiguous()


def _expert_range(case):
    per = case["experts"] // case["ep"]
    return case["ep_rank"] * per, (case["ep_rank"] + 1) * per


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    T, H = case["tokens"], case["hidden"]
    x = _normal(g, (T, H), 0.02 if case["act"] == "f32" else 1.0, _act_dtype(case))
    if case["path"] == "staged":
        return _prepare_staged(g, case, x)
    lo, hi = _expert_range(case)
    w = _workload(case, lo, hi)
    # the weights are drawn on the GPU, so they are attached to the layer as they are
    layer = MoELayerShare(config_from_workload(w), T, {}, {}, {} if case["shared"] else None,
                          fp8_activations=case["fp8_acts"])
    layer.gate = _gate(g, case)
    layer.experts = _expert_weights(g, case, hi - lo)
    if case["shared"]:
        layer.shared = _expert_weights(g, case, 1)
    forced = _forced_routing(g, case) if case["zipf"] else None
    return {"path": "layer", "layer": layer, "x": x, "forced": forced}


def _prepare_staged(g, case, x):
    T, k, H, E, tp, nodes = (case[n] for n in ("tokens", "top_k", "hidden", "experts", "tp", "nodes"))
    A, cols, adt = T * k, H // tp, _act_dtype(case)
    i32 = lambda *s: torch.zeros(*s, dtype=torch.int32, device="cuda")
    whole = config_from_workload(_workload(case, 0, E))
    state = {"path": "staged", "x": x, "cfg": whole, "tokens": T, "tp": tp, "gate": _gate(g, case),
             "ids": i32(T, k), "w": torch.zeros(T, k, device="cuda"),
             "ws": torch.zeros(moe.moe_workspace_bytes(whole, T), dtype=torch.uint8, device="cuda"),
             "out": torch.zeros(T, cols, device="cuda"), "nodes": []}
    per = E // nodes
    for n in range(nodes):
        state["nodes"].append({
            "cfg": config_from_workload(_workload(case, n * per, (n + 1) * per)),
            "counts": i32(per), "offsets": i32(per + 1), "perm": i32(A), "inv": i32(A),
            "send": torch.zeros(A, cols, dtype=adt, device="cuda"),      # this rank's columns, to node n
            "back": _normal(g, (A, cols), 1.0, adt)})                   # what node n returned
    return state


def run(state):
    if state["path"] == "layer":
        layer = state["layer"]
        out = layer.forward(state["x"], state["forced"])
        return {"out": out, "ids": layer.topk_ids, "weights": layer.topk_w, "counts": layer.counts,
                "inv": layer.inv}
    T, tp, gate = state["tokens"], state["tp"], state["gate"]
    moe.moe_route(state["cfg"], T, state["x"], gate["gate_w"], gate.get("logit_bias"),
                  gate.get("select_bias"), None, state["ids"], state["w"], state["ws"])
    for n in state["nodes"]:
        moe.moe_dispatch_shard(n["cfg"], T, state["x"], state["ids"], 0, tp, n["counts"], n["offsets"],
                               n["perm"], n["inv"], n["send"], state["ws"])
    for i, n in enumerate(state["nodes"]):
        moe.moe_combine_stage(n["cfg"], T, n["back"], n["inv"], state["w"], tp, i > 0, state["out"])
    return {"out": state["out"], "ids": state["ids"], "weights": state["w"],
            "counts": [n["counts"] for n in state["nodes"]], "inv": [n["inv"] for n in state["nodes"]],
            "send": [n["send"] for n in state["nodes"]]}


# ---------------------------------------------------------------------------
def _pick_probability(case):
    """Probability that a token picks the expert of each rank (all alike without
    forced routing): min(1, c * rank^-s) with the sum k."""
    E, k = case["experts"], case["top_k"]
    if not case["zipf"]:
        return [k / E] * E
    p = [(r + 1) ** -case["zipf"] for r in range(E)]
    lo, hi = 0.0, 1e6
    for _ in range(80):
        c = (lo + hi) / 2
        lo, hi = (c, hi) if sum(min(1.0, c * q) for q in p) < k else (lo, c)
    return [min(1.0, lo * q) for q in p]


def work(case):
    T, H, E, k = case["tokens"], case["hidden"], case["experts"], case["top_k"]
    ab = 4 if case["act"] == "f32" else 2
    route_bytes = (0 if case["zipf"] else E * H * ab) + T * k * 8
    gate_flops = 0.0 if case["zipf"] else 2.0 * T * H * E
    if case["path"] == "staged":
        cols = H // case["tp"]
        A = T * k        # every assignment goes to one of the nodes
        return {"bytes": T * H * ab + route_bytes + 2 * A * cols * ab + case["nodes"] * A * 4 + T * cols * 4,
                "flops": gate_flops + 2.0 * A * cols}
    inter = case["inter"] // case["tp"]
    p = _pick_probability(case)
    mine = p[case["ep_rank"]::case["ep"]] if case["zipf"] else p[:E // case["ep"]]
    rows, touched = T * sum(mine), sum(1.0 - (1.0 - min(q, 1.0)) ** T for q in mine)
    if case["shared"]:
        rows, touched = rows + T, touched + 1
    expert = 3 * inter * H * {"f32": 4.0, "bf16": 2.0, "fp8": 1.0 + 4.0 / FP8_BLOCK ** 2}[case["weights"]]
    return {"bytes": T * H * ab + route_bytes + touched * expert + T * H * 4,
            "flops": gate_flops + 6.0 * rows * H * inter}


def tolerance(case):
    """About four times what each path differs by from the same layer computed in
    64 bits (the measured relative errors stand behind each line)."""
    if case["act"] == "f32":
        return {"rel": 4e-6, "max": 4e-5}      # 7e-7
    if case["path"] == "staged":
        return {"rel": 1e-5, "max": 1e-4}      # sums 6e-8; the gate weights hold fp32 exponentials of fp32 logits
    if case["fp8_acts"]:
        return {"rel": 3e-2, "max": 0.5}       # 1.7e-2: a code of the intermediate moves by one step
    if case["weights"] == "fp8":
        return {"rel": 1.5e-2, "max": 0.1}     # 3.8e-3
    return {"rel": 1e-2, "max": 0.1}           # 2.4e-3
