"""The work that a user of this library has it do, as timed cases.

A case is one MoE layer configuration and one way of calling the library:

  path "layer"   moe_layer_forward, the one-call entry point that a serving loop uses
  path "calls"   the five separate calls (route, drop, dispatch, grouped FFN, combine), for callers that put
                 their own work between them
  path "plan"    moe_route_topk and moe_capacity_drop_ranked alone: the dispatch plan of a batch, which a
                 deployment computes on every device before it exchanges tokens

Sizes are those of the workloads in paper_2503_05066_amd/synth.py, of the tests and of bench.py, with ragged
ones of the same families between them.  Inputs are drawn on the GPU from the seed: activations N(0, 1), router
weights N(0, 1/d) with a bias that skews the load as the workloads' biases do, expert weights N(0, 1/fan-in).
"""
import math

import numpy as np
import torch

from paper_2503_05066_amd import capmoe

MODES = {"none": capmoe.MODE_NONE, "token": capmoe.MODE_TOKEN_DROP, "expanded": capmoe.MODE_EXPANDED_DROP}
SCOPES = {"local": capmoe.SCOPE_LOCAL, "global": capmoe.SCOPE_GLOBAL, "local_device": capmoe.SCOPE_LOCAL_DEVICE,
          "global_device": capmoe.SCOPE_GLOBAL_DEVICE}
METRICS = {"score": capmoe.METRIC_SCORE, "order": capmoe.METRIC_ORDER, "reverse_order": capmoe.METRIC_REVERSE_ORDER,
           "random": capmoe.METRIC_RANDOM}
DTYPES = {"bf16": (capmoe.DTYPE_BF16, torch.bfloat16), "f32": (capmoe.DTYPE_F32, torch.float32)}


def _case(name, path, dtype, n, d, e, k, h, groups, mode, **more):
    c = {"name": name, "path": path, "dtype": dtype, "tokens": n, "d_model": d, "experts": e, "top_k": k,
         "d_hidden": h, "groups": groups, "mode": mode, "scope": "local", "gamma": 1.0, "metric": "score",
         "overselect": 0, "max_experts": False, "classes": False, "skew": "normal", "skew_param": 1.0}
    c.update(more)
    return c


def listed():
    return [
        # the next token of a single sequence through a fine-grained layer: no capacity applies, latency is all
        _case("decode_1_token", "layer", "bf16", 1, 2048, 64, 8, 1024, 1, "none", skew="zipf", skew_param=1.1),
        # the smallest whole layer, fp32: what a unit test or a toy model of a user runs
        _case("tiny_f32", "layer", "f32", 128, 64, 8, 2, 128, 1, "token"),
        # decoding a small batch with few, wide experts: streams nearly all weights for sixteen tokens
        _case("decode_16_wide_experts", "layer", "bf16", 16, 4096, 8, 2, 14336, 1, "none", skew_param=0.5),
        # decoding an odd batch with a generous capacity over the whole batch
        _case("decode_37_odd", "layer", "bf16", 37, 4096, 64, 6, 1408, 1, "token", scope="global", gamma=2.0,
              skew="one_hot", skew_param=3.0),
        # a full decoding batch over eight simulated devices with the tokens' local experts as extra candidates
        _case("decode_256_expanded", "layer", "bf16", 256, 4096, 64, 6, 1408, 8, "expanded", skew="one_hot",
              skew_param=3.0),
        # a short ragged prompt on a layer whose expert count and token count divide nothing
        _case("prefill_1531_odd", "layer", "bf16", 1531, 2048, 60, 4, 1408, 1, "token", gamma=1.25, skew="zipf",
              skew_param=1.0),
        # an ordinary prompt batch, skewed routing, Token Drop: small experts, the weight stream binds
        _case("prefill_4096", "layer", "bf16", 4096, 2048, 64, 8, 1024, 1, "token", skew="zipf", skew_param=1.1),
        # the separate calls with the over-selected candidate lists and the limit of k experts per token
        _case("calls_3000_limited", "calls", "bf16", 3000, 2048, 64, 8, 1024, 4, "expanded", gamma=1.5, overselect=8,
              max_experts=True, skew="zipf", skew_param=1.1),
        # many small experts over eight devices, Expanded Drop
        _case("prefill_16384_expanded", "layer", "bf16", 16384, 2048, 128, 8, 768, 8, "expanded", skew="zipf",
              skew_param=1.2),
        # few wide experts, Token Drop: the matrix products bind
        _case("prefill_8192_wide", "layer", "bf16", 8192, 4096, 8, 2, 14336, 4, "token", skew_param=1.5),
        # an fp32 layer of a size that people check or fine-tune models at
        _case("layer_f32", "layer", "f32", 1024, 1024, 16, 2, 2048, 1, "token", gamma=1.5),
        # the plan of a long batch under a device-level budget, two token classes, drawn ranks
        _case("plan_65536_device", "plan", "bf16", 65536, 2048, 64, 8, 1024, 8, "expanded", scope="local_device",
              metric="random", classes=True, skew="zipf", skew_param=1.1),
    ]


def _log_int(rng, low, high):
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def draw(rng):
    """A case of the same ranges: a decoding step, a prefill, an fp32 layer or a plan, with any of the options."""
    kind = rng.choice(["decode", "decode", "prefill", "prefill", "f32", "plan"])
    while True:
        e = rng.choice([8, 16, 32, 48, 60, 64, 96, 128])
        groups = rng.choice([g for g in (1, 1, 2, 4, 8) if e % g == 0])
        k = rng.choice([1, 2, 4, 6, 8])
        mode = rng.choice(["none", "token", "token", "expanded"])
        scope = rng.choice(["local", "local", "global", "local_device", "global_device"])
        metric = rng.choice(["score", "score", "score", "order", "reverse_order", "random"])
        gamma = rng.choice([0.5, 1.0, 1.0, 1.25, 1.5, 2.0])
        overselect = rng.choice([0, 0, 0, k, 2 * k]) if k <= e // 4 else 0
        dtype = "f32" if kind == "f32" else "bf16"
        if kind == "decode":
            n = _log_int(rng, 1, 512)
        elif kind == "prefill":
            n = _log_int(rng, 512, 16384)
        elif kind == "f32":
            n = _log_int(rng, 32, 2048)
        else:
            n = _log_int(rng, 4096, 65536)
        n = max(groups, n - n % groups)
        if kind == "f32":
            d, h = 8 * rng.randint(8, 128), _log_int(rng, 96, 2048)
        else:
            d, h = 128 * rng.randint(8, 32), 128 * int(round(math.exp(rng.uniform(math.log(4), math.log(112)))))
        weights = 3 * e * d * h
        flops = 6 * n * (k + overselect + (e // groups if mode == "expanded" else 0)) * d * h
        if mode != "none":  # the capacity bounds the rows
            flops = min(flops, 6 * int(gamma * n * k) * d * h)
        if kind == "f32":
            fits = weights <= 3 * 16 * 1024 * 2048 and flops <= 6 * 3072 * 1024 * 2048
        elif kind == "plan":
            fits = n * d <= 65536 * 2048
        else:
            fits = weights <= 3 * 8 * 4096 * 14336 and flops <= 6 * 16384 * 4096 * 14336 and n * d <= 16384 * 4096
        if not fits:
            continue
        skew = rng.choice(["normal", "zipf", "one_hot"])
        param = {"normal": round(rng.uniform(0.5, 1.5), 2), "zipf": round(rng.uniform(0.8, 1.2), 2), "one_hot": 3.0}[skew]
        path = "plan" if kind == "plan" else rng.choice(["layer", "layer", "calls"])
        c = _case("", path, dtype, n, d, e, k, h, groups, mode, scope=scope, gamma=gamma, metric=metric,
                  overselect=overselect, max_experts=rng.random() < 0.25, classes=rng.random() < 0.25, skew=skew,
                  skew_param=param)
        if capmoe.moe_query(_desc(c))[0] > 0:  # a capacity that truncates to nothing is no layer
            del c["name"]
            return c


def _bias(case):
    """Per-expert logit offsets of the case's skew, largest first (the seed decides which expert gets which)."""
    e, p = case["experts"], case["skew_param"]
    if case["skew"] == "zipf":
        ranks = np.arange(1, e + 1, dtype=np.float64)
        return -p * np.log(ranks) - math.log(float(np.sum(ranks ** -p)))
    if case["skew"] == "one_hot":
        b = np.zeros(e)
        b[0] = p
        return b
    return np.sort(np.random.default_rng(e).standard_normal(e))[::-1] * p


def _desc(case):
    return capmoe.make_desc(case["tokens"], case["d_model"], case["experts"], case["top_k"], case["d_hidden"],
                            case["groups"], MODES[case["mode"]], SCOPES[case["scope"]], case["gamma"],
                            DTYPES[case["dtype"]][0], METRICS[case["metric"]], case["overselect"],
                            int(case["max_experts"]))


def prepare(case, seed):
    desc = _desc(case)
    act = DTYPES[case["dtype"]][1]
    n, d, e, h = case["tokens"], case["d_model"], case["experts"], case["d_hidden"]
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(shape, std, dtype):
        return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, std, generator=gen)

    s = {"case": dict(case), "desc": desc, "seed": seed & 0xFFFFFFFF}
    s["x"] = normal((n, d), 1.0, act)
    s["w_router"] = normal((e, d), d ** -0.5, torch.float32)
    order = torch.randperm(e, generator=gen, device="cuda")
    s["bias"] = torch.tensor(_bias(case), dtype=torch.float32, device="cuda")[order]
    s["token_class"] = None
    if case["classes"]:  # image tokens (class 0, dropped first) among text tokens
        s["token_class"] = torch.randint(0, 2, (n,), generator=gen, device="cuda", dtype=torch.uint8)
    if case["path"] != "plan":
        s["w_gate"] = normal((e, h, d), d ** -0.5, act)
        s["w_up"] = normal((e, h, d), d ** -0.5, act)
        s["w_down"] = normal((e, d, h), h ** -0.5, act)
        s["buf"] = capmoe.LayerBuffers(desc)
    else:
        s["buf"] = _plan_buffers(desc)
    # the plan has fewer rows than its arrays hold, and the calls leave the rest as it is
    s["buf"].row_token.zero_()
    s["buf"].row_weight.zero_()
    return s


class _PlanBuffers:
    pass


def _plan_buffers(desc):
    """What LayerBuffers holds, without the activations: a caller that only plans has none."""
    cap, slots, max_rows, workspace = capmoe.moe_query(desc)
    n, e, k = desc.n_tokens, desc.n_experts, desc.top_k + desc.overselect
    blocks = desc.device_groups if desc.capacity_scope in (capmoe.SCOPE_LOCAL, capmoe.SCOPE_LOCAL_DEVICE) else 1
    rows = max(max_rows, 1)

    def mk(shape, dtype):
        return torch.empty(shape, dtype=dtype, device="cuda")

    b = _PlanBuffers()
    b.logits, b.scores = mk((n, e), torch.float32), mk((n, e), torch.float32)
    b.topk_idx, b.topk_score = mk((n, k), torch.int32), mk((n, k), torch.float32)
    b.expert_count, b.seg_count = mk((e,), torch.int32), mk((blocks, e), torch.int32)
    b.expert_offset = mk((e + 1,), torch.int32)
    b.row_token, b.row_weight = mk((rows,), torch.int32), mk((rows,), torch.float32)
    b.pair_row = mk((n, slots), torch.int32)
    b.workspace = mk((max(workspace, 256),), torch.uint8)
    return b


def run(s):
    case, desc, buf = s["case"], s["desc"], s["buf"]
    if case["path"] == "layer":
        capmoe.moe_layer_forward(desc, s["x"], s["w_router"], s["bias"], s["w_gate"], s["w_up"], s["w_down"],
                                 s["token_class"], s["seed"], buf)
    elif case["path"] == "calls":
        capmoe.layer_forward(buf, s["x"], s["w_router"], s["bias"], s["w_gate"], s["w_up"], s["w_down"],
                             token_class=s["token_class"], seed=s["seed"])
    else:
        capmoe.moe_route_topk(desc, s["x"], s["w_router"], s["bias"], 0, buf.logits, buf.scores, buf.topk_idx,
                              buf.topk_score, buf.workspace)
        capmoe.moe_capacity_drop_ranked(desc, buf.scores, buf.topk_idx, s["token_class"], s["seed"], buf.expert_count,
                                        buf.seg_count, buf.expert_offset, buf.row_token, buf.row_weight, buf.pair_row,
                                        buf.workspace)
    out = {"logits": buf.logits, "scores": buf.scores, "topk_idx": buf.topk_idx, "topk_score": buf.topk_score,
           "expert_count": buf.expert_count, "seg_count": buf.seg_count, "expert_offset": buf.expert_offset,
           "row_token": buf.row_token, "row_weight": buf.row_weight, "pair_row": buf.pair_row}
    if case["path"] != "plan":
        out["y"] = buf.y
    return out


def _expected_rows(case):
    """(kept pairs, experts with at least one) of the case: its routing drawn on the host, because the logits are
    N(0, 1) plus the skew whatever the seed.  Small batches are drawn several times and averaged."""
    rng = np.random.default_rng(1)
    got = [_draw_rows(case, rng) for _ in range(max(1, 512 // case["tokens"]))]
    return tuple(float(np.mean([g[i] for g in got])) for i in (0, 1))


def _draw_rows(case, rng):
    n, e, k, g = case["tokens"], case["experts"], case["top_k"] + case["overselect"], case["groups"]
    m = min(n, 2048)
    scale = n / m
    logits = rng.standard_normal((m, e)) + _bias(case)[rng.permutation(e)]
    cand = np.zeros((m, e), bool)
    np.put_along_axis(cand, np.argpartition(-logits, k - 1, axis=1)[:, :k], True, axis=1)
    device = (np.arange(m) * g) // m
    if case["mode"] == "expanded":
        cand |= device[:, None] == np.arange(e)[None, :] // (e // g)
    if case["mode"] == "none":
        load = cand.sum(axis=0) * scale
    else:
        cap = capmoe.moe_query(_desc(case))[0]
        blocks = device if case["scope"] in ("local", "local_device") else np.zeros(m, int)
        load = np.zeros(e)
        for b in range(int(blocks.max()) + 1):
            c = cand[blocks == b].sum(axis=0) * scale
            if case["scope"].endswith("device"):
                per = c.reshape(g, e // g)
                total = np.maximum(per.sum(axis=1, keepdims=True), 1e-9)
                load += (per * np.minimum(1.0, cap / total)).reshape(e)
            else:
                load += np.minimum(c, cap)
    if case["max_experts"]:
        load = load * min(1.0, n * case["top_k"] / max(load.sum(), 1e-9))
    return float(load.sum()), int((load > 0).sum())


def work(case):
    n, d, e, h = case["tokens"], case["d_model"], case["experts"], case["d_hidden"]
    listed_k = case["top_k"] + case["overselect"]
    slots = listed_k + (e // case["groups"] if case["mode"] == "expanded" else 0)
    elem = 2 if case["dtype"] == "bf16" else 4
    rows, active = _expected_rows(case)
    b = n * d * elem + e * d * 4 + 2 * n * e * 4 + n * listed_k * 8 + rows * 8 + n * slots * 4
    f = 2.0 * n * d * e
    if case["path"] != "plan":
        b += active * 3 * d * h * elem + n * d * elem
        f += 6.0 * d * h * rows
    return {"bytes": float(b), "flops": f}


def tolerance(case):
    # Measured against the same layer in fp32 (bf16 cases) and fp64 (fp32 cases) with the library's own plan: bf16 differs
    # by 2.9e-3 (largest 2.2e-2 of the rms: the hidden activation, the expert outputs and y are each rounded once),
    # fp32 by 1.2e-6 (largest 1e-5).  Four times that.  Routing and plans are whole numbers and stay the same.
    if case["path"] == "plan" or case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-4}
    return {"rel": 1e-2, "max": 1e-1}
