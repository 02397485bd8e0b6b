"""GPU parity: the HIP path (through the C ABI) against the CPU oracle on the same seeded inputs.

Integer results (top-k indices, counts, offsets, the dispatch plan) and the fp32 scores must be
bit-exact given identical fp32 logits; router logits within 1e-4; layer outputs within 1e-4
(fp32) / 2e-2 (bf16) relative error.  Run with `-m gpu` on an MI355X.
"""
import math

import numpy as np
import pytest
import torch

from paper_2503_05066_amd import capmoe, synth

from gpu_util import DeviceLayer, assert_output_close, assert_plan_equal, to_host_f64

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("built_library")]

NONE, TD, ED = synth.MODE_NONE, synth.MODE_TOKEN_DROP, synth.MODE_EXPANDED_DROP
LOCAL, GLOBAL = synth.SCOPE_LOCAL, synth.SCOPE_GLOBAL
W = synth.WORKLOADS
TOL = {synth.DTYPE_F32: 1e-4, synth.DTYPE_BF16: 2e-2}


def note(*a):
    print(*a, flush=True)


def route_and_drop_gpu(desc, logits_host, token_class=None, seed=0):
    """moe_route_topk (given logits) + moe_capacity_drop[_ranked]; returns the buffers."""
    buf = capmoe.LayerBuffers(desc)
    if desc.n_tokens:
        buf.logits.copy_(torch.from_numpy(logits_host))
    capmoe.moe_route_topk(desc, None, None, None, 1, buf.logits, buf.scores, buf.topk_idx, buf.topk_score,
                          buf.workspace)
    if token_class is None and seed == 0:
        capmoe.moe_capacity_drop(desc, buf.scores, buf.topk_idx, buf.expert_count, buf.seg_count, buf.expert_offset,
                                 buf.row_token, buf.row_weight, buf.pair_row, buf.workspace)
    else:
        tc = torch.from_numpy(token_class).cuda() if token_class is not None else None
        capmoe.moe_capacity_drop_ranked(desc, buf.scores, buf.topk_idx, tc, seed, buf.expert_count, buf.seg_count,
                                        buf.expert_offset, buf.row_token, buf.row_weight, buf.pair_row, buf.workspace)
    torch.cuda.synchronize()
    return buf


def check_route_and_plan(orc, logits, n, e, k, g, mode, scope, gamma, what, metric=0, token_class=None, seed=0,
                         overselect=0, max_experts=False):
    note("case", what, dict(n=n, e=e, k=k, g=g, mode=mode, scope=scope, gamma=gamma, metric=metric, seed=seed,
                            classes=token_class is not None, overselect=overselect, max_experts=max_experts))
    desc = capmoe.make_desc(n, 64, e, k, 128, g, mode, scope, gamma, synth.DTYPE_F32, metric, overselect,
                            int(max_experts))
    buf = route_and_drop_gpu(desc, logits, token_class, seed)
    ref = orc.route_and_drop(logits, k, g, mode, scope, gamma, metric, token_class, seed, overselect, max_experts)
    assert buf.cap == ref.cap
    np.testing.assert_array_equal(buf.scores.cpu().numpy().view(np.uint32), ref.scores.view(np.uint32))
    np.testing.assert_array_equal(buf.topk_idx.cpu().numpy(), ref.topk_idx)
    np.testing.assert_array_equal(buf.topk_score.cpu().numpy().view(np.uint32), ref.topk_score.view(np.uint32))
    assert_plan_equal(buf, ref, what)
    assert ref.plan.rows <= buf.max_rows
    assert ref.plan.seg_count.max(initial=0) <= ref.cap      # max load <= C
    return buf, ref


# ------------------------------------------------------------------------------------------------
# router logits
# ------------------------------------------------------------------------------------------------
@pytest.mark.parametrize("name,n", [("tiny", 128), ("olmoe", 1000), ("decode", 256), ("finegrained", 777),
                                    ("mixtral", 8192), ("olmoe", 4096), ("finegrained", 16384)])
def test_router_logits(orc, name, n):
    w = synth.scaled(W[name], n_tokens=n, device_groups=1)
    note("router logits", w)
    x = synth.tokens(w)
    wr, b = synth.router_weight(w), synth.router_bias(w)
    ref = orc.router_logits(x.f32, wr, b)
    desc = capmoe.make_desc(n, w.d_model, w.n_experts, w.top_k, w.d_hidden, 1, TD, LOCAL, 1.0, w.dtype)
    buf = capmoe.LayerBuffers(desc)
    from gpu_util import to_device
    capmoe.moe_route_topk(desc, to_device(x), torch.from_numpy(wr).cuda(), torch.from_numpy(b).cuda(), 0, buf.logits,
                          buf.scores, buf.topk_idx, buf.topk_score, buf.workspace)
    torch.cuda.synchronize()
    got = buf.logits.cpu().numpy()
    assert np.abs(got - ref).max() <= 1e-4 * np.abs(ref).max()
    # without bias
    capmoe.moe_route_topk(desc, to_device(x), torch.from_numpy(wr).cuda(), None, 0, buf.logits, buf.scores,
                          buf.topk_idx, buf.topk_score, buf.workspace)
    torch.cuda.synchronize()
    ref0 = orc.router_logits(x.f32, wr)
    assert np.abs(buf.logits.cpu().numpy() - ref0).max() <= 1e-4 * np.abs(ref0).max()


@pytest.mark.parametrize("n,d,e", [
    (300, 96, 100),     # three k-slabs in all: the shallowest request ring; two expert chunks, the second ragged
    (257, 192, 200),    # seven expert tiles in chunks of 4 + 3
    (129, 256, 250),    # E not a multiple of 4: scalar stores
    (1000, 512, 160),   # five expert tiles in chunks of 3 + 2
    (64, 128, 3),
    (17, 64, 1),        # a single expert
    (5000, 64, 33),
    (40000, 64, 8),     # enough token tiles for a single K slice: the bias is added in the kernel
    (33000, 128, 128),  # the same with two expert chunks
])
def test_router_logits_shapes(orc, n, d, e):
    w = synth.scaled(W["olmoe"], n_tokens=n, d_model=d, n_experts=e, top_k=min(8, e), d_hidden=128, device_groups=1)
    note("router logits, odd shapes", w)
    x = synth.tokens(w)
    wr, b = synth.router_weight(w), synth.router_bias(w)
    ref = orc.router_logits(x.f32, wr, b)
    desc = capmoe.make_desc(n, d, e, w.top_k, w.d_hidden, 1, TD, LOCAL, 1.0, w.dtype)
    buf = capmoe.LayerBuffers(desc)
    from gpu_util import to_device
    capmoe.moe_route_topk(desc, to_device(x), torch.from_numpy(wr).cuda(), torch.from_numpy(b).cuda(), 0, buf.logits,
                          buf.scores, buf.topk_idx, buf.topk_score, buf.workspace)
    torch.cuda.synchronize()
    got = buf.logits.cpu().numpy()
    assert got.shape == ref.shape
    assert np.abs(got - ref).max() <= 1e-4 * np.abs(ref).max()


@pytest.mark.parametrize("n,d,e", [
    (1, 4, 1), (15, 60, 16), (16, 64, 17), (33, 68, 8),        # below, at and above one K slab; edges of both tilings
    (31, 252, 33), (64, 256, 32), (70, 320, 100), (32, 324, 16),  # the ring of four slabs: not full, full, once around
    (130, 1024, 10),
])
def test_router_logits_fp32_chain(n, d, e):
    """A logit of fp32 activations is the chain of fused multiply-adds over ascending k, rounded once per product: bit for
    bit, so that equal inputs route alike whatever the batch they come in.  The reference chain adds in 64-bit
    significands, which hold every product exactly."""
    rng = np.random.default_rng(n * 1000 + d + e)
    x, wr = rng.standard_normal((n, d)).astype(np.float32), rng.standard_normal((e, d)).astype(np.float32)
    b = rng.standard_normal(e).astype(np.float32)
    ref = np.zeros((n, e), np.float32)
    for k in range(d):
        prod = x[:, None, k].astype(np.longdouble) * wr[None, :, k].astype(np.longdouble)
        ref = (ref.astype(np.longdouble) + prod).astype(np.float32)
    ref = ref + b
    desc = capmoe.make_desc(n, d, e, 1, 8, 1, NONE, LOCAL, 1.0, synth.DTYPE_F32)
    buf = capmoe.LayerBuffers(desc)
    storage = torch.zeros(n * d + 1, device="cuda")
    for x_dev in (torch.from_numpy(x).cuda(), storage[1:].view(n, d).copy_(torch.from_numpy(x))):   # also from an odd float
        capmoe.moe_route_topk(desc, x_dev, torch.from_numpy(wr).cuda(), torch.from_numpy(b).cuda(), 0, buf.logits,
                              buf.scores, buf.topk_idx, buf.topk_score, buf.workspace)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(buf.logits.cpu().numpy().view(np.uint32), ref.view(np.uint32))


# ------------------------------------------------------------------------------------------------
# scores, top-k and the dispatch plan, bit-exact from identical logits
# ------------------------------------------------------------------------------------------------
def oracle_logits(orc, w):
    return orc.router_logits(synth.tokens(w).f32, synth.router_weight(w), synth.router_bias(w))


FULL_CASES = [
    ("tiny", NONE, LOCAL, 1.0), ("tiny", TD, LOCAL, 1.0),
    ("olmoe", NONE, LOCAL, 1.0), ("olmoe", TD, LOCAL, 1.0), ("olmoe", TD, LOCAL, 1.5), ("olmoe", TD, LOCAL, 2.0),
    ("mixtral", NONE, LOCAL, 1.0), ("mixtral", TD, LOCAL, 1.0), ("mixtral", ED, LOCAL, 1.0),
    ("mixtral", TD, GLOBAL, 1.0), ("mixtral", ED, GLOBAL, 1.0),
    ("finegrained", TD, LOCAL, 1.0), ("finegrained", ED, LOCAL, 1.0), ("finegrained", ED, LOCAL, 1.25),
    ("finegrained", ED, GLOBAL, 1.25),
    ("decode", TD, LOCAL, 1.0), ("decode", ED, LOCAL, 1.0), ("decode", ED, GLOBAL, 1.0),
]
_logit_cache = {}


@pytest.mark.parametrize("name,mode,scope,gamma", FULL_CASES)
def test_plan_full_size(orc, name, mode, scope, gamma):
    w = W[name]
    if name not in _logit_cache:
        _logit_cache[name] = oracle_logits(orc, w)
    check_route_and_plan(orc, _logit_cache[name], w.n_tokens, w.n_experts, w.top_k, w.device_groups, mode, scope,
                         gamma, f"{name} full size")


@pytest.mark.parametrize("n,e,k,g,mode,scope,gamma", [
    (1000, 8, 2, 1, TD, GLOBAL, 1.0),       # segment longer than a block, ragged tail
    (1000, 10, 3, 5, ED, LOCAL, 0.8),
    (300, 3, 1, 3, ED, GLOBAL, 1.3),
    (96, 12, 12, 4, TD, LOCAL, 1.0),        # k = E: every expert is a candidate of every token
    (64, 100, 7, 4, ED, LOCAL, 2.0),        # E not a multiple of the wave width
    (520, 200, 9, 8, ED, LOCAL, 1.0),
    (64, 256, 64, 1, TD, GLOBAL, 1.0),      # largest top-k
    (4, 4, 2, 4, ED, LOCAL, 1.0),           # one token per device
    (1, 8, 2, 1, TD, GLOBAL, 1.0),
    (512, 16, 4, 4, TD, LOCAL, 0.0),        # gamma = 0 drops everything
    (512, 16, 4, 4, ED, GLOBAL, math.inf),  # no limit: all k+m candidates survive
    (512, 16, 4, 4, NONE, GLOBAL, 0.3),     # mode none ignores gamma
    (5000, 8, 2, 1, TD, GLOBAL, 0.05),
    (9000, 8, 2, 1, TD, GLOBAL, 1.0),       # a segment longer than the single-launch drop holds: three kernels
    (9000, 12, 3, 3, ED, GLOBAL, 0.9),
    (8192, 8, 2, 2, ED, LOCAL, 1.0),        # the longest segments the single launch takes are 8192 tokens: 4096 here,
    (8192, 4, 2, 1, TD, GLOBAL, 1.1),       # and exactly 8192 here
    (1027, 6, 3, 1, TD, GLOBAL, 0.9),       # odd top-k width: scalar list loads; ragged last round of tokens
    (1026, 6, 2, 1, TD, GLOBAL, 0.9),       # two entries per load
])
def test_plan_edge_shapes(orc, n, e, k, g, mode, scope, gamma):
    rng = np.random.default_rng(n * 7 + e)
    logits = (rng.standard_normal((n, e)) * 2 + rng.standard_normal(e)[None, :] * 1.5).astype(np.float32)
    check_route_and_plan(orc, logits, n, e, k, g, mode, scope, gamma, "edge shape")


# Segments around and beyond what a block holds in its registers (65536 keys, 32768 at an odd pitch): the selection re-reads
# its keys or shares them among blocks, and the compaction of a segment is spread over one block per 4096 tokens.
@pytest.mark.parametrize("n,e,k,g,mode,scope,gamma,flat", [
    (70001, 8, 2, 1, TD, GLOBAL, 1.0, False),     # token count not a multiple of 4: scalar key loads
    (65536, 4, 1, 1, TD, GLOBAL, 0.7, False),     # 16-byte key loads
    (65536, 4, 2, 1, TD, GLOBAL, 0.5, True),      # every score equal: the threshold is a tie of 32768 keys
    (49152, 16, 4, 4, ED, GLOBAL, 1.0, False),
    (40000, 16, 2, 4, TD, 3, 1.0, False),         # device budgets over 4 x 40000 keys
    (40000, 16, 2, 4, ED, 3, 0.6, True),
    (36864, 6, 6, 1, TD, GLOBAL, 0.5, False),     # every expert is a candidate of every token
])
def test_plan_long_segments(orc, n, e, k, g, mode, scope, gamma, flat):
    rng = np.random.default_rng(n + e)
    if flat:
        logits = np.zeros((n, e), np.float32)
    else:
        logits = (rng.standard_normal((n, e)) * 2 + rng.standard_normal(e)[None, :] * 1.5).astype(np.float32)
    check_route_and_plan(orc, logits, n, e, k, g, mode, scope, gamma, "long segments")


# 2048 tokens: the single-launch drop; 16384 tokens in one block of tokens: segments too long for it, so the
# three-kernel chain runs with per-expert capacities as well
@pytest.mark.parametrize("mode,scope,g,n", [(TD, GLOBAL, 1, 2048), (TD, LOCAL, 4, 2048), (ED, LOCAL, 4, 2048),
                                            (ED, GLOBAL, 8, 2048), (TD, GLOBAL, 1, 16384), (ED, GLOBAL, 4, 16384)])
def test_plan_with_forced_ties(orc, mode, scope, g, n):
    w = synth.scaled(W["olmoe"], n_tokens=n, n_experts=32, top_k=4, device_groups=g)
    logits = synth.logits_with_ties(w)
    buf, ref = check_route_and_plan(orc, logits, w.n_tokens, w.n_experts, w.top_k, g, mode, scope, 1.0, "ties")
    # the input really ties at thresholds: some segment keeps only part of a run of equal scores
    s, kp, cd = ref.scores, ref.keep.astype(bool), ref.cand.astype(bool)
    partial = 0
    for j in range(w.n_experts):
        kept_scores = set(s[kp[:, j], j].tolist())
        dropped_scores = set(s[cd[:, j] & ~kp[:, j], j].tolist())
        partial += len(kept_scores & dropped_scores)
    assert partial > 0


@pytest.mark.parametrize("name,mode,scope,gamma,metric,classes,seed", [
    ("olmoe", TD, LOCAL, 1.0, 1, False, 0), ("olmoe", TD, LOCAL, 1.0, 2, False, 0), ("olmoe", TD, LOCAL, 1.5, 3, False, 11),
    ("olmoe", TD, LOCAL, 0.5, 0, True, 0), ("olmoe", TD, LOCAL, 1.0, 3, True, 12),
    ("finegrained", ED, LOCAL, 1.0, 1, False, 0), ("finegrained", ED, LOCAL, 1.0, 3, True, 13),
    ("mixtral", ED, GLOBAL, 1.0, 2, True, 0), ("decode", ED, LOCAL, 1.0, 3, False, 14), ("tiny", TD, LOCAL, 1.0, 1, True, 0),
])
def test_plan_other_metrics_and_token_classes(orc, name, mode, scope, gamma, metric, classes, seed):
    """Order / Reverse Order / Random (Sec. 4) and the multimodal class strategies, at full size."""
    w = W[name]
    if name not in _logit_cache:
        _logit_cache[name] = oracle_logits(orc, w)
    cls = None
    if classes:   # about 70 % "image" tokens (class 0, dropped first), the rest "text" (class 1)
        cls = (np.random.default_rng(w.seed(5)).random(w.n_tokens) >= 0.7).astype(np.uint8)
    buf, ref = check_route_and_plan(orc, _logit_cache[name], w.n_tokens, w.n_experts, w.top_k, w.device_groups, mode,
                                    scope, gamma, f"{name} metric {metric}", metric, cls, seed)
    base = orc.route_and_drop(_logit_cache[name], w.top_k, w.device_groups, mode, scope, gamma)
    np.testing.assert_array_equal(ref.plan.seg_count, base.plan.seg_count)   # loads depend on capacity only
    if ref.cand.sum() > ref.keep.sum():
        assert (ref.keep != base.keep).any()


LOCAL_DEV, GLOBAL_DEV = 2, 3


@pytest.mark.parametrize("name,mode,scope,gamma,metric", [
    ("mixtral", TD, LOCAL_DEV, 1.0, 0), ("mixtral", ED, LOCAL_DEV, 1.0, 0), ("mixtral", TD, GLOBAL_DEV, 1.5, 0),
    ("finegrained", TD, LOCAL_DEV, 1.0, 0), ("finegrained", ED, LOCAL_DEV, 1.0, 0), ("finegrained", TD, GLOBAL_DEV, 1.0, 3),
    ("decode", ED, LOCAL_DEV, 1.0, 0), ("decode", TD, LOCAL_DEV, 1.0, 1), ("olmoe", TD, LOCAL_DEV, 1.0, 0),
])
def test_plan_device_level_capacity(orc, name, mode, scope, gamma, metric):
    """One budget per device's experts (Sec. 5.2 of the paper), full size."""
    w = W[name]
    if name not in _logit_cache:
        _logit_cache[name] = oracle_logits(orc, w)
    buf, ref = check_route_and_plan(orc, _logit_cache[name], w.n_tokens, w.n_experts, w.top_k, w.device_groups, mode,
                                    scope, gamma, f"{name} device-level", metric, None, 5 if metric == 3 else 0)
    m = w.n_experts // w.device_groups
    per_device = ref.plan.seg_count.reshape(ref.plan.seg_count.shape[0], w.device_groups, m).sum(2)
    assert per_device.max() <= ref.cap                                  # aggregated device load <= n_l gamma N_bar
    if m > 1 and mode == TD:
        expert_level = orc.route_and_drop(_logit_cache[name], w.top_k, w.device_groups, mode, scope - 2, gamma, metric,
                                          None, 5 if metric == 3 else 0)
        assert ref.plan.rows >= expert_level.plan.rows                  # less restrictive than per-expert limits


@pytest.mark.parametrize("n,e,k,g,mode,scope,gamma", [
    (256, 256, 8, 2, ED, LOCAL, 1.0),          # 136 candidate slots per token
    (256, 256, 8, 1, TD, 3, 1.0),              # one budget over all 256 experts: 65536 keys in one segment
    (2048, 64, 6, 2, ED, 2, 0.7),              # 32 experts x 1024 tokens under one budget
    (4100, 16, 2, 4, TD, 2, 1.0),              # ragged blocks of 1025 tokens
    (64, 8, 2, 8, TD, 3, 1.5),                 # one expert per device: device budget = expert capacity
])
def test_plan_large_segments(orc, n, e, k, g, mode, scope, gamma):
    rng = np.random.default_rng(n + e)
    logits = (rng.standard_normal((n, e)) * 2 + rng.standard_normal(e)[None, :] * 1.5).astype(np.float32)
    check_route_and_plan(orc, logits, n, e, k, g, mode, scope, gamma, "large segment")


@pytest.mark.parametrize("n,e,k,g,mode,scope,gamma,metric,ties", [
    (4100, 32, 4, 1, TD, GLOBAL_DEV, 1.0, 0, None),     # 131200 keys in one segment, ragged last chunk
    (4101, 24, 3, 1, ED, LOCAL_DEV, 0.7, 0, None),         # odd: keys fetched one at a time; every expert a candidate
    (4608, 48, 6, 2, ED, GLOBAL_DEV, 0.9, 3, None),     # two segments, drawn ranks, half of the experts local
    (9000, 64, 2, 4, TD, GLOBAL_DEV, 1.25, 1, None),    # Order: the boundary token holds several equal keys
    (18000, 16, 4, 2, TD, LOCAL_DEV, 0.5, 2, None),     # Reverse Order, capacity per device's own tokens
    (4096, 32, 2, 1, TD, LOCAL_DEV, 40.0, 0, None),     # fewer candidates than the budget
    (4096, 32, 4, 1, TD, GLOBAL_DEV, 0.6, 0, "flat"),   # every score equal: token and expert order decide
    (6001, 24, 4, 1, ED, GLOBAL_DEV, 0.3, 0, "few"),    # three different logits
    (70004, 2, 1, 1, TD, GLOBAL, 0.4, 0, "few"),           # long segments of single experts
    (16389, 3, 1, 1, TD, GLOBAL, 0.4, 0, None),            # odd keys, held by one block
    (10922, 3, 1, 1, TD, LOCAL_DEV, 0.4, 0, None),         # 32766 and 32769 of them: either side of the line
    (10923, 3, 1, 1, TD, LOCAL_DEV, 0.4, 0, None),
    (16384, 4, 1, 1, TD, LOCAL_DEV, 0.4, 0, None),         # the most keys one block holds
    (4096, 32, 2, 1, TD, LOCAL_DEV, 0.0, 0, None),      # no capacity
    (683, 3, 1, 1, TD, GLOBAL_DEV, 0.5, 0, None),          # short segments at an odd pitch: the most keys of each form
    (2049, 1, 1, 1, ED, LOCAL_DEV, 0.5, 0, None),
    (1365, 3, 2, 1, ED, LOCAL_DEV, 0.6, 1, None),
    (585, 7, 2, 1, TD, GLOBAL_DEV, 0.6, 0, "few"),
    (587, 7, 2, 1, TD, GLOBAL_DEV, 0.6, 0, "few"),
])
def test_plan_segments_of_many_blocks(orc, n, e, k, g, mode, scope, gamma, metric, ties):
    """Segments with more keys than one block holds: thresholds from shared histograms, counts per expert, ties."""
    rng = np.random.default_rng(n + e)
    logits = rng.standard_normal((n, e)).astype(np.float32)
    if ties == "flat":
        logits[:] = 0.0
    elif ties == "few":
        logits = rng.integers(-1, 2, size=(n, e)).astype(np.float32)
    classes = rng.integers(0, 2, size=n).astype(np.uint8) if metric == 3 else None
    check_route_and_plan(orc, logits, n, e, k, g, mode, scope, gamma, f"many blocks {n}x{e}", metric, classes, 5)


@pytest.mark.parametrize("n,e,k,g,mode,scope,gamma", [
    (32768, 6, 2, 1, TD, GLOBAL, 0.7),      # eight parts of a segment: the blocks of a part share an XCD
    (36864, 6, 2, 8, ED, LOCAL, 0.7),       # two parts, eight blocks of tokens
    (65536, 3, 1, 1, TD, GLOBAL, 0.7),      # sixteen parts: the parts of a segment are neighbours
    (73728, 2, 1, 2, TD, LOCAL, 0.7),       # nine parts of each of two blocks
])
def test_plan_block_orders_of_the_emit(orc, n, e, k, g, mode, scope, gamma):
    if e % g:
        e *= g
    logits = np.random.default_rng(n + e).standard_normal((n, e)).astype(np.float32)
    check_route_and_plan(orc, logits, n, e, k, g, mode, scope, gamma, f"emit order {n}x{e}")


def tied_logits(rng, n, e, ties):
    logits = rng.standard_normal((n, e)).astype(np.float32)
    if ties == "flat":
        logits[:] = 0.0
    elif ties == "few":
        logits = rng.integers(-1, 2, size=(n, e)).astype(np.float32)
    elif ties == "pad":      # a quarter of the tokens alike, all over the batch
        logits[rng.random(n) < 0.25] = logits[0]
    elif ties == "padend":   # the same at its end
        logits[n - n // 4:] = logits[0]
    return logits


@pytest.mark.parametrize("n,e,k,g,mode,scope,gamma,metric,ties", [
    (6144, 32, 4, 1, TD, GLOBAL_DEV, 0.5, 0, "flat"),     # the budget ends with the last pair of a piece of 1024 tokens
    (6145, 32, 4, 1, ED, GLOBAL_DEV, 0.5, 0, "flat"),     # inside one; odd pitch, every expert a candidate
    (20000, 16, 2, 2, ED, LOCAL_DEV, 0.4, 0, "pad"),
    (20002, 16, 2, 2, ED, LOCAL_DEV, 0.4, 0, "padend"),
    (9000, 64, 2, 4, ED, GLOBAL_DEV, 0.6, 0, "few"),
    (700, 200, 8, 1, ED, GLOBAL_DEV, 0.3, 0, "few"),      # a single ragged piece, more experts than a wave
    (5000, 32, 4, 1, ED, GLOBAL_DEV, 0.7, 1, None),       # Order: every key of a token is equal
    (70004, 3, 2, 1, TD, GLOBAL, 0.4, 0, "pad"),          # single experts: the first equal keys in token order
    (41001, 2, 1, 1, TD, GLOBAL, 0.4, 0, "flat"),
    (98308, 3, 2, 1, TD, GLOBAL, 0.4, 0, "pad"),          # the same in segments that blocks share
    (98305, 2, 1, 1, TD, GLOBAL, 0.4, 0, "flat"),
    (98309, 47, 2, 1, TD, GLOBAL, 0.4, 0, "few"),
])
def test_plan_ties_in_segments_of_many_blocks(orc, n, e, k, g, mode, scope, gamma, metric, ties):
    """More keys equal the threshold than a segment has room for, spread over all of it."""
    logits = tied_logits(np.random.default_rng(n + e), n, e, ties)
    check_route_and_plan(orc, logits, n, e, k, g, mode, scope, gamma, f"ties {n}x{e} {ties}", metric)
    if n * e > 1 << 22:
        return
    check_route_and_plan(orc, logits, n, e, k, g, mode, scope, gamma, f"ties {n}x{e} {ties}, at most k", metric, None, 0,
                         min(2, e - k), True)


@pytest.mark.parametrize("n,e,k,g,mode,scope,gamma", [
    (65540, 4, 2, 1, NONE, GLOBAL, 1.0),        # no drop
    (4500, 32, 4, 1, NONE, GLOBAL_DEV, 1.0),
    (33333, 3, 2, 1, TD, GLOBAL, math.inf),     # odd pitch
    (4097, 32, 3, 1, ED, LOCAL_DEV, 50.0),      # a budget that holds every key of the segment
])
def test_plan_long_segments_with_room_for_all(orc, n, e, k, g, mode, scope, gamma):
    """Segments of many blocks whose capacity every candidate fits: counts only."""
    logits = np.random.default_rng(n + e).standard_normal((n, e)).astype(np.float32)
    check_route_and_plan(orc, logits, n, e, k, g, mode, scope, gamma, f"room for all {n}x{e}")
    check_route_and_plan(orc, logits, n, e, k, g, mode, scope, gamma, f"room for all {n}x{e}, at most k", 0, None, 0, 1, True)


@pytest.mark.parametrize("n,e,k,g,mode,scope,gamma,ties", [
    (65540, 66, 2, 1, TD, GLOBAL, 0.5, None),       # more segments than are shared among blocks
    (65540, 66, 2, 1, TD, GLOBAL, 0.5, "few"),
    (131088, 34, 2, 2, ED, LOCAL, 0.5, "pad"),      # 68 of them in two blocks of tokens
    (32771, 3, 1, 1, TD, GLOBAL, 0.4, None),        # odd pitch: a few, just too long to be held
    (40961, 2, 1, 1, TD, GLOBAL, 0.4, None),
    (40959, 2, 1, 1, TD, GLOBAL, 0.4, "flat"),
    (41001, 65, 3, 1, TD, GLOBAL, 0.7, None),
    (98304, 3, 1, 1, TD, GLOBAL, 0.4, "few"),       # the most keys that are not shared,
    (98305, 48, 2, 1, TD, GLOBAL, 0.5, None),       # and the fewest segments of more
])
def test_plan_segments_read_in_every_pass(orc, n, e, k, g, mode, scope, gamma, ties):
    """Long segments of single experts that one block each selects from."""
    logits = tied_logits(np.random.default_rng(n + e), n, e, ties)
    check_route_and_plan(orc, logits, n, e, k, g, mode, scope, gamma, f"re-read {n}x{e} {ties}")
    if n < 65540:
        check_route_and_plan(orc, logits, n, e, k, g, mode, scope, gamma, f"re-read {n}x{e}, at most k", 0, None, 0, 1, True)


def test_device_level_ties(orc):
    w = synth.scaled(W["olmoe"], n_tokens=2048, n_experts=32, top_k=4, device_groups=4)
    logits = synth.logits_with_ties(w)
    for scope in (LOCAL_DEV, GLOBAL_DEV):
        for mode in (TD, ED):
            check_route_and_plan(orc, logits, w.n_tokens, w.n_experts, w.top_k, 4, mode, scope, 1.0, "device ties")
    flat = np.zeros((512, 16), np.float32)     # every score equal: the tie rule alone decides
    check_route_and_plan(orc, flat, 512, 16, 2, 4, TD, LOCAL_DEV, 0.5, "device ties flat")
    check_route_and_plan(orc, flat, 512, 16, 2, 4, ED, GLOBAL_DEV, 0.5, "device ties flat")


# ------------------------------------------------------------------------------------------------
# over-selected candidate lists and at most k experts per token (appendix "Maximum Number of Selected Experts")
# ------------------------------------------------------------------------------------------------
@pytest.mark.parametrize("name,mode,scope,gamma,m_factor,limit", [
    ("olmoe", TD, LOCAL, 1.0, 2, False), ("olmoe", TD, LOCAL, 1.0, 2, True), ("olmoe", TD, LOCAL, 1.0, 3, True),
    ("olmoe", NONE, LOCAL, 1.0, 2, True), ("mixtral", ED, LOCAL, 1.0, 0, True), ("mixtral", TD, GLOBAL, 1.0, 2, True),
    ("finegrained", ED, LOCAL, 1.0, 0, True), ("finegrained", ED, LOCAL, 1.25, 1, True),
    ("finegrained", TD, LOCAL_DEV, 1.0, 2, True), ("decode", ED, LOCAL, 1.0, 2, True),
    ("decode", TD, GLOBAL_DEV, 1.0, 3, False),
])
def test_plan_overselection_and_max_k(orc, name, mode, scope, gamma, m_factor, limit):
    w = W[name]
    if name not in _logit_cache:
        _logit_cache[name] = oracle_logits(orc, w)
    m = m_factor * w.top_k
    buf, ref = check_route_and_plan(orc, _logit_cache[name], w.n_tokens, w.n_experts, w.top_k, w.device_groups, mode,
                                    scope, gamma, f"{name} overselect {m} limit {limit}", 0, None, 0, m, limit)
    per_token = ref.keep.sum(1)
    if limit:
        assert per_token.max() <= w.top_k
    elif mode != NONE:
        assert per_token.max() > w.top_k


def test_max_k_edge_cases(orc):
    flat = np.zeros((256, 16), np.float32)      # every score equal: expert ids and token order decide everything
    check_route_and_plan(orc, flat, 256, 16, 2, 4, ED, LOCAL, 2.0, "max-k flat", 0, None, 0, 4, True)
    check_route_and_plan(orc, flat, 256, 16, 2, 1, TD, GLOBAL, math.inf, "max-k flat no cap", 0, None, 0, 14, True)
    w = synth.scaled(W["olmoe"], n_tokens=2048, n_experts=32, top_k=4, device_groups=4)
    ties = synth.logits_with_ties(w)
    for mode, scope in [(ED, LOCAL), (ED, GLOBAL), (TD, LOCAL_DEV)]:
        check_route_and_plan(orc, ties, 2048, 32, 4, 4, mode, scope, 1.0, "max-k ties", 0, None, 0, 8, True)
    # other metrics rank the drop, the gating score still ranks which k experts a token keeps
    cls = (np.arange(2048) % 3 == 0).astype(np.uint8)
    check_route_and_plan(orc, ties, 2048, 32, 4, 4, ED, LOCAL, 0.75, "max-k order metric", 1, cls, 0, 4, True)
    check_route_and_plan(orc, ties, 2048, 32, 4, 4, ED, LOCAL, 0.75, "max-k random metric", 3, None, 11, 4, True)
    # a ragged token count and the largest candidate lists
    rng = np.random.default_rng(5)
    lg = rng.standard_normal((77, 64)).astype(np.float32)
    check_route_and_plan(orc, lg, 77, 64, 8, 1, TD, GLOBAL, 1.0, "max-k wide lists", 0, None, 0, 56, True)
    check_route_and_plan(orc, lg[:3], 3, 64, 8, 1, ED, GLOBAL, math.inf, "max-k three tokens", 0, None, 0, 8, True)


def test_plan_random_option_mix(orc):
    """Random combinations of every option (mode, scope, gamma, metric, classes, seed, over-selection, the
    per-token limit) on random shapes, half of them with few distinct logit values (ties everywhere)."""
    rng = np.random.default_rng(2025)
    for trial in range(48):
        g = int(rng.choice([1, 2, 4, 8]))
        mloc = int(rng.choice([1, 2, 4, 8]))
        e = g * mloc
        n = g * int(rng.integers(1, 160))
        k = int(rng.integers(1, min(e, 8) + 1))
        m_over = int(rng.integers(0, min(e - k, 12) + 1)) if rng.random() < 0.4 else 0
        mode = int(rng.choice([NONE, TD, ED]))
        scope = int(rng.integers(0, 4))
        gamma = float(rng.choice([0.0, 0.3, 0.5, 1.0, 1.3, 2.0, math.inf]))
        metric = int(rng.integers(0, 4))
        classes = rng.integers(0, 4, n).astype(np.uint8) if rng.random() < 0.4 else None
        seed = int(rng.integers(1, 1000)) if metric == 3 or rng.random() < 0.3 else 0
        limit = bool(rng.random() < 0.4)
        if trial % 2:
            logits = rng.integers(-3, 4, (n, e)).astype(np.float32) * 0.5
        else:
            logits = (rng.standard_normal((n, e)) * 2).astype(np.float32)
        check_route_and_plan(orc, logits, n, e, k, g, mode, scope, gamma, f"mix {trial}", metric, classes, seed, m_over,
                             limit)


def test_random_metric_ties_and_seeds(orc):
    n, e = 1024, 8
    logits = np.zeros((n, e), np.float32)           # all scores equal: only the draws decide
    a, _ = check_route_and_plan(orc, logits, n, e, 2, 1, TD, GLOBAL, 0.5, "random flat", 3, None, 1)
    b, _ = check_route_and_plan(orc, logits, n, e, 2, 1, TD, GLOBAL, 0.5, "random flat", 3, None, 2)
    assert not torch.equal(a.row_token, b.row_token)


def test_peaked_logits_zero_scores(orc):
    # scores that underflow to exactly 0 are still ranked as candidates
    n, e = 256, 16
    logits = np.zeros((n, e), np.float32)
    logits[:, 3] = 300.0
    check_route_and_plan(orc, logits, n, e, 2, 1, TD, GLOBAL, 1.0, "peaked")
    check_route_and_plan(orc, logits, n, e, 2, 4, ED, LOCAL, 1.0, "peaked expanded")


def test_empty_batch():
    desc = capmoe.make_desc(0, 64, 8, 2, 128, 1, TD, GLOBAL, 1.0, synth.DTYPE_F32)
    buf = route_and_drop_gpu(desc, np.zeros((0, 8), np.float32))
    assert buf.expert_count.cpu().numpy().sum() == 0 and buf.expert_offset.cpu().numpy().max() == 0
    capmoe.moe_dispatch(desc, buf.xp, buf.expert_offset, buf.row_token, buf.xp)
    capmoe.moe_combine(desc, buf.yp, buf.row_weight, buf.pair_row, buf.y)
    torch.cuda.synchronize()


def test_workspace_too_small_is_refused():
    desc = capmoe.make_desc(128, 64, 8, 2, 128, 1, TD, GLOBAL, 1.0, synth.DTYPE_F32)
    buf = capmoe.LayerBuffers(desc)
    small = torch.empty(256, dtype=torch.uint8, device="cuda")
    with pytest.raises(capmoe.CapMoeError) as ei:
        capmoe.moe_capacity_drop(desc, buf.scores, buf.topk_idx, buf.expert_count, buf.seg_count, buf.expert_offset,
                                 buf.row_token, buf.row_weight, buf.pair_row, small)
    assert ei.value.status == 3
    with pytest.raises(capmoe.CapMoeError) as ei:
        capmoe.moe_grouped_ffn(desc, buf.xp, buf.expert_offset, buf.xp, buf.xp, buf.xp, buf.yp, small)
    assert ei.value.status == 3
    bad = capmoe.make_desc(128, 200, 8, 2, 128, 1, TD, GLOBAL, 1.0, synth.DTYPE_BF16)   # d not a multiple of 128
    with pytest.raises(capmoe.CapMoeError) as ei:
        capmoe.moe_grouped_ffn(bad, buf.xp, buf.expert_offset, buf.xp, buf.xp, buf.xp, buf.yp, buf.workspace)
    assert ei.value.status == 2


# ------------------------------------------------------------------------------------------------
# whole layer
# ------------------------------------------------------------------------------------------------
def run_layer(layer: DeviceLayer, desc, logits_host=None):
    buf = capmoe.LayerBuffers(desc)
    given = torch.from_numpy(logits_host).cuda() if logits_host is not None else None
    capmoe.layer_forward(buf, layer.x, layer.w_router, layer.bias, layer.w_gate, layer.w_up, layer.w_down, given)
    torch.cuda.synchronize()
    return buf


def check_layer(orc, layer, mode, scope, gamma, tokens=None, what="", overselect=0, max_experts=False):
    w = layer.w
    note("layer", what, w.name, dict(mode=mode, scope=scope, gamma=gamma, overselect=overselect, max_experts=max_experts))
    logits = orc.router_logits(layer.x_host, layer.w_router_host, layer.bias_host)
    ref = orc.route_and_drop(logits, w.top_k, w.device_groups, mode, scope, gamma, overselect=overselect,
                             max_experts=max_experts)
    desc = layer.desc(mode, scope, gamma)
    desc.overselect, desc.max_experts = overselect, int(max_experts)
    buf = run_layer(layer, desc, logits)
    assert_plan_equal(buf, ref, what)
    rows = ref.plan.rows
    # permutation: rows of xp are the rows of x named by the plan, bit for bit
    xp = buf.xp[:rows].view(torch.int16 if w.dtype == synth.DTYPE_BF16 else torch.int32).cpu().numpy()
    xsrc = layer.x.view(torch.int16 if w.dtype == synth.DTYPE_BF16 else torch.int32).cpu().numpy()
    np.testing.assert_array_equal(xp, xsrc[ref.plan.row_token])
    y_ref = orc.layer_output(layer.x_host, ref.scores, ref.keep, layer.host_gate, layer.host_up, layer.host_down,
                             token_list=tokens)
    y = to_host_f64(buf.y)
    if tokens is not None:
        y = y[tokens]
    assert np.all(np.isfinite(to_host_f64(buf.y)))
    assert_output_close(y, y_ref, TOL[w.dtype], what)
    # dispatch fused into the first GEMM (moe_dispatch_ffn): same bits as the two separate calls
    fused = capmoe.LayerBuffers(desc)
    capmoe.layer_forward(fused, layer.x, layer.w_router, layer.bias, layer.w_gate, layer.w_up, layer.w_down,
                         torch.from_numpy(logits).cuda(), fused_dispatch=True)
    torch.cuda.synchronize()
    assert torch.equal(fused.yp[:rows], buf.yp[:rows]) and torch.equal(fused.y, buf.y)
    return buf, ref


def test_one_call_entry_matches_separate_calls():
    """moe_layer_forward enqueues the same work as the four calls (the tile schedule of the expert GEMMs comes out of
    the drop's last launch instead of a kernel of its own): every output equal bit for bit."""
    cases = [(synth.scaled(W["tiny"], device_groups=4), ED, LOCAL, 1.0, 0, False),
             (synth.scaled(W["olmoe"], name="reduced", n_tokens=640, d_model=256, n_experts=8, top_k=2, d_hidden=384,
                           device_groups=4, skew="normal", skew_param=1.5), TD, LOCAL, 1.0, 2, True),
             (synth.scaled(W["olmoe"], name="reduced", n_tokens=300, d_model=384, n_experts=4, top_k=2, d_hidden=256,
                           device_groups=1), TD, GLOBAL, 0.0, 0, False),
             # many experts, narrow hidden layer: the drop's workspace reaches past the place of the GEMMs' tile
             # schedule, so the schedule kernel runs as in the separate calls
             (synth.scaled(W["olmoe"], name="reduced", n_tokens=512, d_model=128, n_experts=64, top_k=1, d_hidden=128,
                           device_groups=1), TD, GLOBAL, 2.0, 0, False),
             # long segments: the three-kernel drop, whose last launch builds the schedule
             (synth.scaled(W["olmoe"], name="reduced", n_tokens=9000, d_model=128, n_experts=8, top_k=2, d_hidden=256,
                           device_groups=1), TD, GLOBAL, 1.0, 0, False),
             (synth.scaled(W["olmoe"], name="reduced", n_tokens=9000, d_model=128, n_experts=12, top_k=3, d_hidden=128,
                           device_groups=3), ED, GLOBAL, 0.9, 3, True),
             # a budget over 131200 keys, shared among blocks: its workspace, with the schedule from the drop and (many
             # experts, one row per token) without
             (synth.scaled(W["olmoe"], name="reduced", n_tokens=4100, d_model=128, n_experts=32, top_k=4, d_hidden=128,
                           device_groups=1), TD, GLOBAL_DEV, 0.7, 0, False),
             (synth.scaled(W["olmoe"], name="reduced", n_tokens=2052, d_model=128, n_experts=128, top_k=1, d_hidden=128,
                           device_groups=1), TD, GLOBAL_DEV, 0.7, 1, True)]
    for w, mode, scope, gamma, m, limit in cases:
        layer = DeviceLayer(w, host_weights=False)
        desc = layer.desc(mode, scope, gamma)
        desc.overselect, desc.max_experts, desc.metric = m, int(limit), 3 if limit else 0
        cls = torch.from_numpy((np.arange(w.n_tokens) % 2).astype(np.uint8)).cuda() if limit else None
        seed = 9 if limit else 0
        a, b = capmoe.LayerBuffers(desc), capmoe.LayerBuffers(desc)
        capmoe.layer_forward(a, layer.x, layer.w_router, layer.bias, layer.w_gate, layer.w_up, layer.w_down,
                             fused_dispatch=True, token_class=cls, seed=seed)
        capmoe.moe_layer_forward(desc, layer.x, layer.w_router, layer.bias, layer.w_gate, layer.w_up, layer.w_down,
                                 cls, seed, b)
        torch.cuda.synchronize()
        rows = int(a.expert_offset[-1])
        assert rows == int(b.expert_offset[-1])
        for name in ("logits", "scores", "topk_idx", "topk_score", "expert_count", "seg_count", "expert_offset",
                     "pair_row", "y"):
            assert torch.equal(getattr(a, name), getattr(b, name)), name
        assert torch.equal(a.row_token[:rows], b.row_token[:rows]) and torch.equal(a.yp[:rows], b.yp[:rows])
        assert torch.equal(a.row_weight[:rows].view(torch.int32), b.row_weight[:rows].view(torch.int32))


def test_layer_tiny_fp32(orc):
    layer = DeviceLayer(W["tiny"])
    for mode, scope, gamma in [(NONE, LOCAL, 1.0), (TD, LOCAL, 1.0), (TD, LOCAL, 0.5), (TD, LOCAL, math.inf)]:
        check_layer(orc, layer, mode, scope, gamma, what="tiny")
    layer4 = DeviceLayer(synth.scaled(W["tiny"], device_groups=4))
    for scope in (LOCAL, GLOBAL):
        check_layer(orc, layer4, ED, scope, 1.0, what="tiny expanded")


@pytest.mark.parametrize("n,d,e,k,h,g", [(640, 256, 8, 2, 384, 4), (1536, 128, 16, 4, 128, 2), (300, 384, 4, 2, 256, 1)])
def test_layer_reduced_bf16(orc, n, d, e, k, h, g):
    # several row tiles per expert with ragged tails, several column tiles, empty experts possible
    w = synth.scaled(W["olmoe"], name="reduced", n_tokens=n, d_model=d, n_experts=e, top_k=k, d_hidden=h,
                     device_groups=g, skew="normal", skew_param=1.5)
    layer = DeviceLayer(w)
    for mode, scope, gamma in [(NONE, LOCAL, 1.0), (TD, LOCAL, 1.0), (ED, LOCAL, 1.0), (ED, GLOBAL, 1.5),
                               (TD, GLOBAL, 0.0)]:
        check_layer(orc, layer, mode, scope, gamma, what="reduced bf16")
    if e >= 8:   # over-selected lists, with and without the limit of k experts per token
        check_layer(orc, layer, TD, LOCAL, 1.0, what="reduced bf16 overselect", overselect=2 * k)
        check_layer(orc, layer, ED, LOCAL, 1.0, what="reduced bf16 w/ max", overselect=k, max_experts=True)


def test_ffn_ragged_expert_sizes(orc):
    # expert row counts around the tile height: 0, 1, 127, 128, 129, 300, 5, 0
    counts = [0, 1, 127, 128, 129, 300, 5, 0]
    e, n = len(counts), sum(counts)
    w = synth.scaled(W["olmoe"], name="ragged", n_tokens=n, d_model=256, n_experts=e, top_k=1, d_hidden=256,
                     device_groups=1)
    layer = DeviceLayer(w)
    owner = np.repeat(np.arange(e), counts)
    np.random.default_rng(5).shuffle(owner)
    logits = np.zeros((n, e), np.float32)
    logits[np.arange(n), owner] = 6.0
    ref = orc.route_and_drop(logits, 1, 1, NONE, GLOBAL, 1.0)
    np.testing.assert_array_equal(ref.plan.expert_count, counts)
    buf = run_layer(layer, layer.desc(NONE, GLOBAL, 1.0), logits)
    assert_plan_equal(buf, ref, "ragged")
    y_ref = orc.layer_output(layer.x_host, ref.scores, ref.keep, layer.host_gate, layer.host_up, layer.host_down)
    assert_output_close(to_host_f64(buf.y), y_ref, TOL[w.dtype], "ragged")


def test_ffn_nearly_empty_last_round(orc):
    """67 full-height row tiles x 4 column blocks of the down GEMM = 268 work items on 256 compute units: a last
    round of 12 items (K is short here, so they stay whole)."""
    counts = [40 * 256 + 30, 20 * 256, 6 * 256 + 100, 17]
    e, n = len(counts), sum(counts)
    w = synth.scaled(W["olmoe"], name="tail", n_tokens=n, d_model=1024, n_experts=e, top_k=1, d_hidden=256,
                     device_groups=1)
    layer = DeviceLayer(w)
    owner = np.repeat(np.arange(e), counts)
    np.random.default_rng(9).shuffle(owner)
    logits = np.zeros((n, e), np.float32)
    logits[np.arange(n), owner] = 6.0
    ref = orc.route_and_drop(logits, 1, 1, NONE, GLOBAL, 1.0)
    np.testing.assert_array_equal(ref.plan.expert_count, counts)
    buf = run_layer(layer, layer.desc(NONE, GLOBAL, 1.0), logits)
    assert_plan_equal(buf, ref, "tail")
    y_ref = orc.layer_output(layer.x_host, ref.scores, ref.keep, layer.host_gate, layer.host_up, layer.host_down)
    assert_output_close(to_host_f64(buf.y), y_ref, TOL[w.dtype], "tail")


@pytest.mark.parametrize("d,h,counts", [
    (128, 8192, [5 * 256 + 70, 3 * 256, 40]),        # down GEMM: 128 K slabs, 128-column output tiles, 9 big items and one short
    (256, 8192, [256, 300, 17, 0, 2 * 256 + 64]),    # 256-column output tiles; two short items
    (8192, 128, [700, 64]),                          # gate/up GEMM with 128 K slabs: SwiGLU tiles are cut
])
def test_ffn_items_cut_along_k(orc, d, h, counts):
    """Work items left over after the last full round of a long-K GEMM run as several units, each over a share of
    the K slabs, and the unit that finishes last adds the partial tiles in slice order: with so few items every
    one of them is cut (eight units each).  Same tolerance as whole items, and the same bits on every run."""
    e, n = len(counts), sum(counts)
    w = synth.scaled(W["olmoe"], name="cut", n_tokens=n, d_model=d, n_experts=e, top_k=1, d_hidden=h, device_groups=1)
    layer = DeviceLayer(w)
    owner = np.repeat(np.arange(e), counts)
    np.random.default_rng(21).shuffle(owner)
    logits = np.zeros((n, e), np.float32)
    logits[np.arange(n), owner] = 6.0
    ref = orc.route_and_drop(logits, 1, 1, NONE, GLOBAL, 1.0)
    np.testing.assert_array_equal(ref.plan.expert_count, counts)
    desc = layer.desc(NONE, GLOBAL, 1.0)
    buf = run_layer(layer, desc, logits)
    assert_plan_equal(buf, ref, "cut")
    y_ref = orc.layer_output(layer.x_host, ref.scores, ref.keep, layer.host_gate, layer.host_up, layer.host_down)
    assert_output_close(to_host_f64(buf.y), y_ref, TOL[w.dtype], "cut along K")
    for _ in range(3):
        again = run_layer(layer, desc, logits)
        assert torch.equal(again.yp[:n], buf.yp[:n]) and torch.equal(again.y, buf.y)
    fused = capmoe.LayerBuffers(desc)
    capmoe.layer_forward(fused, layer.x, layer.w_router, layer.bias, layer.w_gate, layer.w_up, layer.w_down,
                         torch.from_numpy(logits).cuda(), fused_dispatch=True)
    torch.cuda.synchronize()
    assert torch.equal(fused.y, buf.y)


@pytest.mark.parametrize("d,h,counts", [
    # gate/up: 32 column blocks x 74 tiles = 9.2 rounds on 256 compute units -> joint list; down: 74 items, two lists
    (128, 4096, [1000, 30, 300, 64, 2000, 5, 700, 0, 3000, 61, 4500, 257, 11 * 256 + 63, 2300]),
    # both GEMMs at 4 column blocks x 525 tiles = 8.2 rounds: both walk the joint list
    (1024, 512, [156 * 256 + 64, 17, 35 * 256 + 50, 0, 25000, 64, 117 * 256 + 51, 700, 1, 109 * 256 + 62]),
    # seven column blocks (column groups of one): 298 tiles x 7 = 8.1 rounds in gate/up
    (128, 896, [30010, 17, 25040, 20064, 300]),
])
def test_ffn_joint_tile_list(orc, d, h, counts):
    """A GEMM that is never cut along K and is at least eight rounds of work items long walks one list that holds
    the big and the short row tiles expert by expert.  Experts with only a short tile, with big tiles and a short
    remainder, with a partly filled big tile, and an empty one: every token against the oracle (Eq. 2)."""
    e, n = len(counts), sum(counts)
    w = synth.scaled(W["olmoe"], name="joint", n_tokens=n, d_model=d, n_experts=e, top_k=1, d_hidden=h, device_groups=1)
    layer = DeviceLayer(w)
    owner = np.repeat(np.arange(e), counts)
    np.random.default_rng(33).shuffle(owner)
    logits = np.zeros((n, e), np.float32)
    logits[np.arange(n), owner] = 6.0
    ref = orc.route_and_drop(logits, 1, 1, NONE, GLOBAL, 1.0)
    np.testing.assert_array_equal(ref.plan.expert_count, counts)
    desc = layer.desc(NONE, GLOBAL, 1.0)
    buf = run_layer(layer, desc, logits)
    assert_plan_equal(buf, ref, "joint")
    y_ref = orc.layer_output(layer.x_host, ref.scores, ref.keep, layer.host_gate, layer.host_up, layer.host_down)
    assert_output_close(to_host_f64(buf.y), y_ref, TOL[w.dtype], "joint tile list")
    fused = capmoe.LayerBuffers(desc)
    capmoe.layer_forward(fused, layer.x, layer.w_router, layer.bias, layer.w_gate, layer.w_up, layer.w_down,
                         torch.from_numpy(logits).cuda(), fused_dispatch=True)
    torch.cuda.synchronize()
    assert torch.equal(fused.y, buf.y)


@pytest.mark.parametrize("d,h", [(128, 128), (384, 640), (1024, 256)])
def test_ffn_single_tile_experts(orc, d, h):
    """Experts with one row tile stream their weights with a walk over K that starts at another slab for every column
    block: short and partly filled big tiles at their edges, beside experts with several tiles, from two slabs of K
    up.  Every token against the oracle (Eq. 2), and the same bits with the gather fused into the first GEMM."""
    counts = [1, 63, 64, 65, 130, 255, 256, 257, 320, 321, 0, 33]
    e, n = len(counts), sum(counts)
    w = synth.scaled(W["olmoe"], name="alone", n_tokens=n, d_model=d, n_experts=e, top_k=1, d_hidden=h, device_groups=1)
    layer = DeviceLayer(w)
    owner = np.repeat(np.arange(e), counts)
    np.random.default_rng(35).shuffle(owner)
    logits = np.zeros((n, e), np.float32)
    logits[np.arange(n), owner] = 6.0
    ref = orc.route_and_drop(logits, 1, 1, NONE, GLOBAL, 1.0)
    np.testing.assert_array_equal(ref.plan.expert_count, counts)
    desc = layer.desc(NONE, GLOBAL, 1.0)
    buf = run_layer(layer, desc, logits)
    y_ref = orc.layer_output(layer.x_host, ref.scores, ref.keep, layer.host_gate, layer.host_up, layer.host_down)
    assert_output_close(to_host_f64(buf.y), y_ref, TOL[w.dtype], "single-tile experts")
    fused = capmoe.LayerBuffers(desc)
    capmoe.layer_forward(fused, layer.x, layer.w_router, layer.bias, layer.w_gate, layer.w_up, layer.w_down,
                         torch.from_numpy(logits).cuda(), fused_dispatch=True)
    torch.cuda.synchronize()
    assert torch.equal(fused.y, buf.y)


@pytest.mark.parametrize("d,h", [(2048, 2432), (2432, 2048)])
def test_ffn_single_tile_experts_of_a_large_layer(orc, d, h):
    """As above with more expert weights (359 MB) than the memory-side cache holds, where such experts stream them: the first
    and the last row of every row tile against the oracle, and the same bits with the fused gather."""
    counts = [1, 63, 64, 65, 130, 255, 256, 257, 320, 321, 0, 33]
    e, n = len(counts), sum(counts)
    w = synth.scaled(W["olmoe"], name="alone, large", n_tokens=n, d_model=d, n_experts=e, top_k=1, d_hidden=h, device_groups=1)
    layer = DeviceLayer(w)
    owner = np.repeat(np.arange(e), counts)
    np.random.default_rng(39).shuffle(owner)
    logits = np.zeros((n, e), np.float32)
    logits[np.arange(n), owner] = 6.0
    ref = orc.route_and_drop(logits, 1, 1, NONE, GLOBAL, 1.0)
    desc = layer.desc(NONE, GLOBAL, 1.0)
    buf = run_layer(layer, desc, logits)
    tokens = sorted({int(np.flatnonzero(owner == j)[r]) for j in range(e) if counts[j]
                     for first in range(0, counts[j], 64) for r in (first, min(first + 63, counts[j] - 1))})
    y_ref = orc.layer_output(layer.x_host, ref.scores, ref.keep, layer.host_gate, layer.host_up, layer.host_down, tokens)
    assert_output_close(to_host_f64(buf.y)[tokens], y_ref, TOL[w.dtype], "single-tile experts of a large layer")
    fused = capmoe.LayerBuffers(desc)
    capmoe.layer_forward(fused, layer.x, layer.w_router, layer.bias, layer.w_gate, layer.w_up, layer.w_down,
                         torch.from_numpy(logits).cuda(), fused_dispatch=True)
    torch.cuda.synchronize()
    assert torch.isfinite(buf.y.float()).all() and torch.equal(fused.y, buf.y)


@pytest.mark.parametrize("d,h,counts", [
    (4, 1, [1, 0, 5]),                                    # less than one K slab in both products, a single hidden column
    (64, 33, [16, 17, 64, 65, 1, 0, 31, 48, 49, 130]),    # edges of sub-tiles and tiles; the down product has K = 33
    (100, 97, [32, 33, 63, 128, 129, 2]),                 # rows whose pitch is no multiple of 16 bytes
    (160, 250, [300, 7, 200]),                            # several tiles per expert: four-wave blocks
    (36, 1000, [3, 40, 0, 90, 64, 64]),
    (1024, 31, [3, 1, 12]),
    (84, 7, [16, 17, 100, 0, 31, 160, 33, 72]),           # a block per 16-row piece: whole, ragged and empty ones
    (100, 97, [17, 33, 50, 64] + [0] * 20 + [3]),         # few rows on average: one-wave blocks of two, three and four sub-tiles
    (1024, 250, [17, 33, 50, 64] + [0] * 20 + [3]),
    (260, 1030, [20, 40, 60] + [5] * 13),                 # the same where many column blocks keep the tiles whole
])
def test_ffn_fp32_shapes(orc, d, h, counts):
    """The fp32 expert products at the edges of their tiles, column blocks and K slabs, permuted rows and fused gather.
    Both products are fp32 sums of at most 1024 terms: their relative error in the 2-norm is about sqrt(K) 2^-24 < 2e-6."""
    e, n = len(counts), sum(counts)
    w = synth.scaled(W["tiny"], name="f32 shapes", n_tokens=n, d_model=d, n_experts=e, top_k=1, d_hidden=h, device_groups=1)
    layer = DeviceLayer(w)
    owner = np.repeat(np.arange(e), counts)
    np.random.default_rng(36).shuffle(owner)
    logits = np.zeros((n, e), np.float32)
    logits[np.arange(n), owner] = 6.0
    ref = orc.route_and_drop(logits, 1, 1, NONE, GLOBAL, 1.0)
    np.testing.assert_array_equal(ref.plan.expert_count, counts)
    desc = layer.desc(NONE, GLOBAL, 1.0)
    buf = run_layer(layer, desc, logits)
    y_ref = orc.layer_output(layer.x_host, ref.scores, ref.keep, layer.host_gate, layer.host_up, layer.host_down)
    assert_output_close(to_host_f64(buf.y), y_ref, 1e-5, "fp32 shapes")
    fused = capmoe.LayerBuffers(desc)
    capmoe.layer_forward(fused, layer.x, layer.w_router, layer.bias, layer.w_gate, layer.w_up, layer.w_down,
                         torch.from_numpy(logits).cuda(), fused_dispatch=True)
    torch.cuda.synchronize()
    assert torch.equal(fused.y, buf.y)


@pytest.mark.parametrize("d,h", [(128, 128), (384, 640), (1024, 256), (256, 2048)])
@pytest.mark.parametrize("counts", [[1], [16, 0, 1, 15], [17, 1, 0, 30, 16], [33, 0, 0, 31], [0, 64, 0, 0],
                                    [30, 34, 0]])    # 21 rows on average: the narrow products only
def test_ffn_few_rows(orc, d, h, counts):
    """Batches of at most 64 tokens: one and two sub-tiles of 16 rows, tiles done in two passes, waves without a K slab
    (d = 128 has two slabs for four waves).  Every token against the oracle (Eq. 2), and the same bits with the gather
    fused into the first GEMM."""
    e, n = len(counts), sum(counts)
    w = synth.scaled(W["olmoe"], name="few rows", n_tokens=n, d_model=d, n_experts=e, top_k=1, d_hidden=h, device_groups=1)
    layer = DeviceLayer(w)
    owner = np.repeat(np.arange(e), counts)
    np.random.default_rng(37).shuffle(owner)
    logits = np.zeros((n, e), np.float32)
    logits[np.arange(n), owner] = 6.0
    ref = orc.route_and_drop(logits, 1, 1, NONE, GLOBAL, 1.0)
    np.testing.assert_array_equal(ref.plan.expert_count, counts)
    desc = layer.desc(NONE, GLOBAL, 1.0)
    buf = run_layer(layer, desc, logits)
    y_ref = orc.layer_output(layer.x_host, ref.scores, ref.keep, layer.host_gate, layer.host_up, layer.host_down)
    assert_output_close(to_host_f64(buf.y), y_ref, TOL[w.dtype], "few rows")
    fused = capmoe.LayerBuffers(desc)
    capmoe.layer_forward(fused, layer.x, layer.w_router, layer.bias, layer.w_gate, layer.w_up, layer.w_down,
                         torch.from_numpy(logits).cuda(), fused_dispatch=True)
    torch.cuda.synchronize()
    assert torch.equal(fused.y, buf.y)


@pytest.mark.parametrize("d,h,counts", [(2048, 3584, [1, 0, 16, 17, 0, 0, 30, 0]), (3584, 2048, [0, 33, 0, 15, 0, 0, 1, 2])])
def test_ffn_few_rows_of_a_large_layer(orc, d, h, counts):
    """As above with expert weights (352 MB) beyond what the memory-side cache keeps, which are streamed."""
    e, n = len(counts), sum(counts)
    w = synth.scaled(W["olmoe"], name="few rows, large", n_tokens=n, d_model=d, n_experts=e, top_k=1, d_hidden=h,
                     device_groups=1)
    layer = DeviceLayer(w)
    owner = np.repeat(np.arange(e), counts)
    np.random.default_rng(40).shuffle(owner)
    logits = np.zeros((n, e), np.float32)
    logits[np.arange(n), owner] = 6.0
    ref = orc.route_and_drop(logits, 1, 1, NONE, GLOBAL, 1.0)
    buf = run_layer(layer, layer.desc(NONE, GLOBAL, 1.0), logits)
    y_ref = orc.layer_output(layer.x_host, ref.scores, ref.keep, layer.host_gate, layer.host_up, layer.host_down)
    assert_output_close(to_host_f64(buf.y), y_ref, TOL[w.dtype], "few rows of a large layer")


@pytest.mark.parametrize("counts", [
    {0: 100, 1: 3, 5: 65, 31: 1},                  # above the capacity of a descriptor whose experts have 64 rows at most
    {3: 321, 7: 64, 8: 65, 20: 30},                # several full tiles and a remainder on one expert
    {e: 16 for e in range(32)},                    # every expert its average
    {31: 512},                                     # all rows on one expert
])
def test_ffn_plans_of_the_caller(orc, counts):
    """expert_offset is the caller's: an expert may hold more rows than the descriptor's own capacity would leave it (rows
    exchanged between devices, an edited plan), as long as all of them fit max_rows.  64 tokens, top-8 of 32 experts: a
    descriptor whose experts have few rows.  Every row against the oracle's SwiGLU, rows past the plan untouched."""
    e, n, k, d, h = 32, 64, 8, 256, 384
    w = synth.scaled(W["olmoe"], name="caller's plan", n_tokens=n, d_model=d, n_experts=e, top_k=k, d_hidden=h,
                     device_groups=1)
    layer = DeviceLayer(w)
    desc = layer.desc(NONE, GLOBAL, 1.0)
    max_rows, rows = capmoe.moe_query(desc)[2], sum(counts.values())
    assert rows <= max_rows == n * k
    per_expert = [counts.get(j, 0) for j in range(e)]
    offset = torch.from_numpy(np.concatenate([[0], np.cumsum(per_expert)]).astype(np.int32)).cuda()
    row_token = np.random.default_rng(38).integers(0, n, size=max_rows).astype(np.int32)
    tokens = torch.from_numpy(row_token).cuda()
    xp = layer.x[tokens.long()].contiguous()
    workspace = torch.empty(capmoe.moe_query(desc)[3], dtype=torch.uint8, device="cuda")
    separate = torch.full((max_rows, d), 7.0, dtype=torch.bfloat16, device="cuda")
    fused = separate.clone()
    capmoe.moe_grouped_ffn(desc, xp, offset, layer.w_gate, layer.w_up, layer.w_down, separate, workspace)
    capmoe.moe_dispatch_ffn(desc, layer.x, offset, tokens, layer.w_gate, layer.w_up, layer.w_down, fused, workspace)
    torch.cuda.synchronize()
    # the oracle's layer with one expert per row and weight one is that expert's FFN
    keep = np.zeros((rows, e), np.uint8)
    keep[np.arange(rows), np.repeat(np.arange(e), per_expert)] = 1
    ref = orc.layer_output(layer.x_host[row_token[:rows]], keep.astype(np.float32), keep, layer.host_gate, layer.host_up,
                           layer.host_down)
    assert_output_close(to_host_f64(separate[:rows]), ref, TOL[w.dtype], "caller's plan")
    assert (separate[rows:] == 7.0).all() and torch.equal(separate, fused)


@pytest.mark.parametrize("d,h", [(512, 1000), (100, 97), (1024, 256)])
def test_ffn_fp32_rows_do_not_depend_on_the_batch(d, h):
    """An fp32 token gets the same bits alone, in a batch of few rows (narrow column blocks) and in a larger one (wide ones)."""
    e, k = 8, 2
    big = synth.scaled(W["tiny"], name="batch", n_tokens=400, d_model=d, n_experts=e, top_k=k, d_hidden=h, device_groups=1)
    layer = DeviceLayer(big, host_weights=False)
    outs = {}
    for n in (400, 40, 1):
        desc = capmoe.make_desc(n, d, e, k, h, 1, NONE, GLOBAL, 1.0, synth.DTYPE_F32)
        buf = capmoe.LayerBuffers(desc)
        capmoe.layer_forward(buf, layer.x[:n].contiguous(), layer.w_router, layer.bias, layer.w_gate, layer.w_up,
                             layer.w_down)
        torch.cuda.synchronize()
        outs[n] = buf.y
    assert torch.equal(outs[40], outs[400][:40]) and torch.equal(outs[1], outs[400][:1])


def test_ffn_leftover_items_in_row_pieces(orc):
    """A GEMM too short in K to be cut there, with one big item per XCD left over after a full round (66 big
    tiles x 4 column blocks = 33 items per XCD): the leftover items run as four 64-row blocks each, the last of them
    on a partly filled tile (100 rows: a whole piece, a piece of 36 rows, two empty ones).  Every token against the
    oracle (Eq. 2), and the same bits with the gather fused into the first GEMM."""
    d, h = 128, 512
    counts = [20 * 256, 30 * 256 + 30, 0, 50, 15 * 256 + 100]
    e, n = len(counts), sum(counts)
    w = synth.scaled(W["olmoe"], name="pieces", n_tokens=n, d_model=d, n_experts=e, top_k=1, d_hidden=h, device_groups=1)
    layer = DeviceLayer(w)
    owner = np.repeat(np.arange(e), counts)
    np.random.default_rng(34).shuffle(owner)
    logits = np.zeros((n, e), np.float32)
    logits[np.arange(n), owner] = 6.0
    ref = orc.route_and_drop(logits, 1, 1, NONE, GLOBAL, 1.0)
    np.testing.assert_array_equal(ref.plan.expert_count, counts)
    desc = layer.desc(NONE, GLOBAL, 1.0)
    buf = run_layer(layer, desc, logits)
    assert_plan_equal(buf, ref, "row pieces")
    y_ref = orc.layer_output(layer.x_host, ref.scores, ref.keep, layer.host_gate, layer.host_up, layer.host_down)
    assert_output_close(to_host_f64(buf.y), y_ref, TOL[w.dtype], "row pieces")
    fused = capmoe.LayerBuffers(desc)
    capmoe.layer_forward(fused, layer.x, layer.w_router, layer.bias, layer.w_gate, layer.w_up, layer.w_down,
                         torch.from_numpy(logits).cuda(), fused_dispatch=True)
    torch.cuda.synchronize()
    assert torch.equal(fused.y, buf.y)


def test_ffn_many_experts(orc):
    """200 experts (the tile schedule walks them 64 at a time), most with a handful of rows, some empty, a few with
    several tiles."""
    rng = np.random.default_rng(77)
    counts = [int(c) for c in rng.choice([0, 1, 3, 17, 40, 64, 65, 130, 300, 520], size=200,
                                         p=[0.1, 0.1, 0.2, 0.2, 0.15, 0.05, 0.05, 0.05, 0.05, 0.05])]
    e, n = len(counts), sum(counts)
    w = synth.scaled(W["olmoe"], name="many", n_tokens=n, d_model=128, n_experts=e, top_k=1, d_hidden=128,
                     device_groups=1)
    layer = DeviceLayer(w)
    owner = np.repeat(np.arange(e), counts)
    rng.shuffle(owner)
    logits = np.zeros((n, e), np.float32)
    logits[np.arange(n), owner] = 9.0
    ref = orc.route_and_drop(logits, 1, 1, NONE, GLOBAL, 1.0)
    np.testing.assert_array_equal(ref.plan.expert_count, counts)
    buf = run_layer(layer, layer.desc(NONE, GLOBAL, 1.0), logits)
    assert_plan_equal(buf, ref, "many experts")
    y_ref = orc.layer_output(layer.x_host, ref.scores, ref.keep, layer.host_gate, layer.host_up, layer.host_down)
    assert_output_close(to_host_f64(buf.y), y_ref, TOL[w.dtype], "many experts")


@pytest.mark.parametrize("trial", range(5))
def test_ffn_random_expert_sizes(orc, trial):
    """Random row counts per expert (empty experts, 1 row, around every tile boundary, several tiles) and random
    widths: both tile kinds, partly filled tiles, both output-tile widths of the down GEMM."""
    rng = np.random.default_rng(300 + trial)
    e = int(rng.integers(1, 10))
    choices = [0, 1, 63, 64, 65, 128, 191, 192, 193, 255, 256, 257, 320, 383, 512, 600]
    counts = [int(rng.choice(choices)) for _ in range(e)]
    if sum(counts) == 0:
        counts[0] = 70
    d, h = int(rng.choice([128, 256, 384, 512])), int(rng.choice([128, 256, 640]))
    n = sum(counts)
    w = synth.scaled(W["olmoe"], name="ragged", n_tokens=n, d_model=d, n_experts=e, top_k=1, d_hidden=h,
                     device_groups=1)
    note("ffn random", dict(counts=counts, d=d, h=h))
    layer = DeviceLayer(w, trial=trial)
    owner = np.repeat(np.arange(e), counts)
    rng.shuffle(owner)
    logits = np.zeros((n, e), np.float32)
    logits[np.arange(n), owner] = 6.0
    ref = orc.route_and_drop(logits, 1, 1, NONE, GLOBAL, 1.0)
    np.testing.assert_array_equal(ref.plan.expert_count, counts)
    desc = layer.desc(NONE, GLOBAL, 1.0)
    buf = run_layer(layer, desc, logits)
    assert_plan_equal(buf, ref, "ffn random")
    y_ref = orc.layer_output(layer.x_host, ref.scores, ref.keep, layer.host_gate, layer.host_up, layer.host_down)
    assert_output_close(to_host_f64(buf.y), y_ref, TOL[w.dtype], "ffn random")
    fused = capmoe.LayerBuffers(desc)
    capmoe.layer_forward(fused, layer.x, layer.w_router, layer.bias, layer.w_gate, layer.w_up, layer.w_down,
                         torch.from_numpy(logits).cuda(), fused_dispatch=True)
    torch.cuda.synchronize()
    assert torch.equal(fused.y, buf.y)


# ------------------------------------------------------------------------------------------------
# full size: the launch configuration the benchmark times
# ------------------------------------------------------------------------------------------------
_layers = {}


def full_layer(name):
    """The workload's inputs on the device and on the host, shared by the full-size tests (one at a time)."""
    if name not in _layers:
        _layers.clear()
        torch.cuda.empty_cache()
        _layers[name] = DeviceLayer(W[name])
    return _layers[name]


def stratified_rows(plan, seed):
    """Rows of the plan chosen so that every GEMM tile of the timed launch holds a checked row: one row in
    every 64-row piece of every expert's rows (64 rows is the shortest tile, and the tiles of a cut last round
    are 64-row pieces of 256-row tiles, so every full-height tile gets four), plus the first and last row of
    every expert."""
    rng = np.random.default_rng(seed)
    off = plan.expert_offset
    rows = []
    for e in range(len(off) - 1):
        lo, hi = int(off[e]), int(off[e + 1])
        if hi == lo:
            continue
        rows += [lo, hi - 1]
        for p0 in range(lo, hi, 64):
            rows.append(int(rng.integers(p0, min(p0 + 64, hi))))
    return np.array(sorted(set(rows)), np.int64)


def check_rows_of_yp(orc, layer, buf, ref, rows, what):
    """yp[r,:] = E_e(x[row_token[r]]) for the listed rows: the oracle computes each row as a one-expert layer with
    gate weight 1 (Eq. 2 with a single term)."""
    w = layer.w
    tok = ref.plan.row_token[rows]
    expert = np.searchsorted(ref.plan.expert_offset, rows, side="right") - 1
    ones = np.ones((len(rows), w.n_experts), np.float32)
    keep = np.zeros((len(rows), w.n_experts), np.uint8)
    keep[np.arange(len(rows)), expert] = 1
    ref_rows = orc.layer_output(layer.x_host[tok], ones, keep, layer.host_gate, layer.host_up, layer.host_down)
    got = to_host_f64(buf.yp[torch.from_numpy(rows).cuda()])
    assert np.all(np.isfinite(got))
    assert_output_close(got, ref_rows, TOL[w.dtype], what + " yp rows")


def special_tokens(ref, n):
    kept_per_token = ref.keep.sum(1)
    picks = [0, n - 1, int(np.argmax(kept_per_token))]          # ends of the batch, the token with most experts
    picks += list(np.flatnonzero(kept_per_token == 0)[:4])      # tokens that lost every expert
    return picks


# (mode, scope, gamma) per workload; full = every token of the batch is compared, otherwise the tokens of a
# stratified row sample (at least 512)
FULL_LAYER_CASES = [
    ("olmoe", True, [(TD, LOCAL, 1.0), (TD, LOCAL, 2.0), (NONE, LOCAL, 1.0)]),
    ("decode", True, [(TD, LOCAL, 1.0), (ED, LOCAL, 1.0)]),
    ("finegrained", False, [(ED, LOCAL, 1.0), (ED, LOCAL, 1.25), (TD, LOCAL, 1.0)]),
    ("mixtral", False, [(NONE, LOCAL, 1.0), (TD, LOCAL, 1.0), (ED, LOCAL, 1.0)]),
]


@pytest.mark.parametrize("name,full,cases", FULL_LAYER_CASES)
def test_layer_full_size(orc, name, full, cases):
    """The launch configuration the benchmark times: y on the whole batch (OLMoE- and decode-shaped) or on at
    least 512 tokens that cover every row tile of every expert, and sampled rows of yp one by one."""
    w = W[name]
    layer = full_layer(name)
    logits = orc.router_logits(layer.x_host, layer.w_router_host, layer.bias_host)
    for mode, scope, gamma in cases:
        ref = orc.route_and_drop(logits, w.top_k, w.device_groups, mode, scope, gamma)
        rows = stratified_rows(ref.plan, 11)
        if full:
            toks = None
        else:
            picks = set(int(t) for t in ref.plan.row_token[rows]) | set(int(t) for t in special_tokens(ref, w.n_tokens))
            extra = np.random.default_rng(12).permutation(w.n_tokens)
            for t in extra:                     # top up to 512 tokens
                if len(picks) >= 512:
                    break
                picks.add(int(t))
            toks = np.array(sorted(picks), np.int32)
        note("full size", name, dict(mode=mode, gamma=gamma, rows=ref.plan.rows, sampled_rows=len(rows),
                                     tokens=w.n_tokens if toks is None else len(toks)))
        buf, _ = check_layer(orc, layer, mode, scope, gamma, tokens=toks, what=f"{name} full size")
        check_rows_of_yp(orc, layer, buf, ref, rows, f"{name} full size")
        del buf


@pytest.mark.parametrize("name,mode,full", [("mixtral", TD, False), ("mixtral", ED, False), ("finegrained", ED, False),
                                            ("decode", ED, True), ("olmoe", TD, True)])
def test_layer_full_size_own_router(orc, name, mode, full):
    """The path the benchmark times end to end: the library's own router GEMM feeds the drop.  Its logits are
    read back and handed to the oracle: scores, top-k and the plan must then be bit-equal, and y within
    tolerance (whole batch, or at least 512 tokens covering every row tile)."""
    w = W[name]
    layer = full_layer(name)
    desc = layer.desc(mode, LOCAL, 1.0)
    buf = capmoe.LayerBuffers(desc)
    capmoe.layer_forward(buf, layer.x, layer.w_router, layer.bias, layer.w_gate, layer.w_up, layer.w_down,
                         fused_dispatch=True)
    torch.cuda.synchronize()
    logits = buf.logits.cpu().numpy()
    ref_logits = orc.router_logits(layer.x_host, layer.w_router_host, layer.bias_host)
    assert np.abs(logits - ref_logits).max() <= 1e-4 * np.abs(ref_logits).max()
    ref = orc.route_and_drop(logits, w.top_k, w.device_groups, mode, LOCAL, 1.0)
    np.testing.assert_array_equal(buf.scores.cpu().numpy().view(np.uint32), ref.scores.view(np.uint32))
    np.testing.assert_array_equal(buf.topk_idx.cpu().numpy(), ref.topk_idx)
    assert_plan_equal(buf, ref, f"{name} own router")
    assert ref.plan.seg_count.max(initial=0) <= ref.cap
    rows = stratified_rows(ref.plan, 13)
    if full:
        toks = None
    else:
        picks = set(int(t) for t in ref.plan.row_token[rows]) | set(int(t) for t in special_tokens(ref, w.n_tokens))
        for t in np.random.default_rng(14).permutation(w.n_tokens):
            if len(picks) >= 512:
                break
            picks.add(int(t))
        toks = np.array(sorted(picks), np.int32)
    note("own router", name, dict(mode=mode, rows=ref.plan.rows, tokens=w.n_tokens if toks is None else len(toks)))
    y_ref = orc.layer_output(layer.x_host, ref.scores, ref.keep, layer.host_gate, layer.host_up, layer.host_down,
                             token_list=toks)
    y = to_host_f64(buf.y)
    assert_output_close(y if toks is None else y[toks], y_ref, TOL[w.dtype], f"{name} own router")
    # run to run, and through the one-call entry point (what the benchmark times): the same bits
    again, one = capmoe.LayerBuffers(desc), capmoe.LayerBuffers(desc)
    capmoe.layer_forward(again, layer.x, layer.w_router, layer.bias, layer.w_gate, layer.w_up, layer.w_down,
                         fused_dispatch=True)
    capmoe.moe_layer_forward(desc, layer.x, layer.w_router, layer.bias, layer.w_gate, layer.w_up, layer.w_down, None, 0,
                             one)
    torch.cuda.synchronize()
    for other in (again, one):
        assert torch.equal(other.y, buf.y) and torch.equal(other.yp[:ref.plan.rows], buf.yp[:ref.plan.rows])
        assert torch.equal(other.pair_row, buf.pair_row) and torch.equal(other.expert_offset, buf.expert_offset)


def test_release_full_size_layers():
    _layers.clear()
    torch.cuda.empty_cache()


def test_own_router_end_to_end_properties(orc):
    """The timed path (own router GEMM): its plan obeys the method's invariants for its own scores,
    the result is deterministic, and it agrees with the oracle wherever the routing decisions agree."""
    w = synth.scaled(W["olmoe"], n_tokens=1024, d_model=512, d_hidden=256, n_experts=32, top_k=4)
    layer = DeviceLayer(w)
    desc = layer.desc(TD, LOCAL, 1.0)
    a = run_layer(layer, desc)
    b = run_layer(layer, desc)
    rows_a = int(a.expert_offset[-1])
    assert torch.equal(a.y, b.y) and torch.equal(a.pair_row, b.pair_row)
    assert torch.equal(a.row_token[:rows_a], b.row_token[:rows_a])       # entries beyond P are not written
    scores, idx = a.scores.cpu().numpy(), a.topk_idx.cpu().numpy()
    cnt, off = a.expert_count.cpu().numpy(), a.expert_offset.cpu().numpy()
    rows = int(off[-1])
    tok, wt = a.row_token.cpu().numpy()[:rows], a.row_weight.cpu().numpy()[:rows]
    cand = np.zeros_like(scores, dtype=bool)
    cand[np.arange(w.n_tokens)[:, None], idx] = True
    loads = cand.sum(0)
    np.testing.assert_array_equal(cnt, np.minimum(loads, a.cap))       # kept = min(load, C); max load <= C
    assert loads.sum() == w.n_tokens * w.top_k
    for j in range(w.n_experts):
        t = tok[off[j]:off[j + 1]]
        assert np.all(np.diff(t) > 0) and np.all(cand[t, j])
        np.testing.assert_array_equal(wt[off[j]:off[j + 1]], scores[t, j])
        dropped = np.setdiff1d(np.flatnonzero(cand[:, j]), t)
        if len(dropped):
            assert scores[t, j].min() >= scores[dropped, j].max()
    # against the oracle: logits close, and y close on tokens whose candidate sets agree
    ref_logits = orc.router_logits(layer.x_host, layer.w_router_host, layer.bias_host)
    assert np.abs(a.logits.cpu().numpy() - ref_logits).max() <= 1e-4 * np.abs(ref_logits).max()
    ref = orc.route_and_drop(ref_logits, w.top_k, 1, TD, LOCAL, 1.0)
    keep_gpu = np.zeros_like(ref.keep)
    for j in range(w.n_experts):
        keep_gpu[tok[off[j]:off[j + 1]], j] = 1
    same = np.flatnonzero((keep_gpu == ref.keep).all(1))
    assert len(same) > 0.97 * w.n_tokens
    y_ref = orc.layer_output(layer.x_host, ref.scores, ref.keep, layer.host_gate, layer.host_up, layer.host_down,
                             token_list=same.astype(np.int32))
    assert_output_close(to_host_f64(a.y)[same], y_ref, TOL[w.dtype], "own router")
