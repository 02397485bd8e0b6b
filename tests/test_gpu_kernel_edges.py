"""Sizes at which the rules that choose a kernel, and the kernels' tiles, have their edges."""
import numpy as np
import pytest
import torch

from paper_2503_05066_amd import capmoe

pytestmark = pytest.mark.gpu


# ------------------------------------------------------------------------------------------------
# combine: rows of less than a wave's pieces, a piece more, two pieces a lane; none, all and more than 64 slots taken
# ------------------------------------------------------------------------------------------------
@pytest.mark.parametrize("n,d,slots,dtype", [
    (1, 8, 1, "bf16"), (3, 512, 8, "bf16"), (5, 520, 9, "bf16"), (16384, 64, 2, "bf16"), (16385, 64, 2, "bf16"),
    (16385, 504, 3, "bf16"), (16384, 1024, 5, "bf16"), (16383, 1032, 5, "bf16"), (700, 1024, 130, "bf16"),
    (2048, 64, 2, "bf16"), (2049, 64, 2, "bf16"), (2049, 384, 8, "bf16"), (2049, 392, 8, "bf16"), (3000, 256, 10, "bf16"),
    (4097, 256, 16, "bf16"), (4097, 264, 16, "bf16"), (9601, 128, 24, "bf16"), (2000, 520, 3, "bf16"), (1999, 520, 3, "bf16"),
    (2001, 1016, 4, "bf16"), (1025, 2048, 6, "bf16"), (4097, 2048, 6, "bf16"), (70, 2056, 1, "bf16"), (33, 1032, 4, "bf16"), (16384, 1024, 2, "bf16"),
    (8192, 2048, 9, "bf16"), (4097, 4096, 3, "bf16"),
    (2049, 188, 3, "f32"), (2, 4, 2, "f32"), (129, 260, 17, "f32"), (16385, 252, 3, "f32"), (16384, 512, 2, "f32"), (40, 256, 70, "f32")])
def test_combine(n, d, slots, dtype):
    if slots <= 64:
        desc = capmoe.make_desc(n, d, 64, slots, 128, 1, capmoe.MODE_NONE, capmoe.SCOPE_LOCAL, 1.0,
                                capmoe.DTYPE_BF16 if dtype == "bf16" else capmoe.DTYPE_F32)
    else:  # more slots than one wave has lanes: a device's experts beside the listed ones
        desc = capmoe.make_desc(n, d, 2 * (slots - 4), 4, 128, 2, capmoe.MODE_EXPANDED_DROP, capmoe.SCOPE_LOCAL, 1.0,
                                capmoe.DTYPE_BF16 if dtype == "bf16" else capmoe.DTYPE_F32)
    assert capmoe.moe_query(desc)[1] == slots
    gen = torch.Generator(device="cuda").manual_seed(n + d)
    rows = 3 * n + 1
    act = torch.bfloat16 if dtype == "bf16" else torch.float32
    yp = torch.randn((rows, d), generator=gen, device="cuda").to(act)
    weight = torch.rand(rows, generator=gen, device="cuda")
    pair_row = torch.randint(0, rows, (n, slots), generator=gen, device="cuda", dtype=torch.int32)
    share = torch.rand((n, 1), generator=gen, device="cuda")
    share[: n // 4], share[n - n // 4:] = 0.0, 1.0        # tokens without a row, tokens whose slots all hold one
    pair_row[torch.rand((n, slots), generator=gen, device="cuda") >= share] = -1
    y = torch.full((n, d), 7.0, dtype=act, device="cuda")
    capmoe.moe_combine(desc, yp, weight, pair_row, y)
    torch.cuda.synchronize()
    ref = torch.zeros((n, d), dtype=torch.float64, device="cuda")
    mass = torch.zeros((n, d), dtype=torch.float64, device="cuda")
    for s in range(slots):
        r = pair_row[:, s].long()
        w = torch.where(r >= 0, weight[r.clamp(min=0)], 0.0).double()[:, None]
        v = w * yp[r.clamp(min=0)].double()
        ref += v
        mass += v.abs()
    # one fp32 rounding per slot (half a unit of the running sum, which the mass bounds), one rounding to bf16
    bound = slots * 2.0 ** -24 * mass + (2.0 ** -8 * ref.abs() if dtype == "bf16" else 0.0)
    assert bool(((y.double() - ref).abs() <= bound).all())
    assert bool((y[(pair_row < 0).all(dim=1)] == 0).all())


# ------------------------------------------------------------------------------------------------
# softmax and top-k of long batches (four lanes per token): the same bits as in batches of 64 tokens, which take the kernel
# that the parity tests compare with the oracle
# ------------------------------------------------------------------------------------------------
def _route(logits, k, x=None, w=None, bias=None):
    n, e = logits.shape
    desc = capmoe.make_desc(n, 8 if x is None else x.shape[1], e, k, 128, 1, capmoe.MODE_NONE)
    out = [torch.empty((n, e), device="cuda"), torch.empty((n, k), dtype=torch.int32, device="cuda"),
           torch.empty((n, k), device="cuda")]
    ws = torch.empty(max(capmoe.moe_query(desc)[3], 256), dtype=torch.uint8, device="cuda")
    capmoe.moe_route_topk(desc, x, w, bias, x is None, logits, *out, ws)
    return out


def _assert_same_as_short_batches(logits, k, out):
    for t0 in list(range(0, 1024, 64)) + [logits.shape[0] - 65]:
        part = slice(t0, t0 + 64 + (t0 > 1024))
        for a, b in zip(out, _route(logits[part].clone(), k)):
            assert torch.equal(a[part].view(torch.int32), b.view(torch.int32)), (t0, k)


@pytest.mark.parametrize("n,e,k", [(12288, 1, 1), (12289, 8, 2), (12300, 16, 16), (12351, 17, 3), (12288, 30, 6), (12288, 32, 32),
                                   (20480, 33, 33), (12290, 60, 4), (12288, 61, 7), (12291, 64, 8), (20481, 64, 64),
                                   (12288, 100, 5), (12288, 128, 8), (12288, 130, 9), (20480, 256, 64), (12289, 255, 1),
                                   # where the rule goes over to four lanes, by experts and list length
                                   (12287, 31, 4), (16383, 61, 7), (16384, 61, 7), (24576, 33, 33), (14335, 60, 4), (14336, 60, 4),
                                   (16384, 60, 40), (24576, 64, 64), (16390, 65, 16), (24577, 127, 15), (14339, 100, 5), (16384, 100, 2),
                                   (14336, 132, 9), (14341, 256, 64), (32767, 130, 17), (32768, 130, 17), (32769, 255, 64)])
@pytest.mark.parametrize("kind", ["normal", "ties", "wide"])
def test_softmax_topk_long_batches(n, e, k, kind):
    gen = torch.Generator(device="cuda").manual_seed(n + e)
    logits = torch.randn((n, e), generator=gen, device="cuda") * 2
    if kind == "ties":      # rows of equal scores, and equal scores at the threshold
        logits = logits.round() * 0.5
        logits[::7] = 0.0
    elif kind == "wide":    # scores down to the smallest, and exact zeros
        logits *= 20.0
        logits[::2, e // 2] += 70.0
    _assert_same_as_short_batches(logits, k, _route(logits, k))


@pytest.mark.parametrize("n,d,e,k", [(12288, 256, 64, 6), (16385, 128, 61, 4), (12500, 512, 128, 8), (13000, 1024, 8, 2)])
def test_softmax_topk_long_batches_adds_router_slices(n, d, e, k):
    gen = torch.Generator(device="cuda").manual_seed(n)
    x = torch.randn((n, d), generator=gen, device="cuda").to(torch.bfloat16)
    w = torch.randn((e, d), generator=gen, device="cuda") * d ** -0.5
    bias = torch.randn(e, generator=gen, device="cuda")
    logits = torch.empty((n, e), device="cuda")
    out = _route(logits, k, x, w, bias)
    ref = x.double() @ w.double().T + bias.double()
    # fp32 sums of d exact products: at most d + 2 roundings of partial sums that the mass bounds
    mass = x.double().abs() @ w.double().abs().T + bias.double().abs()
    assert bool(((logits.double() - ref).abs() <= (d + 2) * 2.0 ** -24 * mass).all())
    _assert_same_as_short_batches(logits, k, out)


@pytest.mark.parametrize("n,e,k", [(130, 64, 8), (12288, 64, 8), (130, 5, 5), (12288, 5, 3), (12290, 8, 8), (130, 61, 7), (16384, 61, 7),
                                   (130, 130, 9), (14336, 132, 9), (24576, 127, 8), (16384, 256, 64), (130, 255, 64), (32768, 255, 20),
                                   (70, 64, 64), (24576, 64, 64)])
def test_tokens_without_numbers(n, e, k):
    logits = torch.randn((n, e), generator=torch.Generator(device="cuda").manual_seed(n), device="cuda")
    clean = _route(logits.clone(), k)
    broken = torch.zeros(n, dtype=torch.bool, device="cuda")
    broken[1::5] = True
    logits[1::10, min(3, e - 1)], logits[6::10] = float("nan"), float("-inf")
    scores, idx, score = _route(logits, k)
    assert bool(scores[broken].isnan().all()) and bool(score[broken].isnan().all())
    assert torch.equal(idx[broken], torch.arange(k, dtype=torch.int32, device="cuda").expand(int(broken.sum()), k))
    for a, b in zip((scores, idx, score), clean):
        assert torch.equal(a[~broken], b[~broken])


# ------------------------------------------------------------------------------------------------
# thresholds of the drop: ranges of keys that are one key, a few, a power of two wide and the whole word; bins kept whole and cut
# ------------------------------------------------------------------------------------------------
def _scores_of_range(rng, n, e, width):
    """Scores whose bit patterns lie within `width` of each other, everything listed: the capacity alone cuts."""
    base = np.uint32(0x3d000000)
    return (base + rng.integers(0, width, (n, e)).astype(np.uint32)).view(np.float32)


def _keys_of_pairs(scores, lists, metric, classes, seed, seg_tokens):
    """(candidates [N,E], keys [N,E]) as the drop defines them: rank + 1 above the class's two bits, in 32-bit words; 0 without."""
    n, e = scores.shape
    token, expert = np.meshgrid(np.arange(n, dtype=np.uint32), np.arange(e, dtype=np.uint32), indexing="ij")
    if metric == capmoe.METRIC_SCORE:
        rank = scores.view(np.uint32)
    elif metric == capmoe.METRIC_RANDOM:
        x = token * np.uint32(e) + expert + np.uint32(seed * 0x9E3779B9 & 0xFFFFFFFF)
        for shift, factor in ((16, 0x7FEB352D), (15, 0x846CA68B)):
            x = (x ^ (x >> np.uint32(shift))) * np.uint32(factor)
        rank = (x ^ (x >> np.uint32(16))) >> np.uint32(3)
    else:
        local = token % np.uint32(seg_tokens)
        rank = np.uint32(seg_tokens - 1) - local if metric == capmoe.METRIC_ORDER else local
    cand = np.zeros((n, e), bool)
    np.put_along_axis(cand, lists, True, axis=1)
    cls = np.zeros(n, np.uint32) if classes is None else classes.astype(np.uint32)
    return cand, np.where(cand, rank + (cls << np.uint32(30))[:, None] + np.uint32(1), np.uint32(0))


def _drop_against_sort(n, e, k, groups, scope, gamma, scores, lists, metric=0, classes=None, seed=3):
    """Token Drop of given scores and lists: the whole plan against a sort of (key, token, expert), word for word."""
    desc = capmoe.make_desc(n, 4, e, k, 8, groups, capmoe.MODE_TOKEN_DROP, scope, gamma, capmoe.DTYPE_F32, metric)
    cap, slots, rows, workspace = capmoe.moe_query(desc)
    blocks = groups if scope in (capmoe.SCOPE_LOCAL, capmoe.SCOPE_LOCAL_DEVICE) else 1
    span = e // groups if scope in (capmoe.SCOPE_LOCAL_DEVICE, capmoe.SCOPE_GLOBAL_DEVICE) else 1
    per = n // blocks
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    out = {name: torch.full(shape, -7, dtype=dt, device="cuda") for name, shape, dt in (
        ("expert_count", (e,), torch.int32), ("seg_count", (blocks, e), torch.int32), ("expert_offset", (e + 1,), torch.int32),
        ("row_token", (rows,), torch.int32), ("row_weight", (rows,), torch.float32), ("pair_row", (n, slots), torch.int32))}
    ws = torch.empty(max(workspace, 256), dtype=torch.uint8, device="cuda")
    capmoe.moe_capacity_drop_ranked(desc, dev(scores), dev(lists.astype(np.int32)), None if classes is None else dev(classes), seed,
                                    out["expert_count"], out["seg_count"], out["expert_offset"], out["row_token"], out["row_weight"],
                                    out["pair_row"], ws)
    torch.cuda.synchronize()
    cand, keys = _keys_of_pairs(scores, lists, metric, classes, seed, per)
    keep = np.zeros((n, e), bool)
    token, expert = np.meshgrid(np.arange(n), np.arange(e), indexing="ij")
    for b in range(blocks):
        for g in range(e // span):
            part = (slice(b * per, (b + 1) * per), slice(g * span, (g + 1) * span))
            t, x = token[part].ravel(), expert[part].ravel()
            t, x = t[cand[t, x]], x[cand[t, x]]
            best = np.lexsort((x, t, -keys[t, x].astype(np.int64)))[:cap]   # larger key, then lower token, then lower expert
            keep[t[best], x[best]] = True
    row_expert, row_token = np.nonzero(keep.T)                # rows are expert-major, ascending token
    pair_row = np.full((n, slots), -1, np.int64)
    pair_row[row_token, (np.cumsum(cand, axis=1) - 1)[row_token, row_expert]] = np.arange(len(row_token))
    got = {name: a.cpu().numpy() for name, a in out.items()}
    np.testing.assert_array_equal(got["expert_count"], keep.sum(axis=0))
    np.testing.assert_array_equal(got["expert_offset"], np.concatenate([[0], np.cumsum(keep.sum(axis=0))]))
    np.testing.assert_array_equal(got["seg_count"], keep.reshape(blocks, per, e).sum(axis=1))
    np.testing.assert_array_equal(got["row_token"][: len(row_token)], row_token)
    np.testing.assert_array_equal(got["row_weight"][: len(row_token)].view(np.uint32), scores.view(np.uint32)[row_token, row_expert])
    np.testing.assert_array_equal(got["pair_row"], pair_row)
    assert (got["row_token"][len(row_token):] == -7).all() and (got["row_weight"][len(row_token):] == -7).all()


# a segment of a wave, of 256 and of 1024 threads in one launch; selected by 256 threads (by four, at odd addresses), by 1024, from L2
# and by many blocks; one expert, and several under one budget
FORMS = [(40, 1, 0), (100, 1, 0), (300, 1, 0), (3000, 1, 0), (500, 1, 3), (1000, 1, 3), (999, 1, 3), (2001, 1, 3), (4096, 1, 3), (4099, 1, 3),
         (12003, 1, 0), (16384, 1, 0), (32771, 1, 0), (65544, 1, 0), (98304, 1, 0), (98305, 1, 0), (98308, 1, 0), (65544, 2, 2)]


def _lists(rng, n, e, k):
    return np.sort(np.argsort(rng.random((n, e)), axis=1)[:, :k], axis=1)


@pytest.mark.parametrize("n,groups,scope", [(63, 1, 0), (2048, 1, 0), (2049, 1, 0), (8192, 1, 0), (8196, 1, 0), (12003, 1, 0),
                                            (2048, 2, 3), (24000, 4, 2), (65544, 1, 1), (30, 2, 2), (32, 2, 2), (34, 2, 2),
                                            (8192, 2, 2), (8224, 2, 2), (8226, 2, 2)])
@pytest.mark.parametrize("width", [1, 2, 1024, 2048, 2049, 1 << 21, 1 << 24])
def test_drop_threshold_of_key_ranges(n, groups, scope, width):
    """Expert-level and device-level capacities; runs of 16 tokens that are whole, cut short and at odd addresses, segments of one, two
    and many chunks of 4096 tokens."""
    n -= n % groups
    e = k = 4
    rng = np.random.default_rng(n + width)
    _drop_against_sort(n, e, k, groups, scope, 0.6, _scores_of_range(rng, n, e, width), _lists(rng, n, e, k))


@pytest.mark.parametrize("n,groups,scope", FORMS)
@pytest.mark.parametrize("metric", [capmoe.METRIC_SCORE, capmoe.METRIC_ORDER, capmoe.METRIC_REVERSE_ORDER, capmoe.METRIC_RANDOM])
@pytest.mark.parametrize("gamma", [0.15, 0.7])
def test_drop_threshold_of_classes(n, groups, scope, metric, gamma):
    """Keys over the whole word: four classes above every metric (gathered weights), lists that name half of the experts."""
    n -= n % groups
    rng = np.random.default_rng(n + metric)
    scores = rng.random((n, 4)).astype(np.float32)
    scores[rng.random(n) < 0.2] = 0.0
    _drop_against_sort(n, 4, 2, groups, scope, gamma, scores, _lists(rng, n, 4, 2), metric, rng.integers(0, 4, n).astype(np.uint8))


@pytest.mark.parametrize("n,groups,scope", FORMS)
@pytest.mark.parametrize("bits,cls", [(0x7fc00000, 2), (0xffc00000, 0), (0xffe00000, 0), (0xfff00000, 0), (0xfffffffe, 0)])
def test_drop_of_scores_that_are_no_numbers(n, groups, scope, bits, cls):
    """More tokens without numbers than the capacity keeps, at the top of the 32-bit keys, above lower classes with scores of zero."""
    n -= n % groups
    e, k = 4, 2
    rng = np.random.default_rng(n + cls)
    scores = rng.random((n, e)).astype(np.float32)
    scores[rng.random(n) < 0.3] = 0.0
    classes = rng.integers(0, 2, n).astype(np.uint8) if cls else None
    broken = rng.random(n) < 0.3
    scores.view(np.uint32)[broken] = bits
    if cls:
        classes[broken] = cls
    for gamma in (0.3, 0.8):
        _drop_against_sort(n, e, k, groups, scope, gamma, scores, _lists(rng, n, e, k), classes=classes)


# ------------------------------------------------------------------------------------------------
# the drop of a few tokens: a wave's lanes filled, short by one and exceeded, the limits of its rule on both sides (tokens of a segment,
# lists of 28 and 29, of 14 and 15 entries, 1024 segments), blocks with fewer segments than waves; through the one call that also builds
# the tile schedule, against the oracle's plan
# ------------------------------------------------------------------------------------------------
@pytest.mark.parametrize("n,e,k,groups", [(1, 1, 1, 1), (1, 64, 8, 1), (3, 5, 2, 1), (63, 8, 2, 1), (64, 8, 3, 1), (65, 7, 2, 1), (128, 8, 2, 1),
                                          (129, 8, 2, 1), (512, 16, 6, 4), (513, 9, 2, 9), (512, 128, 9, 8), (512, 130, 4, 10),
                                          (256, 64, 6, 8), (40, 256, 64, 4), (500, 240, 8, 5), (64, 64, 28, 1), (64, 64, 29, 1),
                                          (512, 64, 14, 8), (512, 64, 15, 8), (96, 256, 3, 4), (96, 256, 3, 8), (2048, 32, 2, 32), (1023, 33, 5, 33)])
@pytest.mark.parametrize("mode,metric,classes", [(0, 0, False), (1, 0, False), (1, 1, True), (2, 3, False), (2, 2, True)])
def test_drop_of_a_few_tokens(n, e, k, groups, mode, metric, classes):
    from oracle import oracle

    n, groups = (n, groups) if n % groups == 0 and e % groups == 0 else (n, 1)
    d, h = 128, 128
    rng = np.random.default_rng(n * e + mode)
    logits = np.round(rng.standard_normal((n, e)) * 3).astype(np.float32)     # many equal scores
    cls = rng.integers(0, 3, n).astype(np.uint8) if classes else None
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    for scope in (0, 1):
        for gamma in (0.0, 0.4, 1.0):
            desc = capmoe.make_desc(n, d, e, k, h, groups, mode, scope, gamma, capmoe.DTYPE_F32, metric)
            ref = oracle.route_and_drop(logits, k, groups, mode, scope, gamma, metric=metric, token_class=cls, seed=5)
            buf = capmoe.LayerBuffers(desc)
            buf.logits.copy_(dev(logits))
            capmoe.moe_route_topk(desc, None, None, None, True, buf.logits, buf.scores, buf.topk_idx, buf.topk_score, buf.workspace)
            capmoe.moe_capacity_drop_ranked(desc, buf.scores, buf.topk_idx, None if cls is None else dev(cls), 5, buf.expert_count,
                                            buf.seg_count, buf.expert_offset, buf.row_token, buf.row_weight, buf.pair_row,
                                            buf.workspace)
            torch.cuda.synchronize()
            p = ref.plan
            for got, want in ((buf.expert_count, p.expert_count), (buf.expert_offset, p.expert_offset), (buf.seg_count, p.seg_count),
                              (buf.row_token[: p.rows], p.row_token), (buf.row_weight[: p.rows], p.row_weight),
                              (buf.pair_row, p.pair_row)):
                np.testing.assert_array_equal(got.cpu().numpy(), want)
            # the layer in one call: the drop's last block builds the tile schedule
            x = rng.standard_normal((n, d)).astype(np.float32)
            w_router = (rng.standard_normal((e, d)) / 12).astype(np.float32)
            ws = [dev((rng.standard_normal(s) / 12).astype(np.float32)) for s in ((e, h, d), (e, h, d), (e, d, h))] if e <= 16 else None
            if ws and gamma == 0.4:
                one, four = capmoe.LayerBuffers(desc), capmoe.LayerBuffers(desc)
                capmoe.moe_layer_forward(desc, dev(x), dev(w_router), None, *ws, None if cls is None else dev(cls), 5, one)
                capmoe.layer_forward(four, dev(x), dev(w_router), None, *ws, token_class=None if cls is None else dev(cls), seed=5)
                torch.cuda.synchronize()
                assert torch.equal(one.y, four.y) and torch.equal(one.pair_row, four.pair_row)


# ------------------------------------------------------------------------------------------------
# at most k experts per token: blocks of tokens filled, short by one and exceeded, blocks that straddle two capacity blocks, one to four
# experts per lane, more candidates than lanes, equal scores; against the oracle's plan
# ------------------------------------------------------------------------------------------------
@pytest.mark.parametrize("n,e,k,over,groups", [(1, 8, 2, 4, 1), (15, 8, 2, 4, 1), (16, 64, 8, 8, 1), (17, 64, 8, 8, 1), (63, 65, 4, 8, 1),
                                               (65, 128, 8, 16, 4), (257, 130, 14, 50, 1), (120, 256, 8, 56, 8), (1030, 30, 4, 6, 2),
                                               (16384, 8, 2, 3, 1), (16385, 16, 2, 3, 1), (16416, 70, 4, 4, 4),
                                               (16400, 130, 3, 2, 1)])
@pytest.mark.parametrize("mode,gamma", [(2, 1.0), (2, 3.0), (1, 1.0)])
def test_limit_of_experts_per_token(n, e, k, over, groups, mode, gamma):
    from oracle import oracle

    n, groups = (n, groups) if n % groups == 0 and e % groups == 0 else (n, 1)
    rng = np.random.default_rng(n * e + mode)
    logits = np.round(rng.standard_normal((n, e)) * 3).astype(np.float32)     # many equal scores
    desc = capmoe.make_desc(n, 128, e, k, 128, groups, mode, 0, gamma, capmoe.DTYPE_F32, 0, over, True)
    ref = oracle.route_and_drop(logits, k, groups, mode, 0, gamma, metric=0, token_class=None, seed=5, overselect=over, max_experts=True)
    buf = capmoe.LayerBuffers(desc)
    buf.logits.copy_(torch.from_numpy(logits).cuda())
    capmoe.moe_route_topk(desc, None, None, None, True, buf.logits, buf.scores, buf.topk_idx, buf.topk_score, buf.workspace)
    capmoe.moe_capacity_drop_ranked(desc, buf.scores, buf.topk_idx, None, 5, buf.expert_count, buf.seg_count, buf.expert_offset,
                                    buf.row_token, buf.row_weight, buf.pair_row, buf.workspace)
    torch.cuda.synchronize()
    p = ref.plan
    assert (p.pair_row >= 0).sum(axis=1).max() <= k
    for got, want in ((buf.expert_count, p.expert_count), (buf.expert_offset, p.expert_offset), (buf.seg_count, p.seg_count),
                      (buf.row_token[: p.rows], p.row_token), (buf.row_weight[: p.rows], p.row_weight), (buf.pair_row, p.pair_row)):
        np.testing.assert_array_equal(got.cpu().numpy(), want)


# ------------------------------------------------------------------------------------------------
# a batch without tokens: its arrays are null, its plan is zeros, whatever ranks the pairs
# ------------------------------------------------------------------------------------------------
@pytest.mark.parametrize("metric", [capmoe.METRIC_SCORE, capmoe.METRIC_ORDER, capmoe.METRIC_REVERSE_ORDER, capmoe.METRIC_RANDOM])
@pytest.mark.parametrize("classes", [False, True])
@pytest.mark.parametrize("mode,scope,over,limit", [(0, 1, 0, False), (1, 0, 0, False), (1, 3, 2, True), (2, 2, 0, False), (2, 0, 3, True)])
def test_empty_batch_of_every_metric(metric, classes, mode, scope, over, limit):
    e, groups = 8, 4
    desc = capmoe.make_desc(0, 128, e, 2, 128, groups, mode, scope, 1.0, capmoe.DTYPE_BF16, metric, over, limit)
    cls = torch.ones(1, dtype=torch.uint8, device="cuda") if classes else None     # an array that is there, though nothing is in it
    weights = [torch.zeros((e, 128, 128), dtype=torch.bfloat16, device="cuda") for _ in range(3)]
    w_router = torch.zeros((e, 128), device="cuda")
    for call in ("drop", "layer"):
        buf = capmoe.LayerBuffers(desc)
        assert buf.scores.data_ptr() == 0 and buf.topk_idx.data_ptr() == 0 and buf.pair_row.data_ptr() == 0
        for a in (buf.expert_count, buf.seg_count, buf.expert_offset):
            a.fill_(7)
        if call == "drop":
            capmoe.moe_capacity_drop_ranked(desc, buf.scores, buf.topk_idx, cls, 5, buf.expert_count, buf.seg_count,
                                            buf.expert_offset, buf.row_token, buf.row_weight, buf.pair_row, buf.workspace)
        else:
            capmoe.moe_layer_forward(desc, buf.y, w_router, None, *weights, cls, 5, buf)
        torch.cuda.synchronize()
        for a in (buf.expert_count, buf.seg_count, buf.expert_offset):
            assert bool((a == 0).all())


# ------------------------------------------------------------------------------------------------
# expert products: row tiles filled to every step of 32 rows, and one row less and more
# ------------------------------------------------------------------------------------------------
def _ffn_against_fp64(d, h, counts, seed):
    """moe_grouped_ffn over experts with these rows; every row against the product in 64 bits of the bf16 hidden activations."""
    e, n = len(counts), sum(counts)
    desc = capmoe.make_desc(n, d, e, 1, h, 1, capmoe.MODE_NONE, capmoe.SCOPE_GLOBAL, 1.0, capmoe.DTYPE_BF16)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    act = {}
    for name, shape, fan in (("x", (n, d), 1), ("g", (e, h, d), d), ("u", (e, h, d), d), ("w", (e, d, h), h)):
        act[name] = (torch.randn(shape, generator=gen, device="cuda") * fan ** -0.5).to(torch.bfloat16)
    offset = torch.tensor(np.concatenate([[0], np.cumsum(counts)]), dtype=torch.int32, device="cuda")
    ws = torch.empty(capmoe.moe_query(desc)[3], dtype=torch.uint8, device="cuda")
    yp = torch.full((n + 1, d), 7.0, dtype=torch.bfloat16, device="cuda")
    capmoe.moe_grouped_ffn(desc, act["x"], offset, act["g"], act["u"], act["w"], yp, ws)
    torch.cuda.synchronize()
    at = 0
    for j, c in enumerate(counts):
        rows = slice(at, at + c)
        x = act["x"][rows].double()
        g, u = x @ act["g"][j].double().T, x @ act["u"][j].double().T
        hidden = g * torch.sigmoid(g) * u
        ref, mass = hidden @ act["w"][j].double().T, hidden.abs() @ act["w"][j].double().abs().T
        # every hidden value and the output are rounded to bf16 once (2^-9 each); fp32 sums of d and h products add (d + h) 2^-24
        # of the mass, and the fp32 silu a few 2^-24
        bound = (2.0 ** -8 + (2 * d + h + 64) * 2.0 ** -24) * mass + 2.0 ** -8 * ref.abs() + 1e-6
        assert bool(((yp[rows].double() - ref).abs() <= bound).all()), (j, c)
        at += c
    assert bool((yp[n:] == 7.0).all())
    return yp


@pytest.mark.parametrize("d,h", [(128, 128), (256, 384), (384, 256)])
def test_ffn_partly_filled_tiles(d, h):
    _ffn_against_fp64(d, h, [65, 95, 96, 97, 128, 129, 160, 161, 191, 192, 193, 224, 225, 255, 256 + 66, 512 + 127], d + h)


@pytest.mark.parametrize("slabs_up,slabs_down", [(2, 4), (4, 6), (6, 8), (8, 2)])
def test_ffn_short_walks_of_low_tiles(slabs_up, slabs_down):
    """Fewer slabs of K than the rings of low tiles hold, as many, and more; every height a ring serves."""
    _ffn_against_fp64(64 * slabs_up, 64 * slabs_down, [1, 32, 33, 64, 65, 96, 128, 129, 160, 161, 5, 256 + 20], slabs_up)


@pytest.mark.parametrize("counts", [[70], [0, 129, 0, 33], [200, 1, 17], [256], [1, 16, 17, 100, 65], [257], [3] * 32, [9] * 29])
def test_ffn_few_tokens_on_experts_without_a_bound(counts):
    """Up to 256 tokens and 8 per expert on average the few-row kernels run whatever the plan puts on one expert, above them the
    others."""
    _ffn_against_fp64(256, 384, counts + [0] * (32 - len(counts)), sum(counts))


@pytest.mark.parametrize("counts", [[276] * 66, [256] * 64 + [1], [256, 40] * 64, [256, 40] * 64 + [33] * 12, [257] * 63])
def test_ffn_shared_last_round(counts):
    """Short items after a round of big ones (four column blocks, 256 compute units), which all XCDs share at the end: eight more
    than a round, one tile, exactly a round, more, and just under a round of big items, where none are shared."""
    _ffn_against_fp64(1024, 512, counts, len(counts))


@pytest.mark.parametrize("d,h,counts", [
    (768, 384, [256] * 86 + [21] * 40), (768, 384, [256] * 86 + [64]), (768, 384, [256] * 86 + [33] * 90),
    (1280, 640, [256, 21] * 52), (256, 128, [512] * 57 + [256] * 143 + [64] * 56),
])
def test_ffn_blocks_that_start_in_the_shared_round(d, h, counts):
    """257 to 260 big items: 33 per XCD leave the last one with fewer positions than compute units, and its other blocks begin
    with shared items: fewer of these than such blocks, fewer than a round, and more."""
    _ffn_against_fp64(d, h, counts, len(counts))


@pytest.mark.parametrize("counts", [[256] * 64, [256] * 65, [256] * 32 + [64] * 32, [256] * 32 + [64] * 33, [33] * 64, [200] * 63])
def test_ffn_about_an_item_per_compute_unit(counts):
    """Four column blocks: as many items as compute units, after which no block looks for another one, a few less and more."""
    _ffn_against_fp64(1024, 512, counts, len(counts))
