"""Edges of the tiles and of the dispatch rules of single kernels, against the oracle: sizes at
which a kernel's loop, remainder or variant changes.  (What the calls do as a whole is in
test_gpu_parity.py.)"""
from __future__ import annotations

import math

import numpy as np
import pytest
import torch

from oracle import d2o_ref as ref
from paper_2406_13035_amd import binding, synth
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,n,hidden,Hq,Hkv", [
    (1, 1, 32, 2, 1),        # one token, half of a 64-column k-tile
    (5, 37, 96, 3, 1),       # five sequences inside one 256-token tile, an odd head count, a k-tile and a half
    (1, 257, 64, 1, 1),      # one token past the tile, one k-tile
    (3, 200, 160, 4, 2),     # tiles that hold the end of a sequence
    (1, 1600, 96, 32, 32),   # more output tiles than workgroups, two k-tiles in each (the last one half)
    (1, 1600, 32, 32, 32),   # the same with a single half k-tile: every load opens another output tile
    (1, 1600, 64, 32, 32),   # ... a single whole one
    (1, 1600, 192, 32, 32),  # ... three: a workgroup's second output tile starts in the other weight stage
    (3, 1000, 160, 31, 6),   # ... two and a half; 22 head pairs (no XCD order), the last half empty, sequence ends in tiles
])
def test_projection_tile_edges(B, n, hidden, Hq, Hkv):
    """|got - want| <= 2e-3 |row|_inf + 2^-8 |want|: the oracle's fp64 product and rotation against
    fp32 accumulation and one rounding to bf16, as in test_qkv_projection_with_rotary_embedding."""
    g = torch.Generator().manual_seed(n + hidden)
    X = torch.randn(B, n, hidden, generator=g).to(torch.bfloat16)
    W = (torch.randn((Hq + 2 * Hkv) * 128, hidden, generator=g) / hidden ** 0.5).to(torch.bfloat16)
    out = binding.d2o_qkv_project(X.cuda(), W.cuda(), Hq, Hkv, 128, 7, 10000.0)
    Xd, Wd = binding.tensor_to_f64(X), binding.tensor_to_f64(W)
    for b in range(B):
        for got, want in zip(out, ref.qkv_project(Xd[b], Wd, Hq, Hkv, 128, 7, 10000.0)):
            got = binding.tensor_to_f64(got[b])
            assert np.all(np.abs(got - want) <= H.FLOAT_TOL * np.abs(want).max(axis=-1, keepdims=True)
                          + 2.0 ** -8 * np.abs(want))


def test_projection_rotates_a_token_alike_in_every_tile():
    """A tile inside one sequence forms its angles four tokens at a time, a tile with a sequence's end one by
    one; both reduce every token's angle to half a turn before its one rounding to fp32, so the same
    tokens give the same bits.  (The two fp64 angles differ by about 2^-53 * 10^3 turns, which changes one fp32
    rounding in 10^5, of which one in 10^4 shows in a bf16 result: 10^-9 per element, 10^7 elements.  An angle
    rounded at up to a turn changes about a hundred of them.)"""
    n, part, pos0, Hq, Hkv = 4096, 128, 3, 16, 8
    g = torch.Generator().manual_seed(4)
    X = torch.randn(1, n, 32, generator=g).to(torch.bfloat16).cuda()
    W = (torch.randn((Hq + 2 * Hkv) * 128, 32, generator=g) / 32 ** 0.5).to(torch.bfloat16).cuda()
    whole = binding.d2o_qkv_project(X, W, Hq, Hkv, 128, pos0)
    for s in range(0, n, part):
        for got, want in zip(binding.d2o_qkv_project(X[:, s:s + part].contiguous(), W, Hq, Hkv, 128, pos0 + s), whole):
            assert torch.equal(got, want[:, :, s:s + part])


@pytest.mark.parametrize("hidden", [(1 << 22) - 64, (1 << 22) - 32, 1 << 22])
def test_projection_of_very_wide_rows(hidden):
    """Rows so wide that a tile's offsets pass 31 bits, and the last width below: two sequences of
    two tokens against a product in 64 bits; the bar of test_projection_tile_edges plus the fp32 sum's own
    error (hidden / 16 steps whose roundings add like a random walk: 2^-24 * 500 of the row's norm, below 2e-4)."""
    B, n, Hq, Hkv = 2, 2, 1, 1
    g = torch.Generator(device="cuda").manual_seed(hidden)
    X = torch.randn(B, n, hidden, generator=g, device="cuda").to(torch.bfloat16)
    W = torch.empty((Hq + 2 * Hkv) * 128, hidden, dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    W *= hidden ** -0.5
    got = binding.d2o_qkv_project(X, W, Hq, Hkv, 128, 5)
    Y = torch.zeros(B * n, W.shape[0], dtype=torch.float64, device="cuda")
    for c in range(0, hidden, 1 << 18):
        Y += X.view(B * n, hidden)[:, c:c + (1 << 18)].double() @ W[:, c:c + (1 << 18)].double().t()
    Y = Y.view(B, n, -1).cpu().numpy()
    for b in range(B):
        for t, want in zip(got, ref.qkv_project(Y[b], np.eye(W.shape[0]), Hq, Hkv, 128, 5)):
            err = np.abs(binding.tensor_to_f64(t[b]) - want)
            assert np.all(err <= (H.FLOAT_TOL + 2e-4) * np.abs(want).max(axis=-1, keepdims=True) + 2.0 ** -8 * np.abs(want))


@pytest.mark.parametrize("n", [1, 15, 16, 17, 31, 32, 33, 255, 257, 300])
@pytest.mark.parametrize("d,Hq,Hkv", [(64, 4, 2), (128, 2, 2)])
def test_fp32_prompt_attention_tile_edges(n, d, Hq, Hkv):
    """16 query rows and 32 keys per tile, 8 wavefronts (256 keys) per round, 32 keys per column-sum
    block.  A logit of magnitude s carries at most (d / 16 + 4) roundings of 2^-24 s (four chains of d / 16
    products of four, added pairwise and scaled), which a probability shows as a relative error; the
    sums behind it add a few units of 2^-24 each.  |s| <= 20 here: 20 * 12 * 6e-8 = 1.4e-5, and twice
    that for the normaliser."""
    rng = np.random.RandomState(n + d)
    Q, K, V = (rng.randn(h, n, d).astype(np.float32) for h in (Hq, Hkv, Hkv))
    ctx = binding.D2O(1, 1, Hq, Hkv, d, n, n + 2, dtype="f32")
    Qg, Kg, Vg = (torch.from_numpy(x)[None].cuda() for x in (Q, K, V))
    O = torch.empty(1, Hq, n, d, device="cuda:0")
    ctx.d2o_prefill_attend(0, Qg, Kg, Vg, O)
    score, F = ctx.d2o_scores_export(0, n), ctx.d2o_get_density()
    got, G, var = O[0].double().cpu().numpy(), Hq // Hkv, []
    for h in range(Hkv):
        o, s, v = ref.prefill_kv_head(Q[h * G:(h + 1) * G].astype(np.float64), K[h].astype(np.float64),
                                         V[h].astype(np.float64))
        assert np.abs(got[h * G:(h + 1) * G] - o).max() <= 3e-5 * np.abs(V[h]).max()
        assert np.abs(score[0, h] - s).max() <= 3e-5 * s.max()
        var += list(v)
    assert abs(F[0, 0] - np.mean(var)) <= 1e-4 * max(np.mean(var), 1e-3)
    ctx.close()


@pytest.mark.parametrize("budget", [15359, 15360])
def test_grouping_counters_in_lds_and_in_memory(budget):
    """Merge groups of a head with as many retained tokens as the grouping kernel has counters in
    LDS, and one more (counters in memory): selections, targets and flags identical, merged rows
    within the float bar (check_compress_against_oracle)."""
    w = synth.WORKLOADS[3].scaled(n_q_heads=1, n_kv_heads=1, n_clusters=32)
    n, recent = 16500, 4000
    _, K, V = H.make_inputs(w, 1, 5, n)
    score32 = np.random.default_rng(budget).random((1, 1, n), dtype=np.float32)
    ctx = H.new_ctx(w, 1, 1, n, budget + 8)
    ctx.d2o_scores_import(0, score32)
    ctx.d2o_compress_layer(0, K, V, budget, recent)
    stats, _ = H.check_compress_against_oracle(ctx, 0, K, V, score32, budget, recent, 0, w.dtype)
    assert stats["evicted"] == n - budget and 0 < stats["passed"] < n - budget
    ctx.close()


@pytest.mark.parametrize("n,row,bad", [
    (1, 0, float("inf")),
    (40, 39, float("nan")),      # the last row, which also stands in for the rows behind the end
    (300, 0, float("inf")),
    (300, 17, float("-inf")),    # the second row of a 16-row block, inside a 32-key tile
    (300, 31, float("nan")),
    (300, 160, float("inf")),
])
@pytest.mark.parametrize("d,Hq,Hkv", [(64, 4, 2), (128, 2, 2)])
def test_fp32_prompt_attention_keeps_later_non_finite_values_out(n, row, bad, d, Hq, Hkv):
    """An infinite or NaN element in V row `row` of KV head 0 reaches that column of the rows from `row` on and
    nothing else: every other element has the bits of the run without it, and those columns hold
    what one term of that kind gives."""
    rng = np.random.RandomState(n + d + row)
    Q, K, V = (torch.from_numpy(rng.randn(1, h, n, d).astype(np.float32)).cuda() for h in (Hq, Hkv, Hkv))
    cols = [3, d - 1]
    ctx = binding.D2O(1, 1, Hq, Hkv, d, n, n + 2, dtype="f32")
    out = []
    for value in (None, bad):
        Vv = V.clone()
        if value is not None:
            Vv[0, 0, row, cols] = value
        O = torch.empty(1, Hq, n, d, device="cuda:0")
        ctx.d2o_reset()
        ctx.d2o_prefill_attend(0, Q, K, Vv, O)
        out.append(O[0].cpu())
    ctx.close()
    clean, got = out
    assert torch.isfinite(clean).all()
    hit = torch.zeros(Hq, n, d, dtype=torch.bool)
    hit[:Hq // Hkv, row:, cols] = True
    want = torch.full_like(got, bad)     # every softmax weight of these inputs is positive
    assert torch.equal(got[~hit], clean[~hit])
    assert torch.equal(got[hit].nan_to_num(7.0), want[hit].nan_to_num(7.0))


def _imported_state(ctx, g, dtype, storage, Hkv, d, count, n0):
    """`count` survivors of an n0-token prompt in every head of layer 0, and the oracle's copies."""
    caches = []
    for h in range(Hkv):
        K, V = (ref.round_storage(g.standard_normal((count, d)), dtype) for _ in range(2))
        score = 1.0 + g.random(count)
        pos = np.sort(g.choice(n0, count, replace=False)).astype(np.int32)
        ctx.d2o_cache_import(0, 0, h, K, V, score, pos, 0.1, n0)
        K, V = ref.round_storage(K, storage), ref.round_storage(V, storage)
        caches.append(ref.HeadCache(K, V, score.copy(), pos.astype(np.int64), 0.1, storage))
    return caches


@pytest.mark.parametrize("G", [1, 2, 4, 8])
@pytest.mark.parametrize("dtype,d,fp8", [("bf16", 128, False), ("bf16", 128, True), ("f32", 64, False), ("f32", 128, False)])
def test_generation_step_at_the_edges_of_its_tiles(dtype, d, fp8, G):
    """Every form of the K pass (operand vectors in groups of four and left over, an operand copy per wavefront
    or per workgroup, every element type), at entry counts around its wavefront (64) and chunk (256) and around
    the rows that the second pass over the keys takes per round (32 to 128).  An imported cache has
    no candidates, so the first step makes that second pass; the next two do not."""
    storage, Hkv, beta, steps = ("fp8" if fp8 else dtype), 2, 0.7, 3
    for total in (2, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 321):
        budget, n0 = total - 1, 400
        g = np.random.default_rng(1000 * G + total)
        ctx = binding.D2O(1, 1, G * Hkv, Hkv, d, n0, budget + 8, dtype=dtype, beta=beta, out_f32=True, cache_fp8=fp8)
        ctx.d2o_layer_reserve(0, n0, budget, 0)
        caches = _imported_state(ctx, g, dtype, storage, Hkv, d, budget, n0)
        x = [ref.round_storage(g.standard_normal((steps, 1, 1, h, d)), dtype) for h in (G * Hkv, Hkv, Hkv)]
        q, k, v = (torch.from_numpy(a).to(torch.float32 if dtype == "f32" else torch.bfloat16).cuda() for a in x)
        out = torch.empty(1, 1, G * Hkv, d, device="cuda:0")
        for t in range(steps):
            ctx.d2o_decode_step(0, 1, q[t], k[t], v[t], out)
            ev, tg, us = ctx.d2o_last_events(0)
            got = out[0, 0].double().cpu().numpy()
            for h in range(Hkv):
                want, e = ref.decode_step_head(caches[h], x[0][t, 0, 0, h * G:(h + 1) * G], x[1][t, 0, 0, h], x[2][t, 0, 0, h],
                                               n0 + t, budget, 0, 0, beta)
                assert (ev[0, h], tg[0, h]) == (e.evicted_pos, e.target_pos), f"total {total} step {t} head {h}"
                assert e.evicted_pos >= 0 and abs(us[0, h] - e.u_star) < 1e-13
                assert H.rownorm_err(got[h * G:(h + 1) * G], want) <= H.FLOAT_TOL, f"total {total} step {t} head {h}"
        assert ctx.d2o_candidate_misses() >= Hkv
        for h, cache in enumerate(caches):
            gK, gV, gs, gp, gtau = ctx.d2o_cache_export(0, 0, h, budget + 1)
            assert np.array_equal(gp, cache.pos) and np.array_equal(gK, cache.K) and np.array_equal(gV, cache.V)
            np.testing.assert_allclose(gs, cache.score, rtol=1e-12)
            assert abs(gtau - cache.tau) < 1e-13
        ctx.close()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("tau_force", [float("nan"), float("-inf")])
def test_an_evicted_key_that_is_not_finite_merges_into_nothing(dtype, tau_force):
    """Its cosines are NaN (inf / inf), which no threshold admits, also where everything is to be merged: the
    oracle's targets and flags, and the other evicted tokens' merges unchanged."""
    n, budget, recent, d, bad = 300, 100, 20, 128, 57
    g = np.random.default_rng(9)
    K, V = (ref.round_storage(g.standard_normal((n, d)), dtype) for _ in range(2))
    score = g.random(n).astype(np.float32)
    score[bad] = 0.0
    K[bad, 5] = np.inf
    ctx = binding.D2O(1, 1, 1, 1, d, n, budget + 8, dtype=dtype, tau_force=tau_force)
    Kg, Vg = (torch.from_numpy(x)[None, None].to(torch.float32 if dtype == "f32" else torch.bfloat16).cuda() for x in (K, V))
    ctx.d2o_scores_import(0, score[None, None])
    ctx.d2o_compress_layer(0, Kg, Vg, budget, recent)
    with np.errstate(invalid="ignore"):
        cache, want = ref.compress_head(K, V, score.astype(np.float64), budget, recent, 0, dtype, tau_force)
    ret, evi, tgt, us, ps = ctx.d2o_prefill_events(0, 0, 0, n)
    row = int(np.flatnonzero(evi == bad)[0])
    assert np.isnan(us[row]) and not ps[row] and ps.any() == (tau_force == float("-inf"))
    assert np.array_equal(ret, want.retained) and np.array_equal(tgt, want.target) and np.array_equal(ps, want.passed)
    gK, gV = ctx.d2o_cache_export(0, 0, 0, budget + 1)[:2]
    assert H.rownorm_err(gK, cache.K) <= H.FLOAT_TOL and H.rownorm_err(gV, cache.V) <= H.FLOAT_TOL
    ctx.close()


@pytest.mark.parametrize("split_rows", [0, 256])
@pytest.mark.parametrize("cache_fp8", [False, True])
def test_a_head_whose_scores_are_nan_stays_inside_its_cache(cache_fp8, split_rows):
    """A NaN in one query makes every score of its KV head NaN; no entry then compares as the lowest, and every
    step drops the token it brought.  Everything beside that head has the bytes of the run without the NaN: the
    layer before it (whose last slot precedes the head's first), the other heads, the densities."""
    L, Hkv, d, budget, n0, steps = 2, 2, 128, 600, 700, 4
    res = []
    for poison in (False, True):
        g = np.random.default_rng(3)
        ctx = binding.D2O(1, L, Hkv, Hkv, d, n0, L * (budget + 8), dtype="bf16", tau_force=float("-inf"), out_f32=True,
                          cache_fp8=cache_fp8, split_rows=split_rows)
        for l in range(L):
            ctx.d2o_layer_reserve(l, n0, budget, 0)
            for h in range(Hkv):
                K, V = (ref.round_storage(g.standard_normal((budget, d)), "bf16") for _ in range(2))
                ctx.d2o_cache_import(l, 0, h, K, V, 1.0 + g.random(budget), np.arange(budget, dtype=np.int32), 0.1, n0)
        q, k, v = (torch.from_numpy(g.standard_normal((steps, L, 1, Hkv, d))).to(torch.bfloat16).cuda() for _ in range(3))
        if poison:
            q[0, 1, 0, 0, 7] = float("nan")
        out = torch.empty(L, 1, Hkv, d, device="cuda:0")
        outs, events = [], []
        for t in range(steps):
            ctx.d2o_decode_step(0, L, q[t], k[t], v[t], out)
            outs.append(out.cpu().clone())
            events.append([ctx.d2o_last_events(l) for l in range(L)])
        caches = {(l, h): ctx.d2o_cache_export(l, 0, h, budget + 1) for l in range(L) for h in range(Hkv)}
        res.append((outs, events, caches, ctx.d2o_get_density()))
        ctx.close()
    (o0, e0, c0, f0), (o1, e1, c1, f1) = res
    assert np.array_equal(f0, f1, equal_nan=True)
    for t in range(steps):
        assert e1[t][1][0][0, 0] == n0 + t                      # the poisoned head evicts the new token
        for l, h in ((0, 0), (0, 1), (1, 1)):
            assert torch.equal(o0[t][l, 0, h], o1[t][l, 0, h])
            assert all(np.array_equal(x[0, h], y[0, h]) for x, y in zip(e0[t][l], e1[t][l]))
    for lh in ((0, 0), (0, 1), (1, 1)):
        assert all(np.array_equal(x, y, equal_nan=True) for x, y in zip(c0[lh], c1[lh]))
    K, V, s, p, _ = c1[(1, 0)]
    assert np.isnan(s).all() and np.array_equal(np.sort(p), np.arange(budget)) and np.isfinite(K).all() and np.isfinite(V).all()


@pytest.mark.parametrize("total", [1, 2, 63, 64, 65, 256, 257, 2049, 4095, 4096, 4097, 4353])
@pytest.mark.parametrize("dtype,d,G", [("bf16", 128, 1), ("bf16", 128, 2), ("bf16", 128, 4), ("f32", 64, 1), ("f32", 128, 4)])
def test_closing_work_of_heads_of_any_number_of_chunks(dtype, d, G, total):
    """Output rows, scores and the evicted token at the edges of the forms of a head's closing work: one sub-chunk and one chunk,
    as many chunks as there are groups of threads, one more, the last head whose wavefronts close it each
    for itself (64 sub-chunks) and the first beyond; an infinite element of V in the last chunk."""
    Hkv, n, bad = 3, total - 1, 3
    g = np.random.default_rng(total + G)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    ctx = binding.D2O(1, 1, G * Hkv, Hkv, d, 4480, total + 16, dtype=dtype, out_f32=True, beta=0.7)
    ctx.d2o_layer_reserve(0, 4480, max(n, 1), 0)  # full: a token leaves, unless the cache is empty
    caches = []
    for h in range(Hkv):
        K, V = (ref.round_storage(g.standard_normal((n, d)), dtype) for _ in range(2))
        if h == 0 and n:
            V[n - 1, bad] = np.inf
        score, pos = 1.0 + g.random(n), np.arange(n)
        if n:
            ctx.d2o_cache_import(0, 0, h, K, V, score, pos.astype(np.int32), 0.1, n)
        caches.append(ref.HeadCache(K, V, score.copy(), pos.astype(np.int64), 0.1 if n else float("nan"), dtype))
    x = [ref.round_storage(g.standard_normal((1, 1, h, d)), dtype) for h in (G * Hkv, Hkv, Hkv)]
    out = torch.empty(1, 1, G * Hkv, d, device="cuda:0")
    next_pos = n if n else 4480
    cache_v = [np.r_[c.V[np.isfinite(c.V)], x[2][0, 0, h]] for h, c in enumerate(caches)]
    ctx.d2o_decode_step(0, 1, *(torch.from_numpy(a).to(tdt).cuda() for a in x), out)
    got = out[0, 0].double().cpu().numpy()
    for h, cache in enumerate(caches):
        with np.errstate(invalid="ignore"):
            want, _ = ref.decode_step_head(cache, x[0][0, 0, h * G:(h + 1) * G], x[1][0, 0, h], x[2][0, 0, h], next_pos, max(n, 1), 0, 0, 0.7)
        cols = np.arange(d) != bad if h == 0 and n else np.arange(d) >= 0
        assert np.isinf(got[h * G:(h + 1) * G, ~cols]).all()
        # (64 rows, 3 terms, 4 wavefronts, up to 18 chunks, each a rounding of at most max |v|)
        vmax = np.abs(cache_v[h]).max()
        assert np.abs(got[h * G:(h + 1) * G, cols] - want[:, cols]).max() <= 90 * 2.0 ** -24 * vmax
        sc, ps = ctx.d2o_cache_export(0, 0, h, total + 1)[2:4]
        order = np.argsort(cache.pos)
        assert np.array_equal(ps, cache.pos[order])
        np.testing.assert_allclose(sc, cache.score[order], rtol=1e-13)
    ctx.close()


@pytest.mark.parametrize("G", [1, 2, 4, 8])
@pytest.mark.parametrize("fp8", [False, True])
def test_generation_step_outputs_to_fp32_accuracy(fp8, G):
    """P V multiplies on the matrix core with every fp32 probability as three bf16 terms.  The products are
    exact; an output passes through the sums of 64 rows, 3 terms, 4 wavefronts and the chunks, about 75
    roundings of 2^-24 of a value of at most max |v|, and the probability and the chunk's factor are rounded
    once each: 5e-6 max |v|.  Entry counts around the wavefront (64 rows) and the chunk (256), values at both
    ends of the range (the terms of a small probability times a small row must not be lost)."""
    storage, Hkv, d = ("fp8" if fp8 else "bf16"), 2, 128
    for total, vscale in ((1, 1.0), (2, 1.0), (63, 1.0), (64, 1.0), (65, 1.0), (257, 1.0), (700, 1.0), (130, 1e-30), (130, 1e30)):
        g = np.random.default_rng(100 * G + total)
        ctx = binding.D2O(1, 1, G * Hkv, Hkv, d, 1024, 1100, dtype="bf16", out_f32=True, cache_fp8=fp8)
        ctx.d2o_layer_reserve(0, 1000, 1000, 0)  # (nothing is evicted)
        caches = []
        for h in range(Hkv):
            K = ref.round_storage(g.standard_normal((total - 1, d)), "bf16")
            V = ref.round_storage(vscale * g.standard_normal((total - 1, d)), "bf16")
            pos, score = np.arange(total - 1, dtype=np.int32), np.ones(total - 1)
            ctx.d2o_cache_import(0, 0, h, K, V, score, pos, 0.1, 1000)
            caches.append(ref.HeadCache(ref.round_storage(K, storage), ref.round_storage(V, storage), score.copy(),
                                        pos.astype(np.int64), 0.1, storage))
        x = [ref.round_storage(s * g.standard_normal((1, 1, h, d)), "bf16") for h, s in ((G * Hkv, 2.0), (Hkv, 1.0), (Hkv, vscale))]
        out = torch.empty(1, 1, G * Hkv, d, device="cuda:0")
        ctx.d2o_decode_step(0, 1, *(torch.from_numpy(a).to(torch.bfloat16).cuda() for a in x), out)
        got = out[0, 0].double().cpu().numpy()
        for h, cache in enumerate(caches):
            want, _ = ref.decode_step_head(cache, x[0][0, 0, h * G:(h + 1) * G], x[1][0, 0, h], x[2][0, 0, h], 1000, 1000, 0, 0, 0.7)
            err = np.abs(got[h * G:(h + 1) * G] - want).max() / np.abs(cache.V).max()
            assert err <= 5e-6, f"total {total} scale {vscale} head {h}: {err}"
        ctx.close()


@pytest.mark.parametrize("G", [4, 8])
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("value", [float("inf"), float("-inf")])
def test_generation_step_with_an_infinite_value(dtype, d, G, value):
    """One infinite element of V makes its column infinite, with its sign, and leaves the others alone: in the row with the
    largest logit and in others, first and last of the cache, in the middle of it, and the new token's."""
    Hkv, n = 4, 300
    g = torch.Generator().manual_seed(d + G)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    q, K, V = (torch.randn(1, h, t, d, generator=g).to(dt) for h, t in ((Hkv * G, 1), (Hkv, n + 1), (Hkv, n + 1)))
    rows = [0, 77, n - 1, n]
    for h, r in enumerate(rows):
        K[0, h, r] = 0.5 * q[0, h * G, 0]  # the largest logit of the head's first query
        V[0, h, r, r % d] = value
    ctx = binding.D2O(1, 1, Hkv * G, Hkv, d, n, n + 16, dtype=dtype, out_f32=True)
    ctx.d2o_scores_import(0, np.ones((1, Hkv, n), dtype=np.float32))
    ctx.d2o_compress_layer(0, K[:, :, :n].cuda(), V[:, :, :n].cuda(), n + 8, 4)
    out = torch.empty(1, 1, Hkv * G, d, device="cuda:0")
    ctx.d2o_decode_step(0, 1, q[:, :, 0].cuda()[None], K[:, :, n].cuda()[None], V[:, :, n].cuda()[None], out)
    got = out[0, 0].double().cpu().numpy()
    qd, Kd, Vd = (binding.tensor_to_f64(t) for t in (q, K, V))
    for h, r in enumerate(rows):
        logit = qd[0, h * G:(h + 1) * G, 0] @ Kd[0, h].T / np.sqrt(d)
        p = np.exp(logit - logit.max(-1, keepdims=True))
        want = (p / p.sum(-1, keepdims=True)) @ Vd[0, h]
        o, others = got[h * G:(h + 1) * G], np.arange(d) != r % d
        assert np.all(o[:, r % d] == value), f"row {r}: {o[:, r % d]}"
        assert np.abs(o[:, others] - want[:, others]).max() <= H.FLOAT_TOL * np.abs(want[:, others]).max()
    ctx.close()


@pytest.mark.parametrize("G", [1, 4, 8])
@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("gap", [30.0, 87.0, 88.4, 90.5, 200.0])
def test_generation_step_of_large_values_with_small_probabilities(fp8, G, gap):
    """One V row near the end of the number range, its logit `gap` below the others': what it adds to the output, down to
    fp32 probabilities without their full 24 bits, and what it leaves of the other rows' values, which are small beside it.  A
    probability is rounded to fp32 (2^-150 off at most, which the large value multiplies), sums of 41 terms are fp32."""
    d, n, far, large = 128, 40, 11, 2.0 ** 127
    g = torch.Generator().manual_seed(G)
    q, K, V = (torch.randn(1, h, t, d, generator=g) for h, t in ((G, 1), (1, n + 1), (1, n + 1)))
    q[..., 0], K[..., 0] = 64.0, 0.0
    K[0, 0, far] = 0.0
    K[0, 0, far, 0] = -gap * math.sqrt(d) / 64
    V[0, 0, far] = large * torch.linspace(0.5, 1.0, d)
    if gap > 100:
        V[0, 0, :far] *= 1e-6
        V[0, 0, far + 1:] *= 1e-6
    q, K, V = (t.to(torch.bfloat16) for t in (q, K, V))
    ctx = binding.D2O(1, 1, G, 1, d, n, n + 16, dtype="bf16", out_f32=True, cache_fp8=fp8)
    ctx.d2o_scores_import(0, np.ones((1, 1, n), dtype=np.float32))
    ctx.d2o_compress_layer(0, K[:, :, :n].cuda(), V[:, :, :n].cuda(), n + 8, 4)
    out = torch.empty(1, 1, G, d, device="cuda:0")
    ctx.d2o_decode_step(0, 1, q[:, :, 0].cuda()[None], K[:, :, n].cuda()[None], V[:, :, n].cuda()[None], out)
    qd, Kd, Vd = (binding.tensor_to_f64(t)[0] for t in (q, K, V))
    if fp8:
        Kd, Vd = (ref.round_storage(x[0], "fp8")[None] for x in (Kd, Vd))
    logit = qd[:, 0] @ Kd[0].T / np.sqrt(d)
    p = np.exp(logit - logit.max(-1, keepdims=True))
    p /= p.sum(-1, keepdims=True)
    want, got = p @ Vd[0], out[0, 0].double().cpu().numpy()
    bound = 41 * 2.0 ** -24 * (p @ np.abs(Vd[0])) + (2.0 ** -149 * large if gap < 100 else 0.0)
    assert np.all(np.abs(got - want) <= bound), (np.abs(got - want) / bound).max()
    ctx.close()


@pytest.mark.parametrize("n", [60, 200])  # the twins in one 64-row sub-chunk and in two
@pytest.mark.parametrize("dtype,d,G", [("f32", 64, 1), ("f32", 64, 4), ("f32", 128, 1), ("f32", 128, 4), ("bf16", 128, 1)])
def test_the_new_token_ties_with_the_twin_of_its_key(dtype, d, G, n):
    """Eq. 9 takes the first maximum in ascending position: where the new token's key equals a cached one and the evicted
    key lies next to both, the older of the two is its match.  32 heads (the sums of the two rows in different orders
    make the new row's cosine the larger one in a third of them)."""
    B, Hkv, twin, leaves = 2, 16, 20, 50
    g = torch.Generator().manual_seed(n + d + G)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    K, V, k, v = (torch.randn(B, Hkv, t, d, generator=g) for t in (n, n, 1, 1))
    K[:, :, leaves] = K[:, :, twin] + 0.05 * torch.randn(B, Hkv, d, generator=g)
    k[:, :, 0] = K[:, :, twin]
    q = torch.randn(1, B, Hkv * G, d, generator=g)
    score = 100.0 + np.random.default_rng(n).random((B, Hkv, n)).astype(np.float32)
    score[:, :, leaves] = 0.0
    ctx = binding.D2O(B, 1, Hkv * G, Hkv, d, n, n + 8, dtype=dtype, tau_force=float("-inf"), out_f32=True)
    ctx.d2o_scores_import(0, score)
    ctx.d2o_compress_layer(0, K.to(dt).cuda(), V.to(dt).cuda(), n, 4)
    out = torch.empty(1, B, Hkv * G, d, device="cuda:0")
    ctx.d2o_decode_step(0, 1, q.to(dt).cuda(), k[:, :, 0].to(dt).cuda()[None], v[:, :, 0].to(dt).cuda()[None], out)
    evicted, target, _ = ctx.d2o_last_events(0)
    assert np.all(evicted == leaves) and np.all(target == twin), (evicted, target)
    assert ctx.d2o_candidate_misses() == 0
    ctx.close()


@pytest.mark.parametrize("G", [1, 4])
@pytest.mark.parametrize("d", [64, 128])
def test_the_evicted_keys_norm_has_one_order_of_additions(d, G):
    """With fp32 keys a last bit of the evicted key's norm can decide the threshold test of twins, so its squares are added
    by halves of every 64 elements (32, 16, 8, 4, 2 and 1 apart).  The match points along the first axis: its products with
    the evicted key and its own norm are exact, and the similarity is the first element over the evicted key's norm."""
    B, Hkv, n, leaves = 2, 16, 60, 50
    g = torch.Generator().manual_seed(d)
    K, V, v = (torch.randn(B, Hkv, t, d, generator=g) for t in (n, n, 1))
    e = torch.randn(B, Hkv, d, generator=g)
    e[..., 0] = e[..., 0].abs()
    K[:], K[..., 0] = 0.0, -1.0
    K[:, :, 20, 0] = 1.0
    K[:, :, leaves] = e
    q = torch.randn(1, B, Hkv * G, d, generator=g)
    score = 100.0 + np.random.default_rng(n).random((B, Hkv, n)).astype(np.float32)
    score[:, :, leaves] = 0.0
    ctx = binding.D2O(B, 1, Hkv * G, Hkv, d, n, n + 8, dtype="f32", out_f32=True)
    ctx.d2o_scores_import(0, score)
    ctx.d2o_compress_layer(0, K.cuda(), V.cuda(), n, 4)
    out = torch.empty(1, B, Hkv * G, d, device="cuda:0")
    ctx.d2o_decode_step(0, 1, q.cuda(), K[:, :, 0].cuda()[None], v[:, :, 0].cuda()[None], out)
    evicted, _, u = ctx.d2o_last_events(0)
    assert np.all(evicted == leaves) and ctx.d2o_candidate_misses() == 0
    s = e.double().numpy().reshape(B, Hkv, d // 64, 64) ** 2
    for step in (32, 16, 8, 4, 2, 1):
        s = s[..., :step] + s[..., step:2 * step]
    norm = np.sqrt(s.sum((-1, -2)))  # (one or two sums of 64)
    assert np.array_equal(u, e[..., 0].double().numpy() / norm)
    ctx.close()


@pytest.mark.parametrize("B,Hq,Hkv,n", [
    (1, 2, 1, 1), (1, 2, 2, 127), (2, 2, 1, 128), (1, 4, 1, 129), (1, 8, 8, 255), (1, 8, 2, 257), (1, 3, 3, 700),
    (1, 16, 4, 2049),     # 128-row blocks up to the last that the chip holds at once (272), key blocks in pairs
    (1, 16, 4, 2305),     # key blocks of 128 in pairs, with tiles of 128 queries, the last of one
    (2, 64, 16, 700),     # 256-row blocks in pairs with a partial last one
    (2, 128, 16, 513),    # ... and 256-key blocks
])
def test_bf16_prompt_attention_block_edges(B, Hq, Hkv, n):
    """Row blocks of 128 and 256, key blocks of 128 and 256, singly and in pairs, heads in multiples of the
    XCDs and not, against the oracle on up to three KV heads; all scores must add up to the number of rows."""
    d, G = 128, Hq // Hkv
    g = torch.Generator().manual_seed(n + Hq)
    Q, K, V = (torch.randn(B, h, n, d, generator=g).to(torch.bfloat16) for h in (Hq, Hkv, Hkv))
    ctx = binding.D2O(B, 1, Hq, Hkv, d, n, n + 2, dtype="bf16", out_f32=True)
    O = torch.empty(B, Hq, n, d, device="cuda:0")
    ctx.d2o_prefill_attend(0, Q.cuda(), K.cuda(), V.cuda(), O)
    score, (_, var) = ctx.d2o_scores_export(0, n), ctx.d2o_get_density(heads=True)
    Qd, Kd, Vd, got = (binding.tensor_to_f64(t) for t in (Q, K, V, O))
    assert np.abs(score.sum(-1) / (G * n) - 1.0).max() < 1e-5
    for b, h in {(0, 0), (B - 1, Hkv - 1), (0, Hkv // 2)}:
        o, s, v = ref.prefill_kv_head(Qd[b, h * G:(h + 1) * G], Kd[b, h], Vd[b, h])
        assert H.rownorm_err(got[b, h * G:(h + 1) * G], o) <= H.FLOAT_TOL
        assert np.abs(score[b, h] - s).max() <= H.FLOAT_TOL * s.max()
        assert np.abs(var[b, 0, h * G:(h + 1) * G] - v).max() <= H.FLOAT_TOL * max(np.max(v), 1e-3)
    ctx.close()


@pytest.mark.parametrize("B,Hq,Hkv,n", [(1, 2, 1, 1), (1, 3, 3, 700), (1, 16, 4, 2049), (2, 64, 16, 700)])
def test_bf16_prompt_outputs_are_the_fp32_ones_rounded(B, Hq, Hkv, n):
    """Both output types come from the same sums: bf16 rows, whose halves two lanes exchange before they are
    stored, hold the fp32 rows rounded to nearest even, single blocks and pairs, rows up to the last alone."""
    g = torch.Generator().manual_seed(n + Hq)
    Q, K, V = (torch.randn(B, h, n, 128, generator=g).to(torch.bfloat16).cuda() for h in (Hq, Hkv, Hkv))
    out = []
    for out_f32 in (True, False):
        ctx = binding.D2O(B, 1, Hq, Hkv, 128, n, n + 2, dtype="bf16", out_f32=out_f32)
        O = torch.full((B, Hq, n + 1, 128), -7.0, dtype=ctx.out_dtype, device="cuda:0")
        ctx.d2o_prefill_attend(0, Q, K, V, O[:, :, :n])
        torch.cuda.synchronize()
        assert (O[:, :, n] == -7.0).all()  # nothing behind the last row
        out.append(O[:, :, :n].contiguous())
        ctx.close()
    assert torch.equal(out[0].to(torch.bfloat16), out[1])


@pytest.mark.parametrize("n", [17, 20, 27, 32])
def test_column_sums_add_a_tile_of_queries_by_halves(n):
    """The order of a score's fp32 additions decides near-tied selections, so it is held exactly: the 32 queries of a
    tile are added by halves (16 apart, 8, 4, 2, 1).  Keys of zeros make every logit zero: the probability of a query is one
    number for all its keys, and the last key's score is the last query's probability alone."""
    ctx = binding.D2O(1, 1, 1, 1, 128, 32, 34, dtype="bf16", out_f32=True)
    x, zero = torch.ones(1, 1, 32, 128, dtype=torch.bfloat16, device="cuda:0"), torch.zeros(1, 1, 32, 128, dtype=torch.bfloat16, device="cuda:0")
    prob = np.zeros(32, dtype=np.float32)
    for i in range(n):
        ctx.d2o_reset()
        ctx.d2o_prefill_attend(0, x[:, :, :i + 1], zero[:, :, :i + 1], x[:, :, :i + 1])
        score = ctx.d2o_scores_export(0, i + 1)[0, 0]
        prob[i] = score[i]
    for key in range(n):
        v = np.where(np.arange(32) >= key, prob, np.float32(0))
        for step in (16, 8, 4, 2, 1):
            v = v[:step] + v[step:2 * step]
        assert score[key] == v[0], f"key {key}: {score[key]} {v[0]}"
    ctx.close()


@pytest.mark.parametrize("dtype,d,fp8", [("bf16", 128, False), ("bf16", 128, True), ("f32", 64, False), ("f32", 128, False)])
@pytest.mark.parametrize("m,G", [(2, 1), (16, 1), (17, 1), (32, 1), (33, 1), (4, 4), (9, 4), (2, 8), (5, 8), (9, 8)])
def test_block_append_of_few_query_tiles(dtype, d, fp8, m, G):
    """One, two, three and more tiles of 16 queries per head, which four, two or one of a workgroup's wavefronts
    share, on caches that end inside the chunk's 64-row groups and at its end."""
    storage = "fp8" if fp8 else dtype
    for budget in (7, 64 - m, 200, 256 - m, 330):
        if budget < 5:
            continue
        _append_against_oracle(dtype, storage, d, G, m, budget, np.arange(400), 400)


@pytest.mark.parametrize("dtype,d,fp8,value", [
    (dtype, d, fp8, value) for dtype, d, fp8 in (("bf16", 128, False), ("bf16", 128, True), ("f32", 64, False))
    for value in (np.inf, 2.0 ** 127, 2.0 ** 110) if not (fp8 and np.isinf(value))])  # (an 8-bit row has no infinities)
@pytest.mark.parametrize("m", [3, 40])  # wavefronts that share a tile, and one per tile
def test_block_append_with_a_value_at_the_end_of_the_range(dtype, d, fp8, value, m):
    """One element of V infinite: its column of the outputs is infinite; near the end of the range: the outputs that 64
    bits give, in that column and in the others, to fp32 accuracy (300 additions; an 8-bit row keeps four bits)."""
    n, row, col = 300, 70, 5
    g = np.random.default_rng(m)
    K, V = (ref.round_storage(g.standard_normal((n, d)), dtype) for _ in range(2))
    V[row, col] = value
    x = [ref.round_storage(g.standard_normal((1, 1, m, d)), dtype) for _ in range(3)]
    ctx = binding.D2O(1, 1, 1, 1, d, 512, 400, dtype=dtype, out_f32=True, max_append=m, cache_fp8=fp8)
    ctx.d2o_layer_reserve(0, 400, n, 0)
    ctx.d2o_cache_import(0, 0, 0, K, V, np.ones(n), np.arange(n, dtype=np.int32), 0.1, n)
    K, V = ctx.d2o_cache_export(0, 0, 0, n)[:2]  # (as stored)
    out = torch.empty(1, 1, m, d, device="cuda:0")
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    ctx.d2o_append_chunk(0, *(torch.from_numpy(a).to(tdt).cuda() for a in x), out)
    got = out[0, 0].double().cpu().numpy()
    new = (x[1][0, 0], x[2][0, 0]) if not fp8 else [ref.round_storage(a[0, 0], "fp8") for a in x[1:]]
    keys, vals = np.r_[K, new[0]], np.r_[V, new[1]]
    others = np.arange(d) != col
    for i in range(m):
        logit = keys[:n + i + 1] @ x[0][0, 0, i] / np.sqrt(d)
        p = np.exp(logit - logit.max())
        p /= p.sum()
        want = p @ vals[:n + i + 1]
        if np.isinf(value):
            assert got[i, col] == np.inf
        else:
            assert abs(got[i, col] - want[col]) <= 300 * 2.0 ** -24 * want[col]
        bound = 300 * 2.0 ** -24 * (p @ np.abs(vals[:n + i + 1]))
        assert (np.abs(got[i, others] - want[others]) <= bound[others]).all()
    ctx.close()


@pytest.mark.parametrize("budget,m,slots", [
    (512, 320, 1024),   # ten tiles of queries at a time
    (7200, 80, 7296),   # four, the fewest
])
def test_block_append_in_several_passes_over_the_queries(budget, m, slots):
    """128 heads whose exponentials take several passes over the query tiles, against one of the heads alone in a single
    pass: the same outputs, and scores equal but for the order in which a row's fp64 sums over the tiles are added."""
    d, Hkv, B = 128, 32, 4
    g = np.random.default_rng(3)
    K, V = (ref.round_storage(g.standard_normal((budget, d)), "bf16") for _ in range(2))
    score = 1.0 + g.random(budget)
    x = [torch.from_numpy(g.standard_normal((1, 1, m, d))).to(torch.bfloat16).cuda() for _ in range(3)]
    got = []
    for b, h in ((1, 1), (B, Hkv)):
        ctx = binding.D2O(b, 1, h, h, d, slots, slots, dtype="bf16", out_f32=True, max_append=m)
        ctx.d2o_layer_reserve(0, budget, budget, 100)
        full = sorted({(0, 0), (b // 2, h // 2), (b - 1, h - 1)})
        for i, j in full:
            ctx.d2o_cache_import(0, i, j, K, V, score, np.arange(budget, dtype=np.int32), 0.1, budget)
        out = torch.empty(b, h, m, d, device="cuda:0")
        ctx.d2o_append_chunk(0, *(t.expand(b, h, m, d).contiguous() for t in x), out)
        got += [(out[i, j].cpu().numpy(), *ctx.d2o_cache_export(0, i, j, budget + m)) for i, j in full]
        ctx.close()
    for other in got[1:]:
        for i in (0, 1, 2, 4):  # outputs, K, V, positions
            assert np.array_equal(got[0][i], other[i])
        np.testing.assert_allclose(other[3], got[0][3], rtol=m * 2.0 ** -53)  # m additions


@pytest.mark.parametrize("positions,next_pos", [
    (np.arange(0, 32768, 7), 32768),           # one word of the set per thread
    (np.arange(0, 200000, 41), 200003),        # seven
    (np.arange(0, 700000, 101), 700001),       # more positions than the set holds: slots compared with each other
])
def test_block_append_ranks_any_positions(positions, next_pos):
    """The position order of a cache, and so the retained, evicted and matched tokens, for small and large
    positions; three generation steps, which move the last slot into a freed one, run first."""
    _append_against_oracle("bf16", "bf16", 128, 1, 20, 150, positions, next_pos, steps=3)


def test_block_append_keeps_rows_whose_positions_lie_behind_the_next_one():
    """An imported cache may hold any positions; ones beyond the largest set are ranked by comparison.  Nothing is
    evicted, so every row must come out of the reordering with its position and score."""
    g, n, m, d = np.random.default_rng(0), 90, 6, 128
    pos = np.sort(np.r_[g.choice(3000, 60, replace=False), 40000 + g.choice(10 ** 6, 30, replace=False)]).astype(np.int32)
    K, V = (ref.round_storage(g.standard_normal((n, d)), "bf16") for _ in range(2))
    ctx = binding.D2O(1, 1, 1, 1, d, 512, 200, dtype="bf16", out_f32=True, max_append=m)
    ctx.d2o_layer_reserve(0, 400, 120, 0)
    ctx.d2o_cache_import(0, 0, 0, K, V, 1.0 + np.arange(n), pos, 0.1, 3000)
    x = [torch.randn(1, 1, m, d).to(torch.bfloat16).cuda() for _ in range(3)]
    ctx.d2o_append_chunk(0, *x, torch.empty(1, 1, m, d, device="cuda:0"))
    gK, gV, gs, gp, _ = ctx.d2o_cache_export(0, 0, 0, 120)
    order = np.argsort(np.r_[pos, 3000 + np.arange(m)], kind="stable")
    assert np.array_equal(gp, np.r_[pos, 3000 + np.arange(m)][order])
    assert np.array_equal(gK, np.r_[K, binding.tensor_to_f64(x[1])[0, 0]][order])
    assert np.array_equal(gV, np.r_[V, binding.tensor_to_f64(x[2])[0, 0]][order])
    old = order < n  # every score has grown by at most the block's probabilities
    grown = gs[old] - (1.0 + order[old])
    assert grown.min() >= 0 and grown.max() <= m and abs(grown.sum() + gs[~old].sum() - m) < 1e-9
    ctx.close()


def test_block_append_where_positions_lie_behind_the_next_one_is_as_fast():
    """A cache of 20000 entries with positions above the one that its import names as the next takes its position order from
    many workgroups or from the set of bits too, never from one workgroup that compares every slot with
    every other (which took 16.8 ms where positions in order take 0.12 and the many workgroups 0.47)."""
    n, m, d = 20000, 4, 128
    g = torch.Generator().manual_seed(5)
    K, V = (torch.randn(n, d, generator=g).to(torch.bfloat16).double().numpy() for _ in range(2))
    x = [torch.randn(1, 1, m, d, generator=g).to(torch.bfloat16).cuda() for _ in range(3)]
    out = torch.empty(1, 1, m, d, device="cuda:0")

    def milliseconds(pos, next_pos):
        ctx = binding.D2O(1, 1, 1, 1, d, n + 128, n + 96, dtype="bf16", out_f32=True, max_append=m)
        ctx.d2o_layer_reserve(0, n, n + 64, 0)
        ctx.d2o_cache_import(0, 0, 0, K, V, np.ones(n), pos.astype(np.int32), 0.1, next_pos)
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
        for e in ev:
            ctx.d2o_append_chunk(0, *x, out)
            e.record()
        torch.cuda.synchronize()
        got = ctx.d2o_cache_export(0, 0, 0, n + 64)[3]
        assert np.array_equal(got, np.sort(np.r_[pos, next_pos + np.arange(4 * m)]))
        ctx.close()
        return min(a.elapsed_time(b) for a, b in zip(ev, ev[1:]))

    milliseconds(np.arange(n), n)
    plain = milliseconds(np.arange(n), n)
    for step in (20, 100):  # inside the set of bits, and beyond it
        behind = milliseconds(np.arange(n) * step + step - 1, 20000)
        assert behind <= 16 * plain, f"positions {step} apart: {behind:.3f} ms, in order {plain:.3f} ms"


def test_captured_block_append_replayed_on_another_cache():
    """A captured append holds the size of the position set of its capture; replayed on a cache that was imported since,
    with positions outside that set, it still keeps every row with its position, in ascending order."""
    n, m, d, end = 90, 6, 128, 3000
    g = np.random.default_rng(1)
    K, V = (ref.round_storage(g.standard_normal((n, d)), "bf16") for _ in range(2))
    ctx = binding.D2O(1, 1, 1, 1, d, 512, 200, dtype="bf16", out_f32=True, max_append=m)
    ctx.d2o_layer_reserve(0, 400, 120, 0)
    x = [torch.randn(1, 1, m, d).to(torch.bfloat16).cuda() for _ in range(3)]
    out = torch.empty(1, 1, m, d, device="cuda:0")
    near, far = np.arange(n), np.sort(40000 + g.choice(10 ** 5, n, replace=False))
    ctx.d2o_cache_import(0, 0, 0, K, V, np.ones(n), near.astype(np.int32), 0.1, end)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ctx.d2o_append_chunk(0, *x, out)
    for pos in (near, far, near, far):
        ctx.d2o_cache_import(0, 0, 0, K, V, np.ones(n), pos.astype(np.int32), 0.1, end)
        graph.replay()
        torch.cuda.synchronize()
        gK, _, _, gp, _ = ctx.d2o_cache_export(0, 0, 0, 120)
        order = np.argsort(np.r_[pos, end + np.arange(m)], kind="stable")
        assert np.array_equal(gp, np.r_[pos, end + np.arange(m)][order])
        assert np.array_equal(gK, np.r_[K, binding.tensor_to_f64(x[1])[0, 0]][order])
    ctx.close()


@pytest.mark.parametrize("m", [4, 24, 48])  # four, two and one of a workgroup's wavefronts per tile of queries
def test_block_append_with_a_group_of_rows_whose_keys_are_nan(m):
    """64 neighbouring cache rows whose keys are all NaN: outputs are NaN, and so are those rows' scores, but the other
    rows keep the scores that the softmax over them gives."""
    n, d, bad = 200, 128, slice(64, 128)
    g = torch.Generator().manual_seed(m)
    K, V = (torch.randn(n, d, generator=g).to(torch.bfloat16).double().numpy() for _ in range(2))
    K[bad] = np.nan
    x = [torch.randn(1, 1, m, d, generator=g).to(torch.bfloat16) for _ in range(3)]
    ctx = binding.D2O(1, 1, 1, 1, d, 512, 300, dtype="bf16", out_f32=True, max_append=m)
    ctx.d2o_layer_reserve(0, 400, n + m, 0)
    ctx.d2o_cache_import(0, 0, 0, K, V, np.zeros(n), np.arange(n, dtype=np.int32), 0.1, n)
    out = torch.empty(1, 1, m, d, device="cuda:0")
    ctx.d2o_append_chunk(0, *(t.cuda() for t in x), out)
    score = ctx.d2o_cache_export(0, 0, 0, n + m)[2]
    keys = np.r_[K, x[1][0, 0].double().numpy()]
    want = np.zeros(n + m)
    good = np.arange(n + m)
    good = good[(good < bad.start) | (good >= bad.stop)]
    for i in range(m):
        seen = good[good <= n + i]
        logit = keys[seen] @ x[0][0, 0, i].double().numpy() / np.sqrt(d)
        p = np.exp(logit - logit.max())
        want[seen] += p / p.sum()
    assert torch.isnan(out).all() and np.isnan(score[bad]).all()
    np.testing.assert_allclose(score[good], want[good], rtol=1e-12)
    ctx.close()


def _append_against_oracle(dtype, storage, d, G, m, budget, positions, next_pos, steps=0):
    Hkv, beta, g = 2, 0.7, np.random.default_rng(m + budget)
    ctx = binding.D2O(1, 1, G * Hkv, Hkv, d, 512, budget + m + 8, dtype=dtype, beta=beta, out_f32=True, max_append=m,
                      cache_fp8=storage == "fp8")
    ctx.d2o_layer_reserve(0, 400, budget, budget // 4)
    caches, tdt = [], torch.float32 if dtype == "f32" else torch.bfloat16
    for h in range(Hkv):
        K, V = (ref.round_storage(g.standard_normal((budget, d)), dtype) for _ in range(2))
        score, pos = 1.0 + g.random(budget), np.sort(g.choice(positions, budget, replace=False)).astype(np.int32)
        if positions.max() < next_pos:  # (the recent window holds the last positions)
            pos[budget - budget // 4:] = np.arange(next_pos - budget // 4, next_pos)
            pos[:budget - budget // 4] = np.sort(g.choice(positions[positions < next_pos - budget // 4], budget - budget // 4, replace=False))
        ctx.d2o_cache_import(0, 0, h, K, V, score, pos, 0.1, next_pos)
        caches.append(ref.HeadCache(ref.round_storage(K, storage), ref.round_storage(V, storage), score.copy(),
                                    pos.astype(np.int64), 0.1, storage))
    for t in range(steps):
        x = [ref.round_storage(g.standard_normal((1, 1, h, d)), dtype) for h in (G * Hkv, Hkv, Hkv)]
        out = torch.empty(1, 1, G * Hkv, d, device="cuda:0")
        ctx.d2o_decode_step(0, 1, *(torch.from_numpy(a).to(tdt).cuda() for a in x), out)
        for h, cache in enumerate(caches):
            ref.decode_step_head(cache, x[0][0, 0, h * G:(h + 1) * G], x[1][0, 0, h], x[2][0, 0, h], next_pos + t, budget, budget // 4, 0, beta)
    x = [ref.round_storage(g.standard_normal((1, h, m, d)), dtype) for h in (G * Hkv, Hkv, Hkv)]
    out = torch.empty(1, G * Hkv, m, d, device="cuda:0")
    ctx.d2o_append_chunk(0, *(torch.from_numpy(a).to(tdt).cuda() for a in x), out)
    got = out[0].double().cpu().numpy()
    for h, cache in enumerate(caches):
        want, ev = ref.append_chunk_head(cache, x[0][0, h * G:(h + 1) * G], x[1][0, h], x[2][0, h], next_pos + steps, budget,
                                         budget // 4, 0, beta)
        assert H.rownorm_err(got[h * G:(h + 1) * G], want) <= H.FLOAT_TOL, f"budget {budget} head {h}"
        evi, tgt, us, ps = ctx.d2o_append_events(0, 0, h, budget + m)
        assert np.array_equal(evi, ev.evicted) and np.array_equal(tgt, ev.target) and np.array_equal(ps, ev.passed), f"budget {budget} head {h}"
        gK, gV, gs, gp, gtau = ctx.d2o_cache_export(0, 0, h, budget + m)
        assert np.array_equal(gp, cache.pos) and np.array_equal(gK, cache.K) and np.array_equal(gV, cache.V)
        np.testing.assert_allclose(gs, cache.score, rtol=1e-12)
    ctx.close()


# Matching with the rows spread over workgroups of 32 (up to 256 of them) and of 128 (beyond): one row, remainders of
# both tiles, fewer retained keys than wavefronts have sub-tiles for, the last launch of the one kind and the
# first of the other (8 heads x 32 blocks), a padded last tile; with twin retained keys, whose first one wins.
@pytest.mark.parametrize("B,Hkv,n,budget", [
    (1, 1, 33, 32), (1, 2, 40, 7), (1, 1, 65, 32), (1, 2, 97, 33), (2, 3, 700, 191), (1, 1, 3000, 2433), (1, 2, 4000, 64),
    (2, 4, 1124, 100), (2, 4, 1125, 100), (2, 4, 1200, 127), (2, 4, 1200, 128), (2, 4, 1200, 129), (2, 4, 1300, 161)])
def test_matching_of_few_and_of_many_rows(B, Hkv, n, budget):
    g = np.random.default_rng(n + budget)
    K, V = (ref.round_storage(g.standard_normal((B, Hkv, n, 128)), "bf16") for _ in range(2))
    score = g.random((B, Hkv, n)).astype(np.float32)
    top = np.argsort(-score[..., :n - 1], axis=-1)[..., :4]  # (the last position is retained as the recent one)
    if budget > 8:
        for b in range(B):
            for h in range(Hkv):
                K[b, h, top[b, h, 1]] = K[b, h, top[b, h, 0]]
                K[b, h, top[b, h, 3]] = K[b, h, top[b, h, 0]]
    ctx = binding.D2O(B, 1, Hkv, Hkv, 128, n, budget + 8, dtype="bf16")
    ctx.d2o_scores_import(0, score)
    ctx.d2o_compress_layer(0, *(torch.from_numpy(x).to(torch.bfloat16).cuda() for x in (K, V)), budget, 1)
    for b in range(B):
        for h in range(Hkv):
            ret, evi, tgt, _, _ = ctx.d2o_prefill_events(0, b, h, n)
            assert len(ret) == budget and len(evi) == n - budget
            x = K[b, h].astype(np.float64)
            norm = np.sqrt((x * x).sum(-1))
            cos = (x[evi] @ x[ret].T) / (norm[evi][:, None] * norm[ret][None, :])
            assert np.array_equal(tgt, ret[cos.argmax(-1)]), f"sequence {b} head {h}"
    ctx.close()


@pytest.mark.parametrize("copies", [2, 8, 9])  # a row's list of candidates: short, full, too long (searched exhaustively)
@pytest.mark.parametrize("Hkv,n,budget", [(1, 300, 90), (3, 300, 90), (2, 1500, 333), (9, 1300, 90), (70, 900, 90)])
def test_matching_where_every_row_has_equal_candidates(Hkv, n, budget, copies):
    """Every retained key `copies` times over, so that every evicted row is flagged: launches of few and of many
    rows, more flagged rows than a launch has places for at once; a key of zeros on either side."""
    g = np.random.default_rng(n + copies)
    K, V = (ref.round_storage(g.standard_normal((1, Hkv, n, 128)), "bf16") for _ in range(2))
    score = g.random((1, Hkv, n)).astype(np.float32)
    kept = np.sort(np.argsort(-score[..., :n - 1], axis=-1)[..., :budget - 1], axis=-1)
    for h in range(Hkv):
        K[0, h, kept[0, h]] = K[0, h, kept[0, h]][g.permutation(budget - 1) % -(-budget // copies)]
        K[0, h, kept[0, h, 5]] = 0.0
        K[0, h, np.setdiff1d(np.arange(n - 1), kept[0, h])[7]] = 0.0
    ctx = binding.D2O(1, 1, Hkv, Hkv, 128, n, budget + 8, dtype="bf16")
    ctx.d2o_scores_import(0, score)
    ctx.d2o_compress_layer(0, *(torch.from_numpy(x).to(torch.bfloat16).cuda() for x in (K, V)), budget, 1)
    for h in range(Hkv):
        ret, evi, tgt, us, _ = ctx.d2o_prefill_events(0, 0, h, n)
        want, at = ref.match(K[0, h][evi], K[0, h][ret])
        assert np.array_equal(tgt, ret[at]) and np.allclose(us, want, rtol=0, atol=1e-14)
    ctx.close()


@pytest.mark.parametrize("tied", [[0], [5]])  # the only head; one of eight
def test_matching_of_a_head_whose_rows_all_tie_takes_the_whole_chip(tied):
    """Every row of a head flagged, each with more candidates than a list holds: more rows than the head's own workgroups take
    at once.  The first of equal keys wins, and the time is that of this head's work: eight such heads take longer."""
    n, budget, copies = 8192, 1638, 9
    g = torch.Generator().manual_seed(tied[0])

    def matched(Hkv, heads):
        K, V = (torch.randn(1, Hkv, n, 128, generator=g).to(torch.bfloat16) for _ in range(2))
        score = torch.rand(1, Hkv, n, generator=g)
        for h in heads:
            kept = score[0, h, :n - 1].argsort(descending=True)[:budget - 1].sort().values
            K[0, h, kept] = K[0, h, kept][torch.randperm(budget - 1, generator=g) % -(-budget // copies)]
        ctx = binding.D2O(1, 3, Hkv, Hkv, 128, n, 3 * (budget + 8), dtype="bf16")
        ctx.d2o_timing_enable(True)
        ms = []
        for layer in range(3):
            ctx.d2o_scores_import(layer, score.numpy())
            ctx.d2o_timing_read("match_refine")
            ctx.d2o_compress_layer(layer, K.cuda(), V.cuda(), budget, 1)
            ms.append(ctx.d2o_timing_read("match_refine")[0])
        for h in {heads[0], Hkv - 1}:
            ret, evi, tgt, us, _ = ctx.d2o_prefill_events(2, 0, h, n)
            x = K[0, h].double().numpy()
            want, at = ref.match(x[evi], x[ret])
            assert np.array_equal(tgt, ret[at]) and np.allclose(us, want, rtol=0, atol=1e-14)
        ctx.close()
        return min(ms)

    one, eight = matched(8 if tied[0] else 1, tied), matched(8, range(8))
    assert one <= 0.6 * eight, f"one head {one:.3f} ms, eight {eight:.3f} ms"


@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("nret", [1, 5, 8, 31, 33, 63, 64, 90])  # (the padding of the last tile wins, ties with itself, or there is none)
@pytest.mark.parametrize("Hkv,n", [(3, 300), (9, 1300)])  # launches of few and of many rows
def test_matching_against_retained_keys_that_are_not_finite(Hkv, n, nret, value):
    """A head whose retained keys all hold a NaN or an infinity: its evicted tokens match the first retained key (NaN: with
    similarity 0, infinity: with none), never a row behind the last one, and the other heads' caches are those that they are
    beside a finite head.  In another head one evicted key is NaN."""
    g = np.random.default_rng(nret)
    K, V = (ref.round_storage(g.standard_normal((1, Hkv, n, 128)), "bf16") for _ in range(2))
    score = g.random((1, Hkv, n)).astype(np.float32)
    order = [np.argsort(-score[0, h, :n - 1]) for h in range(Hkv)]
    K[0, 2, order[2][-1], 9] = np.nan
    others = []
    for bad in (False, True):
        if bad:
            K[0, 1, np.r_[order[1][:nret - 1], n - 1], 77] = value
        ctx = binding.D2O(1, 1, Hkv, Hkv, 128, n, nret + 8, dtype="bf16")
        ctx.d2o_scores_import(0, score)
        ctx.d2o_compress_layer(0, *(torch.from_numpy(x).to(torch.bfloat16).cuda() for x in (K, V)), nret, 1)
        for h in range(Hkv):
            ret, evi, tgt, us, ps = ctx.d2o_prefill_events(0, 0, h, n)
            with np.errstate(invalid="ignore"):
                want, at = ref.match(K[0, h][evi], K[0, h][ret])
                passed = ref.prefill_threshold(want)[1]
            assert np.array_equal(tgt, ret[at]) and np.allclose(us, want, rtol=0, atol=1e-14, equal_nan=True), f"head {h}"
            if h == 1 and bad:
                assert np.array_equal(ps, passed)
        others.append([ctx.d2o_cache_export(0, 0, h, nret) for h in range(Hkv) if h != 1])
        ctx.close()
    for a, b in zip(*others):
        assert all(np.array_equal(x, y, equal_nan=True) for x, y in zip(a, b))


@pytest.mark.parametrize("fp8", [False, True])
def test_attention_beside_the_compression_of_another_layer(fp8):
    """Attention and compression keep no scratch memory in common: layer 1's attention (grouped queries) on one stream,
    layer 0's compression on another, with keys in pairs of twins so that the matching's lists are in use, give the
    bits of the same calls one after the other."""
    Hq, Hkv, n, budget = 32, 8, 2048, 500
    g = torch.Generator().manual_seed(11)
    x = [[torch.randn(1, h, n, 128, generator=g).to(torch.bfloat16) for h in (Hq, Hkv, Hkv)] for _ in range(2)]
    for _, K, _ in x:
        K[:, :, n // 2:] = K[:, :, :n // 2]
    x = [[t.cuda() for t in layer] for layer in x]
    ctx = binding.D2O(1, 2, Hq, Hkv, 128, n, 2 * budget + 8, dtype="bf16", cache_fp8=fp8)
    streams = [torch.cuda.Stream() for _ in range(2)]

    def results():
        torch.cuda.synchronize()
        out = [ctx.d2o_scores_export(l, n) for l in range(2)]
        out += [a for h in range(Hkv) for a in ctx.d2o_prefill_events(0, 0, h, n)]
        ctx.d2o_compress_layer(1, x[1][1], x[1][2], budget, 100)
        for l in range(2):
            for h in range(Hkv):
                out += [np.asarray(a) for a in ctx.d2o_cache_export(l, 0, h, budget + 1)]
        return out

    ctx.d2o_prefill_attend(0, *x[0])
    ctx.d2o_prefill_attend(1, *x[1])
    ctx.d2o_compress_layer(0, x[0][1], x[0][2], budget, 100)
    want = results()
    for _ in range(3):
        ctx.d2o_reset()
        ctx.d2o_prefill_attend(0, *x[0])
        torch.cuda.synchronize()
        with torch.cuda.stream(streams[0]):
            ctx.d2o_prefill_attend(1, *x[1])
        with torch.cuda.stream(streams[1]):
            ctx.d2o_compress_layer(0, x[0][1], x[0][2], budget, 100)
        for got, first in zip(results(), want):
            assert np.array_equal(got, first, equal_nan=True)
    ctx.close()
