"""Decode attention where its split plan and merge change course, and the fused append at the edges of tiles and pages."""
import numpy as np
import pytest
import torch

import kvq_synth
import paper_2505_18610_amd as kq
from gpu_util import MAX_ABS, REL_L2, append_both, assert_same_cache, attention_errors, check_attention, dev, make_pair

pytestmark = pytest.mark.gpu


# gqa g leaves 16 // g slot groups: 16 splits per group in the first round of loads, eight more in each further one; a lane
# takes the (max, sum) pairs of four splits 32 apart
@pytest.mark.parametrize("g", [1, 3, 5, 7, 16])
def test_merge_of_any_split_count(g):
    T, P = 128 * 32 - 5, 64
    oc, gc = make_pair(1, 1, 2 * g, 2, T, P)
    K, V = kvq_synth.make_kv(71, 0, 1, 2, 0, T)
    append_both(oc, gc, 0, K[:, :, :2048], V[:, :, :2048], 4)
    append_both(oc, gc, 0, K[:, :, 2048:], V[:, :, 2048:], 16)
    q = kvq_synth.make_q(71, 0, 1, 2 * g, T - 1)
    G = 16 // g
    for splits in sorted({1, 2, 3, G, G + 1, 2 * G + 1, 4 * G + 1, 8 * G + 1, 16 * G, 16 * G + 1, 24 * G + 1, 31, 32, 33, 65, 97, 127, 128}):
        if splits <= 128:
            for fused in (1, 0):
                gc.kvq_cache_set_option(kq.KVQ_OPT_SPLITS, splits)
                gc.kvq_cache_set_option(kq.KVQ_OPT_FUSED_MERGE, fused)
                check_attention(oc, gc, 0, q)
    gc.close()


@pytest.mark.parametrize("g", [9, 12])
def test_merge_beyond_the_first_rounds_with_idle_slots(g):
    """One slot group of 9 or 12 heads: the other slots have no split of their own, also in the rounds beyond the sixteenth."""
    test_merge_of_any_split_count(g)


# 16 tiles a range is the most the kernels for short ranges take: one or two tiles a wavefront, of one width or two, of one page or
# two neighbouring ones (pages of one and of three tiles), with and without queries scaled by factors and V scales of 256 and more
@pytest.mark.parametrize("tier16", [0, 1])
@pytest.mark.parametrize("page", [32, 96])
@pytest.mark.parametrize("scaled", [False, True])
def test_ranges_around_the_longest_short_one(page, tier16, scaled):
    B, Hkv, g = 1, 2, 5
    for tiles in (1, 2, 8, 9, 15, 16, 17, 33):
        T = 32 * tiles - 7
        oc, gc = make_pair(1, B, g * Hkv, Hkv, T + 40, page, policy=1, tier16=tier16)
        if scaled:
            lam = (1.0 + np.random.default_rng(5).random((Hkv, 128)) * 3.0).astype(np.float32)
            oc.set_reparam(0, lam)
            gc.kvq_cache_set_reparam(0, dev(lam))
        K, V = kvq_synth.make_kv(75, 0, B, Hkv, 0, T + 40)
        v_size = 600.0 if scaled else 1.0
        V = (V.astype(np.float32) * v_size).astype(np.float16)
        t = 0
        for i in range(T // page):  # widths change from page to page, now and then not
            append_both(oc, gc, 0, K[:, :, t:t + page], V[:, :, t:t + page], (2, 4, 4, 8, 16, 2, 2)[i % 7])
            t += page
        if t < T:
            append_both(oc, gc, 0, K[:, :, t:T], V[:, :, t:T], 16)
        q = kvq_synth.make_q(75, 0, B, g * Hkv, T - 1)
        for splits in (1, 2, 3, 0):
            if splits > tiles:
                continue
            gc.kvq_cache_set_option(kq.KVQ_OPT_SPLITS, splits)
            out = torch.empty(q.shape, dtype=torch.float32, device="cuda")
            gc.kvq_decode_attention(0, dev(q), out)
            ma, rel = attention_errors(out.cpu().numpy(), oc.attention(0, q))
            assert ma <= MAX_ABS * v_size and rel <= REL_L2, (tiles, splits)
            for _ in range(2 if splits else 9):  # steps of one token, across tiles
                k, v = K[:, :, T:T + 1], V[:, :, T:T + 1]
                oc.append(0, k, v, 0)
                gc.kvq_append_decode_attention(0, dev(k), dev(v), dev(q), out)
                T += 1
                ma, rel = attention_errors(out.cpu().numpy(), oc.attention(0, q))
                assert ma <= MAX_ABS * v_size and rel <= REL_L2, (tiles, splits, T)
        assert_same_cache(oc, gc, 0)
        gc.close()


# of 10 to 12 tiles the first wavefronts take two and the others one
@pytest.mark.parametrize("tier16", [0, 1])
@pytest.mark.parametrize("tiles", [10, 11, 12, 13])
def test_ranges_whose_tiles_are_spread_over_the_wavefronts(tiles, tier16):
    T, page, g = 32 * tiles - 7, 96, 5
    oc, gc = make_pair(1, 1, 2 * g, 2, T + 40, page, policy=1, tier16=tier16)
    K, V = kvq_synth.make_kv(76, 0, 1, 2, 0, T + 40)
    widths = (4, 2, 16) if tiles % 2 else (8, 8, 4)
    t = 0
    for i in range(T // page):
        append_both(oc, gc, 0, K[:, :, t:t + page], V[:, :, t:t + page], widths[i % 3])
        t += page
    append_both(oc, gc, 0, K[:, :, t:T], V[:, :, t:T], 16)
    q = kvq_synth.make_q(76, 0, 1, 2 * g, T - 1)
    gc.kvq_cache_set_option(kq.KVQ_OPT_SPLITS, 1)
    check_attention(oc, gc, 0, q)
    out = torch.empty(q.shape, dtype=torch.float32, device="cuda")
    for _ in range(9):  # into the next tile
        k, v = K[:, :, T:T + 1], V[:, :, T:T + 1]
        oc.append(0, k, v, 0)
        gc.kvq_append_decode_attention(0, dev(k), dev(v), dev(q), out)
        T += 1
        ma, rel = attention_errors(out.cpu().numpy(), oc.attention(0, q))
        assert ma <= MAX_ABS and rel <= REL_L2, T
    assert_same_cache(oc, gc, 0)
    gc.close()


def _us_per_launch(tiles, bits, units, n=40):
    gc = make_pair(1, 1, 4 * units, units, 32 * tiles, 64)[1]
    k = torch.randn((1, units, 32 * tiles, 128), device="cuda").half()
    gc.kvq_quantize_append(0, k, k, bits)
    gc.kvq_cache_set_option(kq.KVQ_OPT_SPLITS, 1)
    q = torch.randn((1, 4 * units, 128), device="cuda").half()
    out = torch.empty((1, 4 * units, 128), device="cuda")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        gc.kvq_decode_attention(0, q, out, stream=side)
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            for _ in range(n):
                gc.kvq_decode_attention(0, q, out, stream=side)
    times = []
    for _ in range(12):
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        graph.replay()
        start.record()
        graph.replay()
        end.record()
        torch.cuda.synchronize()
        times.append(start.elapsed_time(end) * 1000 / n)
    gc.close()
    return min(times)


def test_no_simd_takes_more_tiles_of_a_short_range_than_it_has_to():
    """12 tiles are three for each SIMD, 16 four: 5.6 and 6.6 us.  (Two a wavefront from the first on, the first SIMDs take four: 6.4.)"""
    assert _us_per_launch(12, 2, 8) < 0.93 * _us_per_launch(16, 2, 8)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
@pytest.mark.parametrize("splits", [1, 7])
def test_outputs_that_start_at_any_element(dtype, splits):
    oc, gc = make_pair(1, 1, 10, 2, 480, 32)
    K, V = kvq_synth.make_kv(74, 0, 1, 2, 0, 480)
    append_both(oc, gc, 0, K, V, 8)
    q = kvq_synth.make_q(74, 0, 1, 10, 479)
    want = oc.attention(0, q)
    gc.kvq_cache_set_option(kq.KVQ_OPT_SPLITS, splits)
    for off in (0, 1, 2, 3):
        buf = torch.full((q.size + 8,), -7.0, dtype=dtype, device="cuda")
        out = buf[off:off + q.size].view(q.shape)
        gc.kvq_decode_attention(0, dev(q), out)
        ma, rel = attention_errors(out.float().cpu().numpy(), want)
        assert ma <= MAX_ABS + (1e-3 if dtype == torch.float16 else 0.0) and rel <= REL_L2
        assert (buf[:off] == -7.0).all() and (buf[off + q.size:] == -7.0).all()
    gc.close()


@pytest.mark.parametrize("tiles", [1, 8, 19, 20, 21, 22, 33, 100])
def test_planned_splits(tiles):
    T = 32 * tiles - 3
    oc, gc = make_pair(1, 2, 10, 2, T, 32)
    K, V = kvq_synth.make_kv(72, 0, 2, 2, 0, T)
    wide = 32 * (tiles // 2)
    if wide:
        append_both(oc, gc, 0, K[:, :, :wide], V[:, :, :wide], 2)
    append_both(oc, gc, 0, K[:, :, wide:], V[:, :, wide:], 16)
    check_attention(oc, gc, 0, kvq_synth.make_q(72, 0, 2, 10, T - 1))
    gc.close()


@pytest.mark.parametrize("tier16", [0, 1])
@pytest.mark.parametrize("group", [32, 64, 128])
@pytest.mark.parametrize("batched", [False, True])
def test_fused_append_from_the_first_token_on(tier16, group, batched):
    """The first token of a block, of a tile and of a page, and one in the middle of each; the last token of a page."""
    B, Hkv, g, P, T = 2, 2, 3, 64, 135
    oc, gc = make_pair(1, B, g * Hkv, Hkv, T, P, group=group, tier16=tier16)
    K, V = kvq_synth.make_kv(73, 0, B, Hkv, 0, T)
    V[:, :, 40] *= 50.0
    t = 0
    for stop in (3, 31, 34, 63, 66, 95, 98, 127, 130, T):
        while t < stop:
            k, v, q = K[:, :, t:t + 1], V[:, :, t:t + 1], kvq_synth.make_q(73, 0, B, g * Hkv, t)
            out = torch.full(q.shape, float("nan"), dtype=torch.float32, device="cuda")
            oc.append(0, k, v, 0)
            if batched:
                kq.kvq_append_decode_attention_batch([gc], 0, [dev(k)], [dev(v)], [dev(q)], [out])
            else:
                gc.kvq_append_decode_attention(0, dev(k), dev(v), dev(q), out)
            mx, rl = attention_errors(out.cpu().numpy(), oc.attention(0, q))
            # the bounds of every attention test, the absolute one scaled by the largest value
            assert mx <= MAX_ABS * max(1.0, float(np.abs(V[:, :, :t + 1]).max()) / 4) and rl <= REL_L2, (t, mx, rl)
            t += 1
            if t < stop:  # a bulk append in between: both ways of writing a tile meet in it
                n = min(stop - 1 - t, 29)
                if n > 0:
                    append_both(oc, gc, 0, K[:, :, t:t + n], V[:, :, t:t + n], 0)
                    t += n
        assert_same_cache(oc, gc, 0)
    gc.close()


@pytest.mark.parametrize("tier16", [0, 1])
@pytest.mark.parametrize("deterministic", [0, 1])
@pytest.mark.parametrize("splits", [0, 2, 5, 21, 22])
def test_fused_append_behind_split_ranges(splits, deterministic, tier16):
    """Several ranges, up to one per tile: whoever holds the last tile stores the new token.  An infinite value of the new
    token reaches its own channel and no other one."""
    B, Hkv, g, P, n2, n16 = 1, 2, 4, 64, 640, 33
    K, V = kvq_synth.make_kv(74, 0, B, Hkv, 0, n2 + n16 + 3)
    for special in (False, True) if not tier16 else (False,):
        oc, gc = make_pair(1, B, g * Hkv, Hkv, n2 + 4 * P, P, window=P, tier16=tier16)
        gc.kvq_cache_set_option(kq.KVQ_OPT_SPLITS, splits)
        gc.kvq_cache_set_option(kq.KVQ_OPT_DETERMINISTIC, deterministic)
        append_both(oc, gc, 0, K[:, :, :n2], V[:, :, :n2], 2)
        append_both(oc, gc, 0, K[:, :, n2:n2 + n16], V[:, :, n2:n2 + n16], 16)
        for t in range(n2 + n16, n2 + n16 + (1 if special else 3)):
            k, v, q = K[:, :, t:t + 1], V[:, :, t:t + 1].copy(), kvq_synth.make_q(74, 0, B, g * Hkv, t)
            if special:
                k = np.zeros_like(k)  # a score of 0
                v[..., 5] = np.inf
            else:
                oc.append(0, k, v, 0)
            out = torch.full(q.shape, float("nan"), dtype=torch.float32, device="cuda")
            gc.kvq_append_decode_attention(0, dev(k), dev(v), dev(q), out)
            got = out.cpu().numpy()
            if special:
                assert np.isposinf(got[..., 5]).all() and np.isfinite(np.delete(got, 5, axis=-1)).all()
            else:
                mx, rl = attention_errors(got, oc.attention(0, q))
                assert mx <= MAX_ABS and rl <= REL_L2, (t, mx, rl)
        if not special:
            assert_same_cache(oc, gc, 0)
        gc.close()
