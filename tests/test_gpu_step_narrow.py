"""kvq_append_decode_attention of a block without a window that stands below 16 bits: the launch quantizes the new token into the
block's width itself.  Stored bytes, scales and zero points are those of kvq_quantize_append(_rope), bit for bit; the attention of the
step is that of the two calls up to the rounding of probabilities (the token is attended to in fp32 instead of fp16)."""
import numpy as np
import pytest
import torch

import paper_2505_18610_amd as kq
from gpu_util import MAX_ABS, REL_L2, append_both, assert_same_cache, dev, make_pair
from oracle.attention import decode_attention_fp64

pytestmark = pytest.mark.gpu


def _pair(bits, group, tier16, page, start, heads, kv, batch, reparam, seed):
    g = torch.Generator("cuda").manual_seed(seed)
    caches = []
    lam = (1.0 + 3.0 * torch.rand(kv, 128, generator=g, device="cuda")).contiguous()
    k, v = (torch.randn(batch, kv, start, 128, generator=g, device="cuda").half() for _ in range(2))
    for _ in range(2):
        cfg = kq.KvqConfig(1, batch, heads * kv, kv, start + 200, page_tokens=page, policy=kq.KVQ_POLICY_PAPER, group=group)
        arena = torch.full((kq.kvq_arena_bytes(cfg, 32 << 20),), 0xEE, dtype=torch.uint8, device="cuda")
        c = kq.KvqCache(cfg, [1 << 50], [2], arena=arena)
        c.kvq_cache_set_option(kq.KVQ_OPT_TIER16, tier16)
        c.kvq_cache_set_option(kq.KVQ_OPT_DETERMINISTIC, 1)
        if reparam:
            c.kvq_cache_set_reparam(0, lam)
        c.kvq_quantize_append(0, k, v, bits)
        caches.append(c)
    return caches, g


def _same_contents(a, b):
    assert a.kvq_cache_describe(0) == b.kvq_cache_describe(0)
    for i in range(len(a.kvq_cache_describe(0)[0])):
        for which in (0, 1):
            for x, y in zip(a.kvq_cache_export_segment(0, i, which), b.kvq_cache_export_segment(0, i, which)):
                assert (x is None and y is None) or np.array_equal(x.view(np.uint8), y.view(np.uint8)), (i, which)


@pytest.mark.parametrize("bits", [8, 4, 2])
@pytest.mark.parametrize("group,tier16,page,start,heads,kv,batch,rope,reparam", [
    (32, 0, 32, 1, 1, 1, 1, False, False),       # one older token; every 32nd step starts a page
    (64, 0, 64, 61, 5, 2, 1, True, False),       # across a tile and a page
    (128, 0, 96, 94, 8, 1, 2, True, True),       # pages of an odd number of tiles
    (128, 1, 64, 700, 4, 2, 1, False, True),     # integer tier
    (32, 0, 128, 2048, 16, 4, 1, True, True),    # several ranges, sixteen heads: the storing wavefronts merge heads too
    (32, 1, 128, 20000, 7, 2, 1, True, False),   # streamed ranges
])
def test_step_below_16_bits(bits, group, tier16, page, start, heads, kv, batch, rope, reparam):
    (two, one), g = _pair(bits, group, tier16, page, start, heads, kv, batch, reparam, 7 * start + bits)
    for step in range(36):
        k, v = (torch.randn(batch, kv, 1, 128, generator=g, device="cuda").half() for _ in range(2))
        if step == 3:
            k[..., 0:32] = -k[..., 0:32].abs()            # a group of one sign, a constant one, zeros of both signs
            v[..., 32:64] = 1.5
            v[..., 64:96] = torch.where(v[..., 64:96] > 0, v[..., 64:96], torch.zeros_like(v[..., 64:96]) * -1.0)
            k[..., 96:128] = torch.where(k[..., 96:128] > 0, 0.0, -0.0).half()
        if step == 20:
            v[..., 0:32] *= 20000.0                          # scales of 256 and more: the cache is marked from here on
        q = torch.randn(batch, heads * kv, 128, generator=g, device="cuda").half()
        table = torch.randn(1, 128, generator=g, device="cuda") if rope else None
        outs = [torch.empty(batch, heads * kv, 128, device="cuda") for _ in range(4)]
        if rope:
            two.kvq_quantize_append_rope(0, k, v, table)
        else:
            two.kvq_quantize_append(0, k, v)
        two.kvq_decode_attention(0, q, outs[0])
        one.kvq_append_decode_attention(0, k, v, q, outs[1], cos_sin=table)
        assert one.kvq_cache_describe(0)[0][-1][2] == bits
        two.kvq_decode_attention(0, q, outs[2])
        one.kvq_decode_attention(0, q, outs[3])
        a, b, c, d = (o.cpu().numpy() for o in outs)
        assert np.array_equal(c, d), step                    # the cached block, token included, read alike
        # either way rounds p and p * S_v to fp16, 2^-11 each, of sum p |V|, which is the output's size where the large token dominates: 2^-9 of
        # it.  S_v is of one quantization group: the channels of the others are held to their own size.
        for g0 in range(0, 128, group):
            x, y = a[..., g0:g0 + group], b[..., g0:g0 + group]
            assert np.abs(x - y).max() <= MAX_ABS * max(1.0, float(np.abs(x).max())), (step, g0)
            assert np.linalg.norm(x - y) <= REL_L2 * np.linalg.norm(x), (step, g0)
        if step in (0, 3, 20, 35):
            _same_contents(two, one)


@pytest.mark.parametrize("bits", [8, 4, 2])
@pytest.mark.parametrize("group,tier16,page,start", [
    (32, 0, 64, 30),      # into a tile, across its end
    (64, 1, 64, 62),      # across the end of a page
    (128, 0, 96, 95),
    (32, 1, 32, 700),
])
def test_step_below_16_bits_against_the_oracle(bits, group, tier16, page, start):
    rng = np.random.default_rng(100 * start + bits)
    B, H, G = 2, 2, 3
    oc, gc = make_pair(1, B, H * G, H, start + 64, page, group=group, tier16=tier16)
    draw = lambda *shape: rng.standard_normal(shape, dtype=np.float32).astype(np.float16)
    append_both(oc, gc, 0, draw(B, H, start, 128), draw(B, H, start, 128), bits)
    for step in range(6):
        k, v, q = draw(B, H, 1, 128), draw(B, H, 1, 128), draw(B, H * G, 128)
        if step == 3:
            v[..., 32:64] = (v[..., 32:64].astype(np.float32) * 20000.0).clip(-65504, 65504).astype(np.float16)
        out = torch.empty(B, H * G, 128, device="cuda")
        gc.kvq_append_decode_attention(0, dev(k), dev(v), dev(q), out)
        oc.append(0, k, v)
        got, want = out.cpu().numpy().astype(np.float64), oc.attention(0, q)
        size = np.abs(want)
        if step >= 3:  # (what is rounded: the terms of sum p V, which large ones can make larger than the output.  Their size: all V positive.)
            K, V = oc.dequantized(0)
            size = decode_attention_fp64(q, K, np.abs(V))
        for g0 in range(0, 128, group):
            at = slice(g0, g0 + group)
            assert np.abs(got[..., at] - want[..., at]).max() <= MAX_ABS * max(1.0, size[..., at].max()), (step, g0)
            assert np.linalg.norm(got[..., at] - want[..., at]) <= REL_L2 * np.linalg.norm(size[..., at]), (step, g0)
        if step in (0, 2, 5):
            assert_same_cache(oc, gc, 0)
    gc.close()


@pytest.mark.parametrize("group", [32, 128])
@pytest.mark.parametrize("bits", [8, 4, 2])
def test_step_of_elements_that_are_no_numbers(bits, group):
    """NaN beside numbers is code 0 and leaves attention finite; infinities and groups of NaN alone are stored as the append stores them."""
    (two, one), g = _pair(bits, group, 0, 64, 62, 4, 2, 1, False, 9)
    for step in range(4):
        k, v = (torch.randn(1, 2, 1, 128, generator=g, device="cuda").half() for _ in range(2))
        for x in (k, v):
            x[..., 5::17] = float("nan")
            if step == 1:
                x[..., 7::32] = -x[..., 7::32].abs()
                x[..., 40] = torch.tensor(-443, dtype=torch.int16).view(torch.float16)  # a NaN of the other sign, with a payload
            if step == 2:
                x[:, 0, :, 9], x[:, 1, :, 40] = float("inf"), -float("inf")
            if step == 3:
                x[..., 64:96], x[:, 1, :, 70] = float("nan"), float("inf")
        q = torch.randn(1, 8, 128, generator=g, device="cuda").half()
        outs = [torch.empty(1, 8, 128, device="cuda") for _ in range(2)]
        two.kvq_quantize_append(0, k, v)
        two.kvq_decode_attention(0, q, outs[0])
        one.kvq_append_decode_attention(0, k, v, q, outs[1])
        a, b = (o.cpu().numpy() for o in outs)
        if step < 2:
            assert np.isfinite(b).all() and np.abs(a - b).max() <= MAX_ABS and np.linalg.norm(a - b) <= REL_L2 * np.linalg.norm(a), step
        for which in (0, 1):
            got, want = (c.kvq_cache_export_segment(0, 0, which) for c in (one, two))
            assert np.array_equal(got[0], want[0]), (step, which)
            for x, y in zip(got[1:], want[1:]):
                assert np.array_equal(x.astype(np.float32), y.astype(np.float32), equal_nan=True), (step, which)


def test_steps_and_shrinks_take_turns():
    """Down the widths with steps in between: 16 -> 8 -> 4 -> 2, the last page partly filled at every shrink."""
    (two, one), g = _pair(16, 32, 0, 64, 150, 4, 2, 1, False, 5)
    for step in range(60):
        k, v = (torch.randn(1, 2, 1, 128, generator=g, device="cuda").half() for _ in range(2))
        q = torch.randn(1, 8, 128, generator=g, device="cuda").half()
        outs = [torch.empty(1, 8, 128, device="cuda") for _ in range(2)]
        two.kvq_quantize_append(0, k, v)
        two.kvq_decode_attention(0, q, outs[0])
        one.kvq_append_decode_attention(0, k, v, q, outs[1])
        a, b = (o.cpu().numpy() for o in outs)
        assert np.abs(a - b).max() <= MAX_ABS and np.linalg.norm(a - b) <= REL_L2 * np.linalg.norm(a), step
        if step in (10, 25, 45):
            for c in (two, one):
                c.kvq_progressive_requant(0)
            _same_contents(two, one)
    _same_contents(two, one)


@pytest.mark.parametrize("units,tokens,page", [
    (700, 40, 32),     # more workgroups than the device holds at a time: the first end before the last start
    (700, 700, 64),    # the same, streamed
    (264, 8300, 32),   # ranges of more pages than the kernel looks up at a time
])
def test_step_that_sets_the_mark_of_large_scales(units, tokens, page):
    """The step whose token brings the first V scale of 256 and more does not act on it: every other unit's output is, bit for bit, that of
    the same step without that scale, however the workgroups follow one another.  The calls behind it do act on it."""
    H = 4
    B = units // H
    g = torch.Generator("cuda").manual_seed(units)
    half = tokens // 2
    kv = [torch.randn((B, H, half, 128), device="cuda", generator=g).half() for _ in range(2)]
    k, v = (torch.randn(B, H, 1, 128, generator=g, device="cuda").half() for _ in range(2))
    large = v.clone()
    large[0, 0, 0, 64:96] *= 5000.0
    q = torch.randn(B, H, 128, generator=g, device="cuda").half()
    caches = []
    for _ in range(2):
        cfg = kq.KvqConfig(1, B, H, H, tokens + 64, page_tokens=page, policy=kq.KVQ_POLICY_PAPER, group=32)
        arena = torch.empty(kq.kvq_arena_bytes(cfg, (tokens + 4 * page) * units * 104 + (4 << 20)), dtype=torch.uint8, device="cuda")
        c = kq.KvqCache(cfg, [1 << 50], [2], arena=arena)
        c.kvq_cache_set_option(kq.KVQ_OPT_DETERMINISTIC, 1)
        for _ in range(2):
            c.kvq_quantize_append(0, *kv, 2)
        caches.append(c)
    outs = [torch.empty(B, H, 128, device="cuda") for _ in range(2)]
    for c, token, o in zip(caches, (large, v), outs):
        c.kvq_append_decode_attention(0, k, token, q, o)
    a, b = (o.view(units, 128) for o in outs)
    assert torch.equal(a[1:], b[1:])
    assert torch.equal(a[0, :64], b[0, :64]) and torch.equal(a[0, 96:], b[0, 96:]) and not torch.equal(a[0, 64:96], b[0, 64:96])
    for step in range(3):  # the overflow-proof path is another way to round the same
        for c, o in zip(caches, outs):
            if step == 1:
                c.kvq_append_decode_attention(0, k, v, q, o)
            else:
                c.kvq_decode_attention(0, q, o)
        assert not torch.equal(a[1:], b[1:]), step
        assert (a[1:] - b[1:]).abs().max() <= MAX_ABS, step
        assert torch.isfinite(a).all()
