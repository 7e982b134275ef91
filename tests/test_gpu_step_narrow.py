"""kvq_append_decode_attention of a block without a window that stands below 16 bits: the launch quantizes the new token into the
block's width itself.  Stored bytes, scales and zero points are those of kvq_quantize_append(_rope), bit for bit; the attention of the
step is that of the two calls up to the rounding of probabilities (the token is attended to in fp32 instead of fp16)."""
import numpy as np
import pytest
import torch

import paper_2505_18610_amd as kq
from gpu_util import MAX_ABS, REL_L2

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
        # either way rounds p and p * S_v to fp16, 2^-11 each, of sum p |V|, which is the output's size where the large token dominates: 2^-9 of it
        scale = max(1.0, float(np.abs(a).max()))
        assert np.array_equal(c, d), step                    # the cached block, token included, read alike
        assert np.abs(a - b).max() <= MAX_ABS * scale, step
        assert np.linalg.norm(a - b) <= REL_L2 * np.linalg.norm(a), step
        if step in (0, 3, 20, 35):
            _same_contents(two, one)


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
