"""Appends of rotated and reparameterized keys at tile and page edges, from inputs that do not start at a multiple of 16 bytes."""
import numpy as np
import pytest
import torch

import kvq_synth
import paper_2505_18610_amd as kq
from gpu_util import append_both, assert_same_cache, check_attention, make_pair
from oracle import calibrate_lambda, rope_rotate_keys

pytestmark = pytest.mark.gpu


def view(x, odd):
    """The array on the device, `odd` elements behind a multiple of 16 bytes, between NaNs."""
    flat = torch.full((x.size + 16,), float("nan"), dtype=torch.from_numpy(x).dtype, device="cuda")
    flat[odd:odd + x.size] = torch.from_numpy(np.ascontiguousarray(x).reshape(-1)).cuda()
    return flat[odd:odd + x.size].view(x.shape)


@pytest.mark.parametrize("odd", [0, 1, 2])
@pytest.mark.parametrize("reparam", [False, True])
@pytest.mark.parametrize("bits,tier16,group", [(16, 0, 32), (16, 1, 32), (16, 1, 128), (8, 0, 64), (4, 0, 128), (2, 0, 32)])
def test_prepared_keys(bits, tier16, group, reparam, odd):
    """Chunks that start and end inside a tile, at its edge and at a page's; the stored cache equals the oracle's bit for bit."""
    B, H, P, T = 2, 2, 64, 300
    K, V = kvq_synth.make_kv(81, 0, B, H, 0, T, rope_base=None)
    K[:, :, 5] = 0.0                     # rotated zeros
    cos, sin = kvq_synth.rope_tables(np.arange(T), 1.0e6)
    table = np.concatenate([cos, sin], 1).astype(np.float32)
    Krot = rope_rotate_keys(K, cos, sin)
    oc, gc = make_pair(1, B, H, H, T, P, group=group, tier16=tier16)
    if reparam:
        lam = calibrate_lambda(Krot[:, :, :64], 0.5)
        oc.set_reparam(0, lam)
        gc.kvq_cache_set_reparam(0, torch.from_numpy(lam).cuda())
    t = 0
    for n in (1, 30, 1, 33, 63, 64, 100, 8):
        oc.append(0, Krot[:, :, t:t + n], V[:, :, t:t + n], bits)
        gc.kvq_quantize_append_rope(0, view(K[:, :, t:t + n], odd), view(V[:, :, t:t + n], odd), view(table[t:t + n], odd), bits)
        t += n
    assert_same_cache(oc, gc, 0)
    gc.close()


@pytest.mark.parametrize("first", [0, 7])
@pytest.mark.parametrize("pages", [1, 2, 127, 128, 129, 200])
def test_page_entries_of_long_appends(pages, first):
    """Up to 128 pages of an append ride in the kernel arguments and are entered into the table by the kernel; more are
    uploaded.  Later calls (an append to the last page, attention, a shrink of everything) find every page."""
    B, H, P = 1, 1, 32
    n = 32 * pages - (first if pages > 1 else first + 3)
    K, V = kvq_synth.make_kv(82, 0, B, H, 0, first + n + 5)
    oc, gc = make_pair(1, B, 2 * H, H, first + n + 5, P)
    t = 0
    for m in [first, n, 5]:
        if m:
            append_both(oc, gc, 0, K[:, :, t:t + m], V[:, :, t:t + m], 16)
            t += m
    q = kvq_synth.make_q(82, 0, B, 2 * H, t)
    check_attention(oc, gc, 0, q)
    for _ in range(2):
        assert gc.kvq_progressive_requant(0, segment=0) == oc.requant(0, segment=0)
        assert_same_cache(oc, gc, 0)
        check_attention(oc, gc, 0, q)
    gc.close()


@pytest.mark.parametrize("bits", [8, 4, 2])
@pytest.mark.parametrize("B,H,T", [(1, 1, 1), (5, 8, 1024), (5, 8, 1025), (4, 16, 1280)])
def test_strings_shared_by_two_wavefronts(bits, B, H, T):
    """Strings (two per tile and unit) quantized by two wavefronts each or by one, depending on their number: 2,560 of them, one tile
    more, and twice as many; a second append continues the partly filled tile."""
    K, V = kvq_synth.make_kv(83, 0, B, H, 0, T + 6)
    oc, gc = make_pair(1, B, H, H, T + 6, 64)
    append_both(oc, gc, 0, K[:, :, :T], V[:, :, :T], bits)
    append_both(oc, gc, 0, K[:, :, T:], V[:, :, T:], bits)
    assert_same_cache(oc, gc, 0)
    gc.close()


def quantize_any(x, b, group):
    """Eq. 1-2 for any fp16 input: minimum and maximum over the elements that are numbers, a NaN quotient rounds to code 0."""
    g = x.astype(np.float32).reshape(x.shape[:-1] + (-1, group))
    with np.errstate(all="ignore"):
        Z, mx = np.fmin.reduce(g, -1), np.fmax.reduce(g, -1)
        S = ((mx - Z) / np.float32((1 << b) - 1)).astype(np.float16)
        r = np.rint((g - Z[..., None]) / S.astype(np.float32)[..., None])
        r = np.where(np.isnan(r) | (S == 0)[..., None], 0, np.clip(r, 0, (1 << b) - 1))
    return r.reshape(x.shape).astype(np.uint16), S, Z


def unpack(codes, b):
    raw = np.ascontiguousarray(codes).view(np.uint8)
    if b == 16:
        return raw.reshape(raw.shape[:-1] + (-1, 2)).astype(np.uint16) @ np.array([1, 256], np.uint16)
    c = (raw[..., None] >> np.arange(0, 8, b, dtype=np.uint8)) & ((1 << b) - 1)
    return c.reshape(raw.shape[:-1] + (-1,)).astype(np.uint16)


@pytest.mark.parametrize("group", [32, 128])
@pytest.mark.parametrize("bits,way", [(16, "append"), (8, "append"), (4, "append"), (2, "append"), (8, "requant")])
def test_elements_that_are_no_numbers(bits, way, group):
    """NaN (code 0) and infinities in groups of ordinary scales, of scales rounded down to a subnormal, whose top codes are
    clamped, and of scale 0."""
    B, H, P, T = 1, 2, 64, 200
    rng = np.random.default_rng(84)
    X = [rng.standard_normal((B, H, T, 128), dtype=np.float32) for _ in range(2)]
    for x in X:
        # tokens 40 ..: steps of 2^-24 up to 1.4 levels' worth: the scale is 2^-24 and the group's maximum above the top level
        top = 1.4 * ((1 << bits) - 1) * 2.0 ** -24
        x[:, :, 40:80] = rng.random((B, H, 40, 128)) * top
        x[:, :, 40:80, ::32] = 0.0
        x[:, :, 40:80, 1::32] = top
        x[:, :, 80:90] = 0.25
        x[:, :, 0:200:3, 5::32] = np.nan
        x[:, :, 1:200:9, 7::16] = np.nan
        x[:, :, 2:200:21, 9] = np.inf
        x[:, :, 5:200:21, 40] = -np.inf
        x[:, :, 8:200:42] = np.nan
    K, V = (x.astype(np.float16) for x in X)
    sign = rng.random(K.shape) < 0.5
    K[np.isnan(K) & sign] = np.array(0xfe55, np.uint16).view(np.float16)  # the other sign, a payload
    _, gc = make_pair(1, B, H, H, T, P, group=group, tier16=1 if bits == 16 else 0)
    dev = lambda x: torch.from_numpy(x).cuda()
    if way == "append":
        for a, b in ((0, 47), (47, 139), (139, 200)):
            gc.kvq_quantize_append(0, dev(K[:, :, a:b].copy()), dev(V[:, :, a:b].copy()), bits)
    else:
        gc.kvq_quantize_append(0, dev(K), dev(V), 16)
        gc.kvq_progressive_requant(0, segment=0)
    for which, x in ((kq.KVQ_WHICH_K, K), (kq.KVQ_WHICH_V, V)):
        codes, S, Z = gc.kvq_cache_export_segment(0, 0, which)
        want, wS, wZ = quantize_any(x, bits, group)
        got = unpack(codes, bits)
        assert np.array_equal(got, want), np.argwhere(got != want)[:5]
        assert np.array_equal(S, wS, equal_nan=True) and np.array_equal(Z.astype(np.float32), wZ, equal_nan=True)
    gc.close()


@pytest.mark.parametrize("rope", [False, True])
@pytest.mark.parametrize("bits,tier16", [(16, 0), (16, 1), (8, 0)])
def test_one_long_append_writes_what_its_pieces_write(bits, tier16, rope):
    """64 units x 6,250 tokens at once (205 MB of keys and values: the routes of inputs beyond the caches, of 98,304 rows and more)
    and in pieces of 1,000: the same arena, byte for byte."""
    B, H, P, T = 8, 8, 128, 6250
    g = torch.Generator(device="cuda").manual_seed(85)
    k, v = (torch.randn((B, H, T, 128), device="cuda", generator=g).half() for _ in range(2))
    table = torch.randn((T, 128), device="cuda", generator=g)
    cfg = kq.KvqConfig(1, B, H, H, T, page_tokens=P)
    arenas = []
    for step in (T, 1000):
        arena = torch.zeros(kq.kvq_arena_bytes(cfg, T * B * H * 640 + (64 << 20)), dtype=torch.uint8, device="cuda")
        gc = kq.KvqCache(cfg, [1 << 50], [2], arena=arena)
        gc.kvq_cache_set_option(kq.KVQ_OPT_TIER16, tier16)
        for t in range(0, T, step):
            piece = [x[:, :, t:t + step].contiguous() for x in (k, v)]
            if rope:
                gc.kvq_quantize_append_rope(0, *piece, table[t:t + step].contiguous(), bits)
            else:
                gc.kvq_quantize_append(0, *piece, bits)
        torch.cuda.synchronize()
        gc.close()
        arenas.append(arena)
    assert torch.equal(*arenas)


@pytest.mark.parametrize("P,B,H", [(96, 3, 5), (224, 2, 3), (32, 2, 7), (1056, 1, 1)])
@pytest.mark.parametrize("bits,tier16", [(16, 0), (16, 1), (8, 0)])
def test_pages_and_heads_of_every_quotient(bits, tier16, P, B, H):
    """Page, tile in the page and reparameterization row come from multiplied quotients; calls that start in later pages, with a
    second page in sight, and factors that differ from head to head.  Bit for bit the oracle's."""
    T = 2 * P + 75
    K, V = kvq_synth.make_kv(85, 0, B, H, 0, T, rope_base=None)
    cos, sin = kvq_synth.rope_tables(np.arange(T), 1.0e4)
    table = np.concatenate([cos, sin], 1).astype(np.float32)
    Krot = rope_rotate_keys(K, cos, sin)
    lam = calibrate_lambda(Krot[:, :, :64], 0.5)
    oc, gc = make_pair(1, B, H, H, T, P, tier16=tier16)
    oc.set_reparam(0, lam)
    gc.kvq_cache_set_reparam(0, torch.from_numpy(lam).cuda())
    t = 0
    for n in (P - 1, 2, P + 9, T - 2 * P - 10):
        oc.append(0, Krot[:, :, t:t + n], V[:, :, t:t + n], bits)
        gc.kvq_quantize_append_rope(0, view(K[:, :, t:t + n], 0), view(V[:, :, t:t + n], 0), view(table[t:t + n], 0), bits)
        t += n
    assert t == T
    assert_same_cache(oc, gc, 0)
    gc.close()


@pytest.mark.parametrize("bits", [8, 4, 2])
@pytest.mark.parametrize("reparam", [False, True])
@pytest.mark.parametrize("T", [480, 511, 608, 640, 736, 768, 1152, 2300])
def test_prepared_keys_of_every_number_of_strings(bits, reparam, T):
    """64 units x T rotated tokens at once (four strings a token: the sizes at which one or two wavefronts take a string, from 1,920
    to 9,216) and in pieces of 96 tokens, which two wavefronts share: the same arena, byte for byte."""
    B, H, P = 8, 8, 64
    g = torch.Generator(device="cuda").manual_seed(86)
    k, v = (torch.randn((B, H, T, 128), device="cuda", generator=g).half() for _ in range(2))
    table = torch.randn((T, 128), device="cuda", generator=g)
    lam = 1 + torch.rand((H, 128), device="cuda", generator=g)
    cfg = kq.KvqConfig(1, B, H, H, T, page_tokens=P)
    arenas = []
    for step in (T, 96):
        arena = torch.zeros(kq.kvq_arena_bytes(cfg, T * B * H * 640 + (64 << 20)), dtype=torch.uint8, device="cuda")
        gc = kq.KvqCache(cfg, [1 << 50], [2], arena=arena)
        if reparam:
            gc.kvq_cache_set_reparam(0, lam)
        for t in range(0, T, step):
            gc.kvq_quantize_append_rope(0, *(x[:, :, t:t + step].contiguous() for x in (k, v)), table[t:t + step].contiguous(), bits)
        torch.cuda.synchronize()
        gc.close()
        arenas.append(arena)
    assert torch.equal(*arenas)


@pytest.mark.parametrize("bits", [8, 4, 2])
@pytest.mark.parametrize("tiles", [121, 122, 123, 124, 127])
def test_rotated_keys_of_idle_workgroups(bits, tiles):
    """Beyond 120 workgroups a unit up to three idle ones follow: the same arena as from calls of 32 tokens, byte for byte."""
    B, H, T = 1, 3, 32 * tiles - 9
    g = torch.Generator(device="cuda").manual_seed(87)
    k, v = (torch.randn((B, H, T, 128), device="cuda", generator=g).half() for _ in range(2))
    table = torch.randn((T, 128), device="cuda", generator=g)
    cfg = kq.KvqConfig(1, B, H, H, T, page_tokens=96)
    arenas = []
    for step in (T, 32):
        arena = torch.zeros(kq.kvq_arena_bytes(cfg, T * B * H * 640 + (64 << 20)), dtype=torch.uint8, device="cuda")
        gc = kq.KvqCache(cfg, [1 << 50], [2], arena=arena)
        for t in range(0, T, step):
            gc.kvq_quantize_append_rope(0, *(x[:, :, t:t + step].contiguous() for x in (k, v)), table[t:t + step].contiguous(), bits)
        torch.cuda.synchronize()
        gc.close()
        arenas.append(arena)
    assert torch.equal(*arenas)


@pytest.mark.parametrize("rope,reparam", [(True, False), (False, True), (True, True)])
@pytest.mark.parametrize("tiles", [32, 33, 36, 37, 40, 41, 44, 45])
def test_prepared_keys_into_16_bits_of_every_number_of_strings(tiles, rope, reparam):
    """64 units x 32 to 45 tiles are 4,096 to 5,760 strings, between which two kernels take turns: the same arena as from pieces of 96
    tokens, byte for byte."""
    B, H, T, P = 8, 8, 32 * tiles - 5, 64
    g = torch.Generator(device="cuda").manual_seed(88)
    k, v = (torch.randn((B, H, T, 128), device="cuda", generator=g).half() for _ in range(2))
    table = torch.randn((T, 128), device="cuda", generator=g)
    lam = 1 + torch.rand((H, 128), device="cuda", generator=g)
    cfg = kq.KvqConfig(1, B, H, H, T, page_tokens=P)
    arenas = []
    for step in (T, 96):
        arena = torch.zeros(kq.kvq_arena_bytes(cfg, T * B * H * 640 + (64 << 20)), dtype=torch.uint8, device="cuda")
        gc = kq.KvqCache(cfg, [1 << 50], [2], arena=arena)
        if reparam:
            gc.kvq_cache_set_reparam(0, lam)
        for t in range(0, T, step):
            kk, vv = (x[:, :, t:t + step].contiguous() for x in (k, v))
            if rope:
                gc.kvq_quantize_append_rope(0, kk, vv, table[t:t + step].contiguous(), 16)
            else:
                gc.kvq_quantize_append(0, kk, vv, 16)
        torch.cuda.synchronize()
        gc.close()
        arenas.append(arena)
    assert torch.equal(*arenas)


def test_time_of_rotated_appends_does_not_depend_on_the_number_of_tiles_beyond_their_work():
    """191 and 192 tiles x 52 units: with every row of the table read by all eight L2 caches 191 took 1.3 times as long."""
    H, L = 52, 8
    k, v = (torch.randn((1, H, 192 * 32, 128), device="cuda").half() for _ in range(2))
    table = torch.randn((192 * 32, 128), device="cuda")
    cfg = kq.KvqConfig(L, 1, H, H, 192 * 32, page_tokens=256)
    arena = torch.empty(kq.kvq_arena_bytes(cfg, L * 192 * 32 * H * 300 + (64 << 20)), dtype=torch.uint8, device="cuda")
    gc = kq.KvqCache(cfg, [1 << 50] * L, [2] * L, arena=arena)

    def best(tiles):
        T = 32 * tiles
        kk, vv = k.view(-1)[:H * T * 128].view(1, H, T, 128), v.view(-1)[:H * T * 128].view(1, H, T, 128)
        times = []
        for _ in range(6):
            gc.kvq_cache_reset(-1)
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for layer in range(L):
                gc.kvq_quantize_append_rope(layer, kk, vv, table[:T], 8)
            end.record()
            torch.cuda.synchronize()
            times.append(start.elapsed_time(end))
        return min(times)

    assert best(191) < 1.15 * best(192)
    gc.close()
