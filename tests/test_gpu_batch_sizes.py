"""Ragged batches on both sides of the line at which their parameters no longer fit the kernel arguments (16 caches; 320 range ends):
steps and plain attention against the same calls one cache at a time."""
import numpy as np
import pytest
import torch

import paper_2505_18610_amd as kq
from gpu_util import MAX_ABS, REL_L2

pytestmark = pytest.mark.gpu


def _caches(n, tier16, long, seed):
    """Two sets of the same n caches: lengths, widths, heads, page sizes, groups and options differ from cache to cache."""
    sets = ([], [])
    for i in range(n):
        g = torch.Generator("cuda").manual_seed(seed * 100 + i)
        kv, heads, page = (1, 2, 4)[i % 3], (1, 4, 7, 16)[i % 4], (32, 64, 96, 128)[i % 4]
        bulk = page * (i % 5 + (12 if long and i % 4 == 0 else 0))
        newest = (1, 31, 32, 33, page, page + 5)[i % 6]
        T = bulk + newest
        lam = (1.0 + 3.0 * torch.rand(kv, 128, generator=g, device="cuda")).contiguous()
        k, v = (torch.randn(1, kv, T, 128, generator=g, device="cuda").half() for _ in range(2))
        for to in sets:
            cfg = kq.KvqConfig(1, 1, heads * kv, kv, T + 64, page_tokens=page, policy=kq.KVQ_POLICY_OLDEST_FIRST, group=(32, 64, 128)[i % 3])
            arena = torch.full((kq.kvq_arena_bytes(cfg, 8 << 20),), 0xEE, dtype=torch.uint8, device="cuda")
            c = kq.KvqCache(cfg, [1 << 50], [2], arena=arena)
            c.kvq_cache_set_option(kq.KVQ_OPT_TIER16, tier16)
            c.kvq_cache_set_option(kq.KVQ_OPT_DETERMINISTIC, 1)
            c.kvq_cache_set_option(kq.KVQ_OPT_FUSED_MERGE, 0 if i % 7 == 3 else 1)
            if i % 2:
                c.kvq_cache_set_reparam(0, lam)
            if bulk:
                c.kvq_quantize_append(0, k[:, :, :bulk].contiguous(), v[:, :, :bulk].contiguous(), (2, 4, 8)[i % 3])
            c.kvq_quantize_append(0, k[:, :, bulk:].contiguous(), v[:, :, bulk:].contiguous())
            to.append(c)
    return sets


@pytest.mark.parametrize("n,tier16,long,splits", [(1, 0, False, 0), (15, 0, False, 0), (16, 1, True, 0), (16, 0, True, 0), (17, 0, True, 0), (17, 1, False, 0),
                                                  (16, 0, True, 40)])  # 40 ranges a cache: more range ends than fit, 16 caches or not
def test_batch_against_single_calls(n, tier16, long, splits):
    batched, single = _caches(n, tier16, long, n)
    g = torch.Generator("cuda").manual_seed(3)
    for c in batched + single:
        c.kvq_cache_set_option(kq.KVQ_OPT_SPLITS, splits)
    for step in range(4):
        qs, ks, vs, tables = [], [], [], []
        for c in batched:
            kv, heads = c.cfg.n_kv_heads, c.cfg.n_q_heads
            qs.append(torch.randn(1, heads, 128, generator=g, device="cuda").half())
            ks.append(torch.randn(1, kv, 1, 128, generator=g, device="cuda").half())
            vs.append(torch.randn(1, kv, 1, 128, generator=g, device="cuda").half())
            tables.append(torch.randn(1, 128, generator=g, device="cuda"))
        dtype = torch.float32 if step % 2 else torch.float16
        got, want = ([torch.empty(q.shape, dtype=dtype, device="cuda") for q in qs] for _ in range(2))
        if step == 2:
            kq.kvq_decode_attention_batch(batched, 0, qs, got)
            for c, q, o in zip(single, qs, want):
                c.kvq_decode_attention(0, q, o)
        else:
            kq.kvq_append_decode_attention_batch(batched, 0, ks, vs, qs, got, cos_sins=tables)
            for c, k, v, q, o, t in zip(single, ks, vs, qs, want, tables):
                c.kvq_append_decode_attention(0, k, v, q, o, cos_sin=t)
        for i, (a, b) in enumerate(zip(got, want)):
            a, b = a.float().cpu().numpy(), b.float().cpu().numpy()
            assert np.abs(a - b).max() <= MAX_ABS and np.linalg.norm(a - b) <= REL_L2 * np.linalg.norm(b), (step, i)
    for i, (a, b) in enumerate(zip(batched, single)):
        assert a.kvq_cache_describe(0) == b.kvq_cache_describe(0)
        for seg in range(len(a.kvq_cache_describe(0)[0])):
            for which in (0, 1):
                for x, y in zip(a.kvq_cache_export_segment(0, seg, which), b.kvq_cache_export_segment(0, seg, which)):
                    assert (x is None and y is None) or np.array_equal(x.view(np.uint8), y.view(np.uint8)), (i, seg, which)


def test_parameter_blocks_in_the_ring_of_a_larger_batch():
    """17 caches: their parameter blocks, 13 KiB a launch, go round the 4 MiB staging ring more than twice."""
    caches, _ = _caches(17, 0, False, 9)
    g = torch.Generator("cuda").manual_seed(4)
    qs = [torch.randn(1, c.cfg.n_q_heads, 128, generator=g, device="cuda").half() for c in caches]
    outs = [torch.empty(q.shape, dtype=torch.float32, device="cuda") for q in qs]
    kq.kvq_decode_attention_batch(caches, 0, qs, outs)
    torch.cuda.synchronize()
    first = [o.clone() for o in outs]
    for it in range(800):
        kq.kvq_decode_attention_batch(caches, 0, qs, outs)
        if it % 100 == 99:
            torch.cuda.synchronize()
            for o, r in zip(outs, first):
                assert torch.equal(o, r), it  # deterministic mode, same launch shape
                o.fill_(float("nan"))
