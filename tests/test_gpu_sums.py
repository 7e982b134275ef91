"""Reconstruction error and sensitivity: the host takes the workgroups' sums as they arrive.  Calls of different sizes in turn, behind
work that keeps the stream busy, from several threads and over what is no number give what they give by themselves."""
import math
import threading

import pytest
import torch

import paper_2505_18610_amd as kq

pytestmark = pytest.mark.gpu


def _block(units, tokens, bits, seed):
    g = torch.Generator("cuda").manual_seed(seed)
    cfg = kq.KvqConfig(1, 1, units, units, tokens, page_tokens=64, policy=kq.KVQ_POLICY_OLDEST_FIRST)
    arena = torch.empty(kq.kvq_arena_bytes(cfg, tokens * units * 520 + (8 << 20)), dtype=torch.uint8, device="cuda")
    c = kq.KvqCache(cfg, [1 << 50], [2], arena=arena)
    k, v = (torch.randn(1, units, tokens, 128, generator=g, device="cuda").half() for _ in range(2))
    gk, gv = (torch.randn(1, units, tokens, 128, generator=g, device="cuda") for _ in range(2))
    c.kvq_quantize_append(0, k, v, bits)
    return c, k, v, gk, gv


@pytest.mark.parametrize("busy", [False, True])
def test_sums_of_calls_in_turn(busy):
    blocks = [_block(*x) for x in ((1, 5, 2, 1), (16, 700, 4, 2), (64, 2100, 8, 3), (3, 64, 4, 4), (40, 1000, 2, 5))]
    first = [(c.kvq_cache_sensitivity(0, k, v, gk, gv), c.kvq_cache_sq_error(0, k, v)) for c, k, v, gk, gv in blocks]
    for (c, k, v, gk, gv), (l1, _) in zip(blocks, first):  # (a group's rounding at 1e-6 of the sum: fp32 over 32 elements, fp64 beyond)
        assert all(math.isfinite(x) and x > 0 for x in l1)
    a = torch.randn(4096, 4096, device="cuda")
    for _ in range(3):
        for (c, k, v, gk, gv), want in zip(blocks, first):
            if busy:
                for _ in range(6):
                    a = torch.tanh(a @ a)  # some milliseconds in front of the kernel
            assert (c.kvq_cache_sensitivity(0, k, v, gk, gv), c.kvq_cache_sq_error(0, k, v)) == want


def test_sums_of_threads_with_a_cache_each():
    blocks = [_block(*x) for x in ((2, 65, 4, 7), (64, 1500, 2, 8), (16, 300, 8, 9), (8, 4000, 4, 10))]
    want = [(c.kvq_cache_sensitivity(0, k, v, gk, gv), c.kvq_cache_sq_error(0, k, v)) for c, k, v, gk, gv in blocks]
    torch.cuda.synchronize()
    wrong = []

    def work(i):
        c, k, v, gk, gv = blocks[i]
        stream = torch.cuda.Stream()
        for call in range(60):
            got = (c.kvq_cache_sensitivity(0, k, v, gk, gv, stream=stream.cuda_stream), c.kvq_cache_sq_error(0, k, v, stream=stream.cuda_stream))
            if got != want[i]:
                wrong.append((i, call, got, want[i]))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(blocks))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong, wrong[:3]


def test_sums_that_are_no_numbers():
    c, k, v, gk, gv = _block(4, 300, 4, 6)
    want = c.kvq_cache_sensitivity(0, k, v, gk, gv)
    for x in (float("nan"), float("inf")):
        bad = gk.clone()
        bad[0, 1, 17, 3] = x
        got = c.kvq_cache_sensitivity(0, k, v, bad, gv)
        assert not math.isfinite(got[0]) and got[1] == want[1]
        worse = k.clone()
        worse[0, 3, 299, 127] = x
        got = c.kvq_cache_sq_error(0, worse, v)
        assert not math.isfinite(got[0]) and math.isfinite(got[1])
        assert c.kvq_cache_sensitivity(0, k, v, gk, gv) == want
