"""Appends into the 16-bit tiers at the sizes where another kernel or another order of the workgroups takes them."""
import pytest
import torch

import paper_2505_18610_amd as kq

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tier16", [0, 1])
@pytest.mark.parametrize("prepared", [False, True])
@pytest.mark.parametrize("units,T", [(8, 1017), (8, 1050), (8, 2041), (8, 2075), (64, 1535), (64, 1552), (16, 4380), (64, 4100)])
def test_one_append_writes_what_its_pieces_write(units, T, prepared, tier16):
    """Seven tokens and then the rest at once, from inside a tile (512 strings and more, 1,024 and more, 98,304 rows and more of 64
    units, the sizes with five wavefronts a SIMD, an odd number of tiles beyond 16,384 strings), or in pieces of 96, which other tests compare with the oracle: the same arena, byte
    for byte."""
    H, P = 8, 64
    B = units // H
    g = torch.Generator(device="cuda").manual_seed(87)
    k, v = (torch.randn((B, H, T, 128), device="cuda", generator=g).half() for _ in range(2))
    table = torch.randn((T, 128), device="cuda", generator=g)
    lam = torch.rand((H, 128), device="cuda", generator=g) + 0.5
    cfg = kq.KvqConfig(1, B, H, H, T + 64, page_tokens=P)
    arenas = []
    for step in (T, 96):
        arena = torch.zeros(kq.kvq_arena_bytes(cfg, (T + 64) * units * 640 + (16 << 20)), dtype=torch.uint8, device="cuda")
        gc = kq.KvqCache(cfg, [1 << 50], [2], arena=arena)
        gc.kvq_cache_set_option(kq.KVQ_OPT_TIER16, tier16)
        if prepared:
            gc.kvq_cache_set_reparam(0, lam)
        t = 0
        while t < T:
            n = min(step, T - t) if t else 7
            piece = [x[:, :, t:t + n].contiguous() for x in (k, v)]
            if prepared:
                gc.kvq_quantize_append_rope(0, *piece, table[t:t + n].contiguous(), 16)
            else:
                gc.kvq_quantize_append(0, *piece, 16)
            t += n
        torch.cuda.synchronize()
        gc.close()
        arenas.append(arena)
    assert torch.equal(*arenas)


@pytest.mark.parametrize("units,T,prepared,tier16", [(256, 3105, False, 0), (256, 3105, False, 1), (32, 3177, True, 0), (128, 2081, False, 0)])
def test_one_append_of_many_strings_writes_what_its_pieces_write(units, T, prepared, tier16):
    """More than 49,152 strings of ready keys (a string a workgroup), 98,304 rows of 32 units, an odd number of tiles in workgroups of two."""
    test_one_append_writes_what_its_pieces_write(units, T, prepared, tier16)
