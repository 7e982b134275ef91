"""Reconstruction error, sensitivity and factor calibration at the sizes where their kernels change course: one token, tile and
page remainders, more strings than a launch has wavefronts, every tier, references that are not 16-byte aligned."""
import numpy as np
import pytest
import torch

import kvq_synth
import paper_2505_18610_amd as kq
from oracle import calibrate_lambda
from gpu_util import make_pair, append_both

pytestmark = pytest.mark.gpu


def odd_view(x):
    """The array on the device, starting one element behind a 16-byte boundary."""
    flat = torch.empty(x.size + 8, dtype=torch.from_numpy(x).dtype, device="cuda")
    flat.fill_(float("nan"))
    flat[1:1 + x.size] = torch.from_numpy(x.reshape(-1)).cuda()
    return flat[1:1 + x.size].view(x.shape)


@pytest.mark.parametrize("B,Hkv,P,tiers,tier16", [
    (1, 1, 32, ((1, 16),), 0),
    (1, 2, 64, ((64, 2), (64, 4), (64, 8), (33, 16)), 0),
    (2, 3, 32, ((32, 8), (96, 2), (31, 16)), 1),
    (1, 1, 96, ((192, 4), (5, 8)), 0),
    (3, 5, 64, ((4992, 2), (64, 16)), 0),        # 2 x 158 x 15 strings: more than 1,024 workgroups of four
])
def test_errors_against_the_oracle(B, Hkv, P, tiers, tier16):
    T = sum(n for n, _ in tiers)
    K, V = kvq_synth.make_kv(61, 0, B, Hkv, 0, T)
    oc, gc = make_pair(1, B, 2 * Hkv, Hkv, T, P, tier16=tier16)
    t = 0
    for n, bits in tiers:
        append_both(oc, gc, 0, K[:, :, t:t + n], V[:, :, t:t + n], bits)
        t += n
    rng = np.random.default_rng(5)
    Kr = (K.astype(np.float32) + rng.standard_normal(K.shape, dtype=np.float32)).astype(np.float16)
    Vr = (V.astype(np.float32) + rng.standard_normal(V.shape, dtype=np.float32)).astype(np.float16)
    gk, gv = (rng.standard_normal(K.shape, dtype=np.float32) for _ in range(2))
    want = oc.reconstruction_sq_error(0, Kr, Vr)
    Kh, Vh = oc.dequantized(0)
    dk, dv = np.abs(Kh - Kr.astype(np.float64)), np.abs(Vh - Vr.astype(np.float64))
    want_one = (dk.sum(), dv.sum())
    want_g = ((np.abs(gk).astype(np.float64) * dk).sum(), (np.abs(gv).astype(np.float64) * dv).sum())
    for dev in (lambda x: torch.from_numpy(x).cuda(), odd_view):
        got = gc.kvq_cache_sq_error(0, dev(Kr), dev(Vr))
        # a lane adds 8 fp32 terms per accumulator, each rounded twice: 10 x 2^-24, fp64 from there on
        assert np.allclose(got, want, rtol=1e-6, atol=0), (got, want)
        one = gc.kvq_cache_sensitivity(0, dev(Kr), dev(Vr))
        got = gc.kvq_cache_sensitivity(0, dev(Kr), dev(Vr), dev(gk), dev(gv))
        for a, b in ((one, want_one), (got, want_g)):
            assert np.allclose(a, b, rtol=1e-6, atol=0), (a, b)
    gc.close()


@pytest.mark.parametrize("bits,tier16", [(16, 0), (16, 1), (8, 0), (2, 0)])
@pytest.mark.parametrize("T", [1, 7, 32, 45, 129])
def test_sensitivity_with_gradients_of_one_tensor(T, bits, tier16):
    """Gradients of K alone and of V alone weigh that tensor, ones the other: the sums that two calls give."""
    B, H = 2, 3
    g = torch.Generator("cuda").manual_seed(64)
    K, V, Kr, Vr = (torch.randn((B, H, T, 128), generator=g, device="cuda").half() for _ in range(4))
    gk, gv = (torch.randn((B, H, T, 128), generator=g, device="cuda") for _ in range(2))
    _, gc = make_pair(1, B, H, H, T, 96, tier16=tier16)
    gc.kvq_quantize_append(0, K, V, bits)
    both, none = gc.kvq_cache_sensitivity(0, Kr, Vr, gk, gv), gc.kvq_cache_sensitivity(0, Kr, Vr)
    assert tuple(gc.kvq_cache_sensitivity(0, Kr, Vr, gk, None)) == (both[0], none[1])
    assert tuple(gc.kvq_cache_sensitivity(0, Kr, Vr, None, gv)) == (none[0], both[1])
    if bits == 16 and not tier16:  # raw values: the terms themselves
        d = [(a.double() - b.double()).abs() for a, b in ((K, Kr), (V, Vr))]
        # 8 fp32 terms per accumulator and their sum, each rounded at most twice: 10 x 2^-24
        assert np.allclose(none, [float(x.sum()) for x in d], rtol=1e-6, atol=0)
        assert np.allclose(both, [float((x * y.double().abs()).sum()) for x, y in zip(d, (gk, gv))], rtol=1e-6, atol=0)
    gc.close()


@pytest.mark.parametrize("B,Hkv,T", [(1, 1, 1), (1, 2, 15), (2, 1, 129), (3, 4, 257), (1, 8, 4097), (40, 32, 17),
                                     (300, 3, 1), (1000, 2, 3), (77, 1, 16), (33, 2, 31), (2, 1100, 3)])
def test_calibration_at_slice_edges(B, Hkv, T):
    K, _ = kvq_synth.make_kv(62, 0, B, Hkv, 0, T)
    K[0, Hkv - 1, T - 1, 127] = -3000.0  # the last element read decides its channel
    want = calibrate_lambda(K, 0.5)
    for dev in (lambda x: torch.from_numpy(x).cuda(), odd_view):
        lam = torch.full((Hkv, 128), -1.0, dtype=torch.float32, device="cuda")
        kq.kvq_calibrate_lambda(dev(K), 0.5, lam)
        # maxima are exact; pow in fp64 rounded to fp32: one ulp
        assert np.allclose(lam.cpu().numpy(), want, rtol=1.2e-7, atol=0)


@pytest.mark.parametrize("B,H,T", [(1 << 21, 8, 1), (3, 1030, 1400)])
def test_calibration_over_many_sequences_or_heads(B, H, T):
    """2^24 (sequence, head) pairs of one token: 2^32 threads if each had a workgroup of its own.  More heads than a launch wants
    workgroups: several slices of a head all the same."""
    K = torch.empty((B, H, T, 128), dtype=torch.float16, device="cuda").normal_()
    K[B - 1, H - 1, T - 1, 127] = -3000.0
    lam = torch.full((H, 128), -1.0, dtype=torch.float32, device="cuda")
    kq.kvq_calibrate_lambda(K, 1.0, lam)
    assert torch.equal(lam, K.abs_().amax(dim=(0, 2)).float())


@pytest.mark.parametrize("alpha", [0.0, 1e-30, 1e-14, 0.3, 1.0, 4.0])
@pytest.mark.parametrize("B,H,T", [(5, 3, 700), (40, 3, 20)])
def test_the_power_of_the_maximum_is_the_maximum_of_the_powers(B, H, T, alpha):
    """Every workgroup raises its own maxima: the same bits as from one row that holds the maxima, below the floor and at infinity too."""
    K = torch.randn((B, H, T, 128), generator=torch.Generator("cuda").manual_seed(63), device="cuda", dtype=torch.float16)
    K[..., 0], K[..., 1] = 0.0, 6e-8
    K[2, 1, 11, 5] = float("inf")
    lam, want = (torch.full((H, 128), -1.0, device="cuda") for _ in range(2))
    kq.kvq_calibrate_lambda(K, alpha, lam)
    kq.kvq_calibrate_lambda(K.abs().amax(dim=(0, 2)).reshape(1, H, 1, 128), alpha, want)
    assert torch.equal(lam, want)
    # floor and alpha as fp32 holds them; pow in fp64 rounded to fp32: one ulp
    floor, power = (float(np.float32(x)) for x in (1e-5, alpha))
    assert torch.allclose(lam.double(), K.abs().amax(dim=(0, 2)).double().clamp(min=floor) ** power, rtol=1.2e-7, atol=0)


@pytest.mark.parametrize("bits", [0x7e00, 0xfe00, 0x7c01, 0xffff])
@pytest.mark.parametrize("B,H,T", [(5, 3, 700), (40, 3, 20)])
def test_calibration_passes_over_what_is_no_number(B, H, T, bits):
    """NaN of either kind and sign, in the row group, slice and sequence that hold a channel's maximum and elsewhere: the maximum of the rest."""
    K = torch.randn((B, H, T, 128), generator=torch.Generator("cuda").manual_seed(65), device="cuda", dtype=torch.float16)
    K[3, 1, 7, 20] = 50.0
    rest = K.clone()
    at = ((3, 1, 7 + 8, 20), (3, 1, 6, 20), (0, 1, 0, 20), (B - 1, 2, T - 1, 127), (2, 0, 5, 0))
    for i in at:
        K.view(torch.int16)[i] = bits - 0x10000 if bits >= 0x8000 else bits
        rest[i] = 0.0
    K.view(torch.int16)[:, 2, :, 64] = 0x7e00  # a channel without a number: the floor
    rest[:, 2, :, 64] = 0.0
    lam, want = (torch.full((H, 128), -1.0, device="cuda") for _ in range(2))
    kq.kvq_calibrate_lambda(K, 0.5, lam)
    kq.kvq_calibrate_lambda(rest, 0.5, want)
    assert torch.equal(lam, want)


def test_calibration_time_does_not_depend_on_how_the_tokens_are_cut_into_sequences():
    """131,072 tokens of 8 heads as 64 sequences and as 131,072."""
    K = torch.randn((131072, 8, 1, 128), dtype=torch.float16, device="cuda")
    lam = torch.empty((8, 128), dtype=torch.float32, device="cuda")

    def best(x):
        times = []
        for _ in range(6):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            kq.kvq_calibrate_lambda(x, 0.5, lam)
            end.record()
            torch.cuda.synchronize()
            times.append(start.elapsed_time(end))
        return min(times)

    # a workgroup and its atomics per sequence: 90 times as long
    assert best(K) < 4 * best(K.view(64, 8, 2048, 128))
