"""GPU parity of the score on lengths that no factorisation serves (spu_conv: one M-point transform forward and back, zeros
behind the tokens unless N is M itself) against the CPU oracle: both sides of every length limit, the smallest and widest
pass bands (2 sigma = N included), channel counts around a workgroup's share, unaligned rows."""
import numpy as np
import pytest

from paper_2512_09010_amd import binding as lv
from paper_2512_09010_amd import workloads as wl
from gpu_util import to_dev
from test_gpu_spu import SCORE_RTOL, score_case

import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,N,D,sigma,pad", [
    (2, 1999, 70, 300, 0), (1, 2048, 33, 1024, 0), (1, 2047, 9, 1023, 7),      # M = 4096
    (1, 2049, 24, 130, 0), (2, 4095, 6, 2047, 0), (1, 3001, 130, 20, 3),       # M = 8192
    (1, 4097, 5, 60, 0), (1, 8191, 3, 11, 1), (1, 8192, 4, 200, 0),            # M = 16384; N = M = 8192
    (1, 4096, 70, 2048, 0), (2, 4096, 17, 128, 2), (1, 16384, 2, 40, 0),       # N = M
    (1, 1501, 64, 0, 0), (1, 1025, 8, 512, 0),
])
def test_score_any_length(oracle, dtype, B, N, D, sigma, pad):
    rng = np.random.default_rng(N * 7 + D)
    x = wl.cast_io(rng.standard_normal((B, N, D)).astype(np.float32), dtype)
    score_case(oracle, x, dtype, sigma, True, "random", stride_pad=pad)
    walk = wl.cast_io((np.cumsum(rng.standard_normal((B, N, D)), axis=1) / np.sqrt(N)).astype(np.float32), dtype)
    score_case(oracle, walk, dtype, sigma, False, "walk-rect", stride_pad=pad)


def test_many_channel_groups_per_workgroup(oracle):
    """More channel groups than workgroups fit the chip: a workgroup keeps its energies over several of them."""
    rng = np.random.default_rng(5)
    x = wl.cast_io(rng.standard_normal((6, 1026, 1100)).astype(np.float32), "bf16")
    xd, got, _ = score_case(oracle, x, "bf16", 9, True, "groups")
    from paper_2512_09010_amd import binding as lv
    for _ in range(3):
        assert torch.equal(lv.luvc_spu_score(xd, 9, True), got)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,N,D,sigma,pad", [
    (1, 1024, 33, 512, 0), (2, 1023, 15, 511, 1), (1, 513, 17, 3, 0), (3, 1, 3, 0, 0), (1, 9, 5, 4, 0),      # zeros behind the tokens, single elements
    (8, 1000, 514, 100, 0), (8, 1021, 500, 1, 4),                                                            # pairs, several groups of eight
    (1, 2048, 34, 1024, 0), (3, 2048, 30, 200, 0), (1, 2048, 15, 300, 1),                                    # N = M
])
def test_score_on_2048_points(oracle, dtype, B, N, D, sigma, pad):
    rng = np.random.default_rng(N * 11 + D)
    x = wl.cast_io(rng.standard_normal((B, N, D)).astype(np.float32), dtype)
    score_case(oracle, x, dtype, sigma, True, "2048", stride_pad=pad)
    score_case(oracle, x, dtype, sigma, False, "2048-rect", stride_pad=pad)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,N,D,sigma,pad", [
    (1, 767, 17, 380, 0), (1, 768, 9, 384, 1), (1, 769, 15, 0, 0), (13, 700, 514, 70, 0),      # 1536 points
    (1, 1535, 6, 100, 0), (2, 1536, 19, 768, 0), (1, 1537, 10, 3, 0), (2, 1100, 266, 150, 2),  # 3072
    (1, 3071, 6, 1500, 0), (1, 3072, 34, 200, 1), (1, 3073, 4, 60, 0),                         # 6144
    (1, 6143, 4, 2000, 0), (1, 6144, 5, 30, 0), (1, 6145, 3, 700, 0), (2, 4500, 34, 450, 0),   # 12288
])
def test_score_on_three_times_a_power_of_two_points(oracle, dtype, B, N, D, sigma, pad):
    rng = np.random.default_rng(N * 3 + D)
    x = wl.cast_io(rng.standard_normal((B, N, D)).astype(np.float32), dtype)
    score_case(oracle, x, dtype, sigma, True, "3 * 2^n", stride_pad=pad)
    score_case(oracle, x, dtype, sigma, False, "3 * 2^n-rect", stride_pad=pad)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("N,sigma", [(256, 25), (1024, 102), (1500, 150), (2000, 200), (2048, 300), (3000, 300), (4000, 400), (4096, 409), (6000, 150), (8000, 200)])
def test_scores_are_not_short_on_the_mean(oracle, dtype, N, sigma):
    """The fp32 constants of the transforms are all rounded down; what that takes off every score is given back by the weights.
    Left: at most half a unit of the score's own rounding, 2^-25 (5e-8 .. 1e-7 was missing before)."""
    rng = np.random.default_rng(N)
    x = wl.cast_io(rng.standard_normal((1, N, 256)).astype(np.float32), dtype)
    got = lv.luvc_spu_score(to_dev(x, dtype), sigma, True).cpu().numpy().astype(np.float64)
    err = got / oracle.spu_score(wl.widen(x, dtype), sigma, True) - 1.0
    print(f"[spu] N={N} sigma={sigma} {dtype} error mean={err.mean():.2e} rms={np.sqrt((err * err).mean()):.2e}", flush=True)
    assert abs(err.mean()) <= 2.0 ** -25


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("paired", [True, False])           # a channel pair in one access, or channel by channel
@pytest.mark.parametrize("N,sigma,P", [
    (700, 40, 8), (1000, 50, 8), (1500, 20, 4), (2000, 20, 4), (3000, 12, 2), (4000, 12, 2), (6000, 8, 1), (8000, 6, 1),      # zeros behind the tokens: 1536 .. 16384 points
    (2048, 200, 8), (4096, 150, 4), (8192, 9, 2), (16384, 5, 1),                                 # N = M, beyond the bands of spu_fft16q
])
def test_workgroups_that_take_several_steps(oracle, dtype, paired, N, sigma, P):
    """Seven samples of 109 or 110 groups of P pairs: 28 workgroups each, which take four steps, the last one with a part of them.
    The channels are 37 different ones, each with scales of its own per channel: a group left out moves the scores of its sample by
    6e-4 or more (the lowest scale, 1 of 110 groups), one taken in another's place by as much unless all scales agree."""
    rng = np.random.default_rng(N + sigma)
    B, D, K = 7, 220 * P - (2 if paired else 1), 37
    base = wl.cast_io(rng.standard_normal((B, N, K)).astype(np.float32), dtype)
    scale = rng.choice([0.5, 1.0, 2.0], (B, D))              # exact in either type
    x = (to_dev(base, dtype)[:, :, torch.arange(D, device="cuda") % K] * torch.from_numpy(scale).to("cuda", torch.bfloat16 if dtype == "bf16" else torch.float32)[:, None, :]).contiguous()
    print(f"[spu] several steps {tuple(x.shape)} {dtype} sigma={sigma}", flush=True)
    got = lv.luvc_spu_score(x, sigma, True)
    torch.cuda.synchronize()
    _, filtered, _ = oracle.spu_score(wl.widen(base, dtype), sigma, True, want_filtered=True)
    weight = np.stack([np.bincount(np.arange(D) % K, scale[b] ** 2, K) for b in range(B)])
    ref = np.sqrt((filtered * filtered * weight[:, None, :]).sum(axis=2))
    err = np.abs(got.cpu().numpy().astype(np.float64) / ref - 1.0)
    assert err.max() <= SCORE_RTOL, (err.max(), np.unravel_index(err.argmax(), err.shape))
    assert torch.equal(lv.luvc_spu_score(x, sigma, True), got)
