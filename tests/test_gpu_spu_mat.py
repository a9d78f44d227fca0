"""GPU parity of spu_mat (two transforms on the matrix cores, N = N1 N2 with N1 in 9 .. 16) against the CPU oracle: every N1,
numbers of subsequences around multiples of 16, one to four blocks of band rows, several groups of channels per workgroup,
channels that end inside a group, and token values that leave the range of fp16."""
import numpy as np
import pytest
import torch

from paper_2512_09010_amd import binding as lv
from paper_2512_09010_amd import workloads as wl
from gpu_util import to_dev
from test_gpu_spu import SCORE_RTOL, score_case

pytestmark = pytest.mark.gpu


def kernels(call):
    prof = lv.LaunchProfile(8)
    prof.start()
    call()
    prof.stop()
    torch.cuda.synchronize()
    names = [n for n, _ in prof.results()]
    prof.close()
    return names


SHAPES = [
    # B, N, D, sigma                      N1 N2  tiles  blocks of band rows
    (40, 364, 1032, 17),                # 14 26  2      1, three groups of channels per workgroup
    (16, 390, 520, 40),                 # 15 26  2      1
    (40, 400, 328, 60),                 # 16 25  2      1
    (24, 594, 320, 90),                 # 11 54  4      3
    (24, 560, 520, 30),                 # 14 40  3      1
    (8, 1152, 1032, 57),                # 16 72  5      1
    (16, 910, 584, 150),                # 14 65  5      3
    (8, 1170, 1032, 60),                # 13 90  6      2
    (10, 1040, 968, 200),               # 16 65  5      4
    (10, 1280, 968, 150),               # 16 80  5      3
    (8, 1456, 1032, 20),                # 16 91  6      1
    (8, 1680, 1032, 45),                # 15 112 7      1
    (8, 1904, 1032, 100),               # 16 119 8      2
    (8, 2048, 1032, 102),               # 16 128 8      2
    (8, 2016, 1032, 120),               # 16 126 8      2
    (8, 1024, 3592, 112), (8, 1024, 3592, 113), (8, 1280, 3592, 110), (16, 1040, 1544, 100),    # folded rows up to their last multiple, one beyond, two groups
    (8, 1270, 1032, 11), (8, 1332, 1032, 11), (8, 1530, 1032, 30), (16, 909, 1032, 30),         # N1 = 10, 12, 15 and 9
]


@pytest.mark.parametrize("B,N,D,sigma", SHAPES)
def test_score(oracle, B, N, D, sigma):
    rng = np.random.default_rng(N * 3 + D)
    x = rng.standard_normal((B, N, D)) * np.exp(rng.standard_normal((B, N, 1)))
    x = wl.cast_io(x.astype(np.float32), "bf16")
    xd, got, _ = score_case(oracle, x, "bf16", sigma, True, "mat")
    assert kernels(lambda: lv.luvc_spu_score(xd, sigma, True)) in (["spu_mat"], ["spu_fold"])
    for _ in range(2):                                           # same bits whichever workgroup adds up
        assert torch.equal(lv.luvc_spu_score(xd, sigma, True), got)
    if N < 1000:
        score_case(oracle, x, "bf16", sigma, False, "mat-rect", stride_pad=24)


def test_values_out_of_the_range_of_fp16(oracle):
    """A scale per wavefront brings the values into range: it is set by the first ones that are not zero and changed when larger
    ones follow (subsequences 0 .. 15 of the 64 come first), and again for the way back."""
    B, N, D, sigma = 8, 1024, 1032, 60
    rng = np.random.default_rng(7)
    base = rng.standard_normal((B, N, D))
    sub = np.arange(N) % 64                                      # token n belongs to subsequence n mod N2
    late = (sub >= 16)[None, :, None]
    for tag, x in [("tiny", base * 1e-17), ("large", base * 1e15), ("zeros first", base * late), ("growing", base * np.where(late, 1e9, 1.0)),
                   ("falling", base * np.where(late, 1e-3, 1.0)), ("steps", base * 10.0 ** (3 * (sub // 16))[None, :, None]),
                   ("channels", base * 10.0 ** rng.uniform(-6, 6, (1, 1, D))), ("zero", base * 0.0)]:
        xd, _, _ = score_case(oracle, wl.cast_io(x.astype(np.float32), "bf16"), "bf16", sigma, True, tag)
    assert kernels(lambda: lv.luvc_spu_score(xd, sigma, True)) == ["spu_mat"]
    x = base.copy()
    x[0, 5, 3] = np.inf
    x[0, 40, 70] = np.nan
    got = lv.luvc_spu_score(to_dev(wl.cast_io(x.astype(np.float32), "bf16"), "bf16"), sigma, True)
    clean = lv.luvc_spu_score(to_dev(wl.cast_io(base.astype(np.float32), "bf16"), "bf16"), sigma, True)
    assert torch.equal(got[1:], clean[1:])                       # the other samples are not touched


# the first subsequences hold `first`, those behind them `late`: the scale that `first` sets takes `late` beyond fp32 by itself
GROWTHS = [(3e-34, 3e3), (1e-35, 1e4), (1e-38, 1e15), (1e-30, 1e10)]


def growth_case(oracle, B, N, D, sigma, N2, first, late):
    x = np.random.default_rng(N).standard_normal((1, N, D)) * np.where(np.arange(N) % N2 >= 16, late, first)[None, :, None]
    x = wl.cast_io(x.astype(np.float32), "bf16")
    print(f"[spu] growth {first} -> {late} {B}x{N}x{D} sigma={sigma}", flush=True)
    ref = oracle.spu_score(wl.widen(x, "bf16"), sigma, True)
    xd = to_dev(x, "bf16").expand(B, N, D).contiguous()
    got = lv.luvc_spu_score(xd, sigma, True).cpu().numpy().astype(np.float64)
    assert (np.abs(got - ref) <= SCORE_RTOL * ref + 1e-6 * ref.max()).all(), float(np.abs(got / ref - 1).max())
    return kernels(lambda: lv.luvc_spu_score(xd, sigma, True))


@pytest.mark.parametrize("B,N,D,sigma,N2", [(8, 1024, 1032, 60, 64), (8, 1024, 3592, 102, 64), (8, 1024, 3592, 113, 64), (4, 552, 5120, 96, 46), (16, 640, 3584, 250, 40)])
@pytest.mark.parametrize("first,late", GROWTHS)
def test_values_that_grow_beyond_the_first_scale(oracle, B, N, D, sigma, N2, first, late):
    """One block of rows, folded rows, two, three and four blocks, one and several groups of channels per workgroup."""
    growth_case(oracle, B, N, D, sigma, N2, first, late)


@pytest.mark.parametrize("B,N,D,sigma", [(8, 1024, 1024, 102), (8, 720, 1024, 54), (4, 2048, 512, 102), (8, 576, 1024, 57), (4, 1248, 512, 62)])
def test_error_against_fp64(oracle, B, N, D, sigma):
    """Rounding: the score's own (at most 2^-24 / sqrt(3), rms) and those behind a filtered value: six of 2^-24 at most per stage
    (constants, two halves of the data, the sums), four stages, independent over D channels; what is common to all channels is
    given back by the weights but for a fifth of 2^-24 per stage."""
    rng = np.random.default_rng(N)
    x = wl.cast_io((rng.standard_normal((B, N, D)) * np.exp(0.5 * rng.standard_normal((B, N, 1)))).astype(np.float32), "bf16")
    got = lv.luvc_spu_score(to_dev(x, "bf16"), sigma, True).cpu().numpy().astype(np.float64)
    err = got / oracle.spu_score(wl.widen(x, "bf16"), sigma, True) - 1.0
    rms, mean = np.sqrt((err * err).mean()), err.mean()
    print(f"[spu] {N}x{D} error rms={rms:.2e} mean={mean:.2e}", flush=True)
    assert rms <= 2.0 ** -24 * np.sqrt(1.0 / 3.0 + 24.0 ** 2 / D + 0.8 ** 2)


@pytest.mark.parametrize("lengths,D,names", [
    ([520, 576, 576, 448, 312, 570, 392], 2056, ["spu_mat"]),                    # one launch; the last group of channels holds one piece
    ([400 + 16 * i for i in range(18)] + [390, 390], 1032, ["spu_mat", "spu_mat"]),        # more runs than a launch takes
    ([523, 576, 520, 448, 560, 570, 523, 40], 4104, ["spu_mat", "spu_circ"]),    # prime and short ones among them
])
def test_ragged_samples_in_one_launch(oracle, lengths, D, names):
    rng = np.random.default_rng(D)
    x = wl.cast_io((rng.standard_normal((sum(lengths), D)) * np.exp(rng.standard_normal((sum(lengths), 1)))).astype(np.float32), "bf16")
    sigmas = [n // 10 for n in lengths]
    print(f"[spu] ragged {lengths} D={D}", flush=True)
    xd, out = to_dev(x, "bf16"), {}
    got = kernels(lambda: out.update(lv.luvc_spu_stage_ragged(xd, lengths, sigmas, [max(1, n // 5) for n in lengths])))
    assert sorted(got) == sorted(names + ["spu_prune_fused"])
    scores, at = out["scores"].cpu().numpy().astype(np.float64), 0
    for n, s in zip(lengths, sigmas):
        ref = oracle.spu_score(wl.widen(x[None, at:at + n], "bf16"), s, True)[0]
        err = np.abs(scores[at:at + n] - ref)
        assert (err <= SCORE_RTOL * ref + 1e-6 * ref.max()).all(), (n, float((err / ref).max()))
        at += n
