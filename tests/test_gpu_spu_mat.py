"""GPU parity of spu_mat (two transforms on the matrix cores, N = N1 N2 with N1 in 9 .. 16) against the CPU oracle: every N1,
numbers of subsequences around multiples of 16, bands up to the highest multiple of N1 and beyond it (other kernels), one and several
groups of channels per workgroup, channels that end inside a group, and token values that leave the range of fp16."""
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
    # B, N, D, sigma                              N1 N2  tiles, groups of channels per workgroup, highest multiple
    (40, 364, 1032, 17, "spu_mat"),             # 14 26  2 3 2
    (40, 400, 328, 60, "spu_mat"),              # 16 25  2 1 4
    (32, 784, 1032, 49, "spu_mat"),             # 16 49  4 3 4, one subsequence in the last tile
    (24, 560, 520, 30, "spu_mat"),              # 16 35  3 1 2
    (8, 1152, 1032, 57, "spu_mat"),             # 16 72  5 1 4
    (8, 1170, 1032, 60, "spu_mat"),             # 15 78  5 1 4
    (24, 1300, 1032, 60, "spu_mat"),            # 13 100 7 1 5, two rounds
    (8, 1456, 1032, 20, "spu_mat"),             # 16 91  6 1 2
    (12, 1430, 1544, 90, "spu_mat"),            # 13 110 7 1 7
    (8, 1680, 1032, 45, "spu_mat"),             # 16 105 7 1 3
    (8, 1800, 2056, 105, "spu_mat"),            # 15 120 8 1 7, 33 groups of channels
    (8, 1904, 1032, 100, "spu_mat"),            # 16 119 8 1 7
    (8, 2048, 2056, 112, "spu_mat"),            # 16 128 8 1 7
    (12, 594, 2056, 70, "spu_mat"),             # 11 54  4 2 7
    (16, 616, 2056, 77, "spu_mat"),             # 14 44  3 3 6
    (20, 1012, 1544, 70, "spu_mat"),            # 11 92  6 1 7
    (9, 1000, 1032, 65, "spu_mat"),             # 10 100 7 1 7
    (20, 256, 4872, 40, "spu_mat"),             # 16 16  1 7 3, one whole tile
    (30, 224, 4872, 9, "spu_mat"),              # 16 14  1 10 1
    (8, 1024, 3592, 112, "spu_mat"), (8, 1280, 3592, 110, "spu_mat"), (16, 1040, 1544, 100, "spu_mat"),       # the highest multiple is 7; two groups
    (8, 1270, 1032, 11, "spu_mat"), (8, 1332, 1032, 11, "spu_mat"), (8, 1530, 1032, 30, "spu_mat"), (16, 909, 1032, 30, "spu_mat"),         # N1 = 10, 12, 15 and 9
    # odd numbers of up to 1024 tokens and 19, 29 and 32 tiles, whose energies a sample's last workgroup adds two columns to a thread: the last
    # has one, and the next sample's scores are behind it
    (9, 909, 2312, 30, "spu_mat"), (8, 1023, 3592, 60, "spu_mat"), (8, 975, 4096, 45, "spu_mat"), (8, 455, 4096, 20, "spu_mat"),
    # a multiple more, shorter samples: other kernels
    (8, 1024, 3592, 113, "spu_fft16q"), (8, 2016, 1032, 120, "spu_fold"), (16, 910, 584, 150, "spu_fold"), (10, 1040, 968, 200, "spu_fold"),
    (10, 1280, 968, 150, "spu_fold"), (24, 594, 320, 90, "spu_circ"), (16, 390, 520, 40, "spu_circ"),
    # either side of the line where one is quicker
    (6, 351, 3456, 11, "spu_circ"), (14, 368, 1280, 36, "spu_circ"), (2, 576, 3840, 43, "spu_fft16q"), (11, 240, 4480, 6, "spu_mat"), (9, 1485, 1536, 75, "spu_mat"),
    (8, 1600, 1032, 100, "spu_mat"), (3, 1632, 1280, 49, "spu_mat"),
]


@pytest.mark.parametrize("B,N,D,sigma,name", SHAPES)
def test_score(oracle, B, N, D, sigma, name):
    rng = np.random.default_rng(N * 3 + D)
    x = rng.standard_normal((B, N, D)) * np.exp(rng.standard_normal((B, N, 1)))
    x = wl.cast_io(x.astype(np.float32), "bf16")
    xd, got, _ = score_case(oracle, x, "bf16", sigma, True, "mat")
    assert kernels(lambda: lv.luvc_spu_score(xd, sigma, True)) == [name]
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
    assert torch.equal(got[1:], clean[1:]) and not torch.isfinite(got[0]).any()          # the other samples are not touched
    x[0, 5, 3] = 0.0                                             # a NaN alone, in a range that is looked for without it
    got = lv.luvc_spu_score(to_dev(wl.cast_io(x.astype(np.float32), "bf16"), "bf16"), sigma, True)
    assert torch.equal(got[1:], clean[1:]) and torch.isnan(got[0]).all()


@pytest.mark.parametrize("B,N,D,sigma,name", [(8, 2016, 1032, 100, "spu_mat"), (8, 1024, 1032, 60, "spu_mat"), (4, 2044, 1032, 90, "spu_fold")])
def test_largest_energies(oracle, B, N, D, sigma, name):
    """All of a tile's 64 channels at 2.2e18 in every token: their energy, 3.1e38, is just below what fp32 holds."""
    x = wl.cast_io(np.full((1, N, D), 2.2e18, np.float32), "bf16")
    ref = oracle.spu_score(wl.widen(x, "bf16"), sigma, True)
    xd = to_dev(x, "bf16").expand(B, N, D).contiguous()
    got = lv.luvc_spu_score(xd, sigma, True).cpu().numpy().astype(np.float64)
    assert (np.abs(got / ref - 1.0) <= SCORE_RTOL).all()
    assert kernels(lambda: lv.luvc_spu_score(xd, sigma, True)) == [name]


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


@pytest.mark.parametrize("B,N,D,sigma,N2", [(8, 1024, 1032, 60, 64), (8, 1024, 3592, 102, 64), (32, 784, 1032, 49, 49), (8, 1904, 1032, 100, 119)])
@pytest.mark.parametrize("first,late", GROWTHS)
def test_values_that_grow_beyond_the_first_scale(oracle, B, N, D, sigma, N2, first, late):
    """One and several groups of channels per workgroup."""
    assert growth_case(oracle, B, N, D, sigma, N2, first, late) == ["spu_mat"]


def error_case(oracle, B, N, D, sigma, ham):
    """Rounding, in units of 2^-24: the score's own (at most 1 / sqrt(3), rms) and those behind a filtered value: six at most per stage
    (constants, two halves of the data, the sums), four stages, independent over D channels.  What is common to all channels and tokens,
    or to all tokens, shows in the mean: the weights (half a one, the same for all bins under a rectangular mask were they not
    exact), the twiddles of both ways (half a one each in a complex value, of which at least nine different ones meet: a third in all)."""
    rng = np.random.default_rng(N)
    x = wl.cast_io((rng.standard_normal((1, N, D)) * np.exp(0.5 * rng.standard_normal((1, N, 1)))).astype(np.float32), "bf16")
    ref = oracle.spu_score(wl.widen(x, "bf16"), sigma, ham)
    xd = to_dev(x, "bf16").expand(B, N, D).contiguous()
    err = lv.luvc_spu_score(xd, sigma, ham).cpu().numpy().astype(np.float64) / ref - 1.0
    rms, mean = np.sqrt((err * err).mean()), err.mean()
    print(f"[spu] {N}x{D} sigma={sigma} ham={ham} error rms={rms:.2e} mean={mean:.2e}", flush=True)
    assert rms <= 2.0 ** -24 * np.sqrt(1.0 / 3.0 + 24.0 ** 2 / D + 0.8 ** 2)
    assert abs(mean) <= 2.0 ** -24 * (0.5 + 1.0 / 3.0)
    return kernels(lambda: lv.luvc_spu_score(xd, sigma, ham))


@pytest.mark.parametrize("B,N,D,sigma", [(8, 1024, 3584, 102), (16, 720, 4096, 54), (8, 2048, 2056, 102), (8, 576, 1024, 57), (4, 1575, 1152, 39), (3, 1188, 3712, 45),
                                         (19, 256, 4864, 40), (12, 594, 2056, 70), (9, 1000, 1032, 65)])
@pytest.mark.parametrize("ham", [True, False])
def test_error_against_fp64(oracle, B, N, D, sigma, ham):
    assert error_case(oracle, B, N, D, sigma, ham) == ["spu_mat"]


@pytest.mark.parametrize("lengths,D,names,share", [
    ([520, 576, 576, 448, 312, 570, 392], 2056, ["spu_mat"], 10),                # one launch; the last group of channels holds one piece
    ([520, 576, 576, 448, 312, 570, 392], 2056, ["spu_mat"], 30),                # a row per multiple
    ([400 + 16 * i for i in range(18)] + [390, 390], 1032, ["spu_mat", "spu_mat"], 10),    # more runs than a launch takes
    ([523, 576, 520, 448, 560, 570, 523, 40], 4104, ["spu_mat", "spu_circ"], 10),          # prime and short ones among them
])
def test_ragged_samples_in_one_launch(oracle, lengths, D, names, share):
    rng = np.random.default_rng(D)
    x = wl.cast_io((rng.standard_normal((sum(lengths), D)) * np.exp(rng.standard_normal((sum(lengths), 1)))).astype(np.float32), "bf16")
    sigmas = [n // share for n in lengths]
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
