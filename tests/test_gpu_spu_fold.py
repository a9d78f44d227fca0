"""GPU parity of spu_fold (multiples j and -j of N1 folded, up to 4096 tokens) against the CPU oracle: every N1, one and two blocks
of band rows, bands that end on either side of a multiple, tiles that are nearly empty, channels that end inside a group, numbers of
tiles around the four that are added at a time, and token values that leave the range of fp16."""
import numpy as np
import pytest
import torch

from paper_2512_09010_amd import binding as lv
from paper_2512_09010_amd import workloads as wl
from gpu_util import to_dev
from test_gpu_spu import score_case
from test_gpu_spu_mat import GROWTHS, error_case, growth_case, kernels

pytestmark = pytest.mark.gpu

SHAPES = [
    # B, N, D, sigma                      N1 N2  tiles  blocks of band rows
    (8, 4096, 1544, 112),               # 16 256 16     1, the last multiple is 7
    (8, 4096, 1544, 113),               # 16 256 16     2
    (7, 4096, 2056, 240),               # 16 256 16     2, the last multiple is 15
    (8, 3600, 1032, 100),               # 16 225 15     1, one subsequence in the last tile
    (8, 3840, 1032, 119),               # 16 240 15     1
    (8, 3570, 1032, 30),                # 15 238 15     1
    (8, 3472, 1032, 99),                # 16 217 14     1
    (6, 3066, 1032, 200),               # 14 219 14     2
    (6, 2834, 1032, 195),               # 13 218 14     2
    (6, 2508, 1032, 80),                # 12 209 14     1
    (6, 2167, 1032, 77),                # 11 197 13     1, a prime number of subsequences
    (6, 2230, 1032, 150),               # 10 223 14     2
    (6, 2061, 1032, 135),               #  9 229 15     2
    (4, 2064, 1032, 112), (4, 2080, 1032, 1), (4, 2304, 1032, 230),      # 16 129, 16 130, 16 144
    (10, 975, 2184, 140), (8, 1001, 3592, 150),         # odd numbers of up to 1024 tokens, 18 and 29 tiles: two columns to a thread in the last sum
    (30, 420, 2056, 28), (20, 648, 3080, 60), (6, 2736, 2312, 100),      # 15 28, 12 54 and 16 171 with more than 32 groups of channels
]


@pytest.mark.parametrize("B,N,D,sigma", SHAPES)
def test_score(oracle, B, N, D, sigma):
    rng = np.random.default_rng(N * 5 + D + sigma)
    x = wl.cast_io((rng.standard_normal((B, N, D)) * np.exp(rng.standard_normal((B, N, 1)))).astype(np.float32), "bf16")
    xd, got, _ = score_case(oracle, x, "bf16", sigma, True, "fold")
    assert kernels(lambda: lv.luvc_spu_score(xd, sigma, True)) == ["spu_fold"]
    for _ in range(2):                                           # same bits whichever workgroup adds up
        assert torch.equal(lv.luvc_spu_score(xd, sigma, True), got)
    if N % 2:
        score_case(oracle, x, "bf16", sigma, False, "fold-rect", stride_pad=24)


def test_values_out_of_the_range_of_fp16(oracle):
    """As for spu_mat; subsequences 0 .. 15 of the 144 come first."""
    B, N, D, sigma = 4, 2304, 1032, 150
    rng = np.random.default_rng(9)
    base = rng.standard_normal((B, N, D))
    sub = np.arange(N) % 144
    late = (sub >= 16)[None, :, None]
    for tag, x in [("tiny", base * 1e-17), ("large", base * 1e15), ("zeros first", base * late), ("growing", base * np.where(late, 1e9, 1.0)),
                   ("falling", base * np.where(late, 1e-3, 1.0)), ("steps", base * 10.0 ** (sub // 16)[None, :, None]),
                   ("channels", base * 10.0 ** rng.uniform(-6, 6, (1, 1, D))), ("zero", base * 0.0),
                   ("tone", np.cos(2 * np.pi * 37 * np.arange(N) / N)[None, :, None] * np.ones((B, 1, D)))]:
        xd, _, _ = score_case(oracle, wl.cast_io(x.astype(np.float32), "bf16"), "bf16", sigma, True, tag)
    assert kernels(lambda: lv.luvc_spu_score(xd, sigma, True)) == ["spu_fold"]
    x = base.copy()
    x[0, 5, 3] = np.inf
    x[0, 40, 70] = np.nan
    got = lv.luvc_spu_score(to_dev(wl.cast_io(x.astype(np.float32), "bf16"), "bf16"), sigma, True)
    clean = lv.luvc_spu_score(to_dev(wl.cast_io(base.astype(np.float32), "bf16"), "bf16"), sigma, True)
    assert torch.equal(got[1:], clean[1:]) and not torch.isfinite(got[0]).any()


@pytest.mark.parametrize("N,sigma,N2", [(2064, 112, 129), (2304, 150, 144)])
@pytest.mark.parametrize("first,late", GROWTHS)
def test_values_that_grow_beyond_the_first_scale(oracle, N, sigma, N2, first, late):
    """As for spu_mat; one and two blocks of band rows."""
    assert growth_case(oracle, 4, N, 1032, sigma, N2, first, late) == ["spu_fold"]


@pytest.mark.parametrize("B,N,D,sigma", [(6, 2508, 1032, 80), (8, 4096, 1544, 112), (8, 4096, 1544, 200), (6, 3000, 1032, 150), (6, 2880, 1032, 140)])
@pytest.mark.parametrize("ham", [True, False])
def test_error_against_fp64(oracle, B, N, D, sigma, ham):
    """The bounds of spu_mat: the method's roundings are the same."""
    assert error_case(oracle, B, N, D, sigma, ham) == ["spu_fold"]
