"""GPU parity: ragged batches (luvc_oim_merge_ragged, luvc_oim_plan_anyres, luvc_spu_stage_ragged through the C ABI)
against the CPU oracle, item by item: every image / sample of a packed batch must come out exactly as the oracle
computes it on its own."""
import numpy as np
import pytest
import torch

from paper_2512_09010_amd import binding as lv
from paper_2512_09010_amd import workloads as wl
from gpu_util import OIM_MARGIN, RTOL, SPU_MARGIN, assert_close, round_mode, to_dev, to_host_f64

pytestmark = pytest.mark.gpu


def oim_ragged_case(oracle, shapes, D, dtype, max_tokens, seed, with_sizes, schedules=None):
    rng = np.random.default_rng(seed)
    if schedules is None:
        schedules = [lv.luvc_oim_plan_anyres(h, w, max_tokens) for h, w in shapes]
        for (h, w), sch in zip(shapes, schedules):
            assert sch == oracle.plan_anyres(h, w, max_tokens), (h, w)
    imgs = [wl.cast_io(wl.smooth_field(rng, 1, h, w, D, 2.0) + 0.1 * rng.standard_normal((1, h, w, D)).astype(np.float32), dtype)
            for h, w in shapes]
    sizes = [rng.integers(1, 5, (1, h, w)) for h, w in shapes] if with_sizes else None
    print(f"[ragged oim] shapes={shapes} D={D} dtype={dtype} cap={max_tokens} sizes={with_sizes}", flush=True)
    packed = np.concatenate([a.reshape(-1, D) for a in imgs])
    s_dev = None
    if with_sizes:
        s_dev = torch.from_numpy(np.concatenate([s.reshape(-1) for s in sizes]).astype(np.int32)).cuda()
    out = lv.luvc_oim_merge_ragged(to_dev(packed, dtype), shapes, schedules, sizes=s_dev)
    torch.cuda.synchronize()
    gx, gs = to_host_f64(out["x"]), out["sizes"].cpu().numpy().astype(np.int64)
    gm, gk = out["merged_map"].cpu().numpy(), out["kept_map"].cpu().numpy()
    ti = to = 0
    for i, ((h, w), sch) in enumerate(zip(shapes, schedules)):
        ref = oracle.oim_merge(wl.widen(imgs[i], dtype), sch, sizes=None if sizes is None else sizes[i], round_mode=round_mode(oracle, dtype))
        ho, wo = out["out_shapes"][i]
        assert ref["x"].shape == (1, ho, wo, D)
        assert ref["margin"] > OIM_MARGIN or ref["margin"] == 0.0, (i, ref["margin"])
        n_in, n_out = h * w, ho * wo
        np.testing.assert_array_equal(gs[to:to + n_out], ref["sizes"].reshape(-1))
        np.testing.assert_array_equal(gm[ti:ti + n_in], ref["merged_map"].reshape(-1))
        np.testing.assert_array_equal(gk[to:to + n_out], ref["kept_map"].reshape(-1))
        assert_close(gx[to:to + n_out], ref["x"].reshape(n_out, D), RTOL[dtype], f"image {i}")
        if dtype == "bf16":
            np.testing.assert_array_equal(gx[to:to + n_out], ref["x"].reshape(n_out, D))
        ti += n_in
        to += n_out
    assert ti == packed.shape[0] and to == gx.shape[0]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_oim_anyres_batch(oracle, dtype):
    # wide, tall and square images; equal neighbours form runs of 2 and 3; one image is within the budget already
    shapes = [(16, 48), (16, 48), (40, 12), (24, 24), (24, 24), (24, 24), (8, 8), (9, 31), (1, 70)]
    oim_ragged_case(oracle, shapes, 64, dtype, 144, 1, with_sizes=False)
    oim_ragged_case(oracle, shapes, 72, dtype, 64, 2, with_sizes=True)


def test_oim_ragged_explicit_schedules(oracle):
    """Schedules that differ on equal shapes split a run; the paper's merge number 2 on both axes."""
    rng = np.random.default_rng(3)
    shapes = [(10, 12), (10, 12), (10, 12), (6, 6)]
    schedules = [[(1, 2), (0, 2)], [(1, 2), (0, 2)], [(0, 2), (1, 2), (0, 2)], [(1, 3)]]
    D, dtype = 40, "bf16"
    imgs = [wl.cast_io(rng.standard_normal((1, h, w, D)).astype(np.float32), dtype) for h, w in shapes]
    packed = np.concatenate([a.reshape(-1, D) for a in imgs])
    out = lv.luvc_oim_merge_ragged(to_dev(packed, dtype), shapes, schedules)
    torch.cuda.synchronize()
    gx = to_host_f64(out["x"])
    to = 0
    for i, sch in enumerate(schedules):
        ref = oracle.oim_merge(wl.widen(imgs[i], dtype), sch, round_mode=round_mode(oracle, dtype))
        n_out = ref["x"].shape[1] * ref["x"].shape[2]
        assert ref["margin"] > OIM_MARGIN
        np.testing.assert_array_equal(gx[to:to + n_out], ref["x"].reshape(n_out, D))
        to += n_out
    assert to == gx.shape[0]


def spu_ragged_case(oracle, lengths, D, dtype, ratio, seed, origin_shift=None, sigmas=None, keeps=None):
    rng = np.random.default_rng(seed)
    if sigmas is None:
        sigmas = [max(1, int(ratio * n / 2)) if n > 1 else 0 for n in lengths]
    if keeps is None:
        keeps = [lv.luvc_keep_count(n, ratio) for n in lengths]
    xs = [wl.cast_io((rng.standard_normal((1, n, D)) + np.sin(np.arange(n) / 5.0)[None, :, None] * rng.standard_normal((1, 1, D))).astype(np.float32), dtype)
          for n in lengths]
    print(f"[ragged spu] lengths={lengths} D={D} dtype={dtype} keeps={keeps}", flush=True)
    packed = np.concatenate([a.reshape(-1, D) for a in xs])
    org = None
    if origin_shift is not None:
        org = torch.from_numpy(np.concatenate([np.arange(n, dtype=np.int32) * 2 + origin_shift for n in lengths])).cuda()
    out = lv.luvc_spu_stage_ragged(to_dev(packed, dtype), lengths, sigmas, keeps, origin=org)
    torch.cuda.synchronize()
    gsc = out["scores"].cpu().numpy().astype(np.float64)
    gk, go, gx = out["kept_idx"].cpu().numpy(), out["origin"].cpu().numpy(), to_host_f64(out["x"])
    ti = to = 0
    for i, n in enumerate(lengths):
        o_in = None if origin_shift is None else (np.arange(n, dtype=np.int32) * 2 + origin_shift)[None, :]
        ref = oracle.spu_stage(wl.widen(xs[i], dtype), sigmas[i], keeps[i], True, o_in)
        floor = 1e-6 * np.abs(ref["scores"]).max()
        assert (np.abs(gsc[ti:ti + n] - ref["scores"][0]) <= 1e-5 * np.abs(ref["scores"][0]) + floor).all(), i
        assert ref["margin"] > SPU_MARGIN, (i, ref["margin"])
        k = keeps[i]
        np.testing.assert_array_equal(gk[to:to + k], ref["kept_idx"][0])
        np.testing.assert_array_equal(go[to:to + k], ref["origin"][0])
        np.testing.assert_array_equal(gx[to:to + k], ref["x"][0])
        ti += n
        to += k
    assert ti == packed.shape[0] and to == gk.shape[0]
    # scores only
    sc_only = lv.luvc_spu_stage_ragged(to_dev(packed, dtype), lengths, sigmas, None)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(sc_only["scores"].cpu().numpy(), out["scores"].cpu().numpy())


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_spu_ragged_batch(oracle, dtype):
    # lengths with convenient factors (1024, 720, 256) and without, long and short; runs of 2
    lengths = [1024, 1024, 720, 196, 196, 300, 64, 97, 256, 1]
    spu_ragged_case(oracle, lengths, 96, dtype, 0.25, 4)
    spu_ragged_case(oracle, lengths[2:], 70, dtype, 0.1, 5, origin_shift=7)


# seeds: the first from 31 on whose keep sets are all decided by more than the margin of the scores
@pytest.mark.parametrize("n, count, D, dtype, seed", [(729, 12, 3584, "bf16", 31), (500, 12, 3584, "f32", 35), (24, 9, 64, "bf16", 31)])
def test_spu_equal_samples_with_keep_counts_of_their_own(oracle, n, count, D, dtype, seed):
    """Equal samples are scored together whatever they keep: the first two batches score on another kernel together than one
    by one, whose need the workspace query would not have covered."""
    spu_ragged_case(oracle, [n] * count, D, dtype, 0.1, seed, sigmas=[4] * count, keeps=[n // 10 + i for i in range(count)])


def test_results_own_their_memory():
    """Every result is a tensor of its own: kept, resized or saved without the others, and aligned like any allocation."""
    merged = lv.luvc_oim_merge_ragged(torch.randn((3 * 5 + 4 * 4, 16), device="cuda"), [(3, 5), (4, 4)], [[(1, 2)], [(0, 1)]])
    stage = lv.luvc_spu_stage_ragged(torch.randn((9 + 7, 16), device="cuda"), [9, 7], [2, 1], [3, 2])
    torch.cuda.synchronize()
    results = [merged[k] for k in ("x", "sizes", "merged_map", "kept_map")] + [stage[k] for k in ("scores", "kept_idx", "origin", "x")]
    assert len({t.untyped_storage().data_ptr() for t in results}) == len(results)
    assert all(t.storage_offset() == 0 and t.untyped_storage().nbytes() == t.numel() * t.element_size() for t in results)


def test_ragged_errors():
    x = torch.zeros((20, 8), device="cuda")
    with pytest.raises(lv.LuvcError):
        lv.luvc_spu_stage_ragged(x, [12, 8], [7, 1], [3, 3])                   # sigma > N/2 in the first sample
    with pytest.raises(lv.LuvcError):
        lv.luvc_spu_stage_ragged(x, [12, 8], [2, 1], [3, 9])                   # keep > N in the second sample
    with pytest.raises(lv.LuvcError):
        lv.luvc_oim_merge_ragged(x, [(2, 5), (2, 5)], [[(1, 2)], [(1, 4)]])    # m too large for the second image
    with pytest.raises(lv.LuvcError):
        lv.luvc_oim_plan_anyres(0, 4, 10)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_oim_more_runs_than_a_launch_takes(oracle, dtype):
    """Runs that share launches: more of them than one argument list holds, images that stay as they are, take one pass, a pair
    of passes or several steps, and rows that no such launch takes."""
    shapes = [(1 + i % 9, 3 + (5 * i) % 23) for i in range(40)] + [(31, 18), (18, 31), (26, 26)]
    oim_ragged_case(oracle, shapes, 40, dtype, 36, 11, with_sizes=True)
    oim_ragged_case(oracle, shapes[30:], 33, dtype, 36, 12, with_sizes=False)


def halvings(h, w, axes):
    out = []
    for a in axes:
        out.append((a, ((w if a else h) + 1) // 2))
        h, w = (h, w - out[-1][1]) if a else (h - out[-1][1], w)
    return out


# pairs of passes and single ones in either order, so that runs meet in a launch at different steps of theirs; a single pass
# comes first for all of the first batch, a pair for most of the others; one image keeps its tokens
@pytest.mark.parametrize("axes", [["00", "001", "110", "0", "1", "0010"],
                                  ["10", "1", "101", "0101", "0", "10011", "01", "", "01010"],
                                  ["111", "10", "0110", "00", "1101"]])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_oim_runs_that_meet_at_different_steps(oracle, dtype, axes):
    shapes = [(17 + 3 * i, 16 + 5 * i) for i in range(len(axes))]
    schedules = [halvings(h, w, [int(a) for a in ax]) or [(0, 0)] for (h, w), ax in zip(shapes, axes)]
    oim_ragged_case(oracle, shapes, 40, dtype, 0, 13, with_sizes=True, schedules=schedules)


@pytest.mark.parametrize("axes", [["1101", "10101"], ["0010", "10101", "1010"], ["110", "1010"], ["1", "10101", "001"]])
def test_oim_runs_take_no_more_launches_than_step_by_step(oracle, axes):
    """Runs that gather for one kind of step never cost more launches than a launch per step and kind."""
    shapes = [(48 + 3 * i, 40 + 5 * i) for i in range(len(axes))]
    schedules = [halvings(h, w, [int(a) for a in ax]) for (h, w), ax in zip(shapes, axes)]
    kinds = []
    for ax in axes:                                      # a pair is two passes on different axes
        kinds.append([])
        while ax:
            kinds[-1].append(2 if len(ax) > 1 and ax[0] != ax[1] else 1)
            ax = ax[kinds[-1][-1]:]
    by_steps = sum(len({k[s] for k in kinds if s < len(k)}) for s in range(max(map(len, kinds))))
    x = torch.randn((sum(h * w for h, w in shapes), 40), device="cuda").to(torch.bfloat16)
    lv.luvc_oim_merge_ragged(x, shapes, schedules)
    prof = lv.LaunchProfile(64)
    prof.start()
    lv.luvc_oim_merge_ragged(x, shapes, schedules)
    prof.stop()
    torch.cuda.synchronize()
    launches = [name for name, _ in prof.results()]
    prof.close()
    assert 0 < sum(name.startswith("oim_halve") for name in launches) <= by_steps, (by_steps, launches)
    oim_ragged_case(oracle, shapes, 40, "bf16", 0, 14, with_sizes=True, schedules=schedules)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_spu_more_runs_than_a_launch_takes(oracle, dtype):
    """More runs of short samples than one argument list holds, with samples of other kernels between them."""
    lengths = list(range(1, 71)) + [1030, 1030] + list(range(130, 70, -7)) + [4100, 5, 5, 1024]
    spu_ragged_case(oracle, lengths, 34, dtype, 0.2, 21, origin_shift=3)
    spu_ragged_case(oracle, lengths[60:80], 33, dtype, 0.3, 22)
