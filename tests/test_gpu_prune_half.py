"""The prune kernels with four bf16 columns per thread: sizes at which their launch changes form (one wave, a partly filled
workgroup, a thread count that is no multiple of a wave), the largest size that takes them and the first beyond it, padded
strides; vals and meta bit for bit against the oracle."""
import numpy as np
import pytest
import torch

from paper_2203_10991_amd import synth
from gpu_util import DEV, to_dev, to_host

pytestmark = pytest.mark.gpu


def _g(T, O, seed):
    w = synth.Workload("t", T, O, 8, "bf16", "2:4", 0.0, 2.5, 0.2)
    return synth.make_g(w, seed)


@pytest.mark.parametrize("T,O,ld", [(16, 256, 256), (16, 8, 8), (32, 128, 136), (48, 72, 72), (16, 264, 264), (1584, 96, 104), (64, 1024, 1024), (528, 40, 40)])
@pytest.mark.parametrize("which", ["1of2", "2of4", "approx"])
def test_small_sizes_match_the_oracle(oracle, T, O, ld, which):
    import paper_2203_10991_amd as nm
    g = _g(T, O, T + O)
    d = torch.zeros((T, ld), dtype=torch.bfloat16, device=DEV)
    d[:, :O] = to_dev(g)
    if which == "1of2":
        v, m, _ = nm.mvue_prune_1of2(d[:, :O], seed=7, stream_id=3)
        ov, om, _ = oracle.prune_1of2(g, 7, 3)
    elif which == "2of4":
        v, m, _ = nm.mvue_prune_2of4(d[:, :O], seed=7, stream_id=3)
        ov, om, _ = oracle.prune_2of4(g, 7, 3)
    else:
        v, m, _ = nm.mvue_prune_2of4(d[:, :O], seed=7, stream_id=3, mode=1)
        ov, om, _ = oracle.prune_2of4_approx(g, 7, 3)
    assert np.array_equal(to_host(m), om) and np.array_equal(to_host(v), ov)


@pytest.mark.parametrize("T", [16384, 16400])
@pytest.mark.parametrize("which", ["1of2", "2of4", "approx"])
def test_either_side_of_the_line_matches_the_oracle(oracle, T, which):
    import paper_2203_10991_amd as nm
    O = 4096
    g = _g(T, O, 5)
    gd = to_dev(g)
    if which == "1of2":
        v, m, _ = nm.mvue_prune_1of2(gd, seed=9, stream_id=1)
        ov, om, _ = oracle.prune_1of2(g, 9, 1)
    else:
        mode = 1 if which == "approx" else 0
        v, m, _ = nm.mvue_prune_2of4(gd, seed=9, stream_id=1, mode=mode)
        ov, om, _ = (oracle.prune_2of4_approx if mode else oracle.prune_2of4)(g, 9, 1)
    assert np.array_equal(to_host(m), om) and np.array_equal(to_host(v), ov)


@pytest.mark.parametrize("T", [4096, 4112])
def test_either_side_of_a_quad_to_a_lane_matches_the_oracle(oracle, T):
    """the optimal estimator with one quad to a lane up to 4096 x 2560, a padded stride"""
    import paper_2203_10991_amd as nm
    O = 2560
    g = _g(T, O, 6)
    d = torch.zeros((T, O + 24), dtype=torch.bfloat16, device=DEV)
    d[:, :O] = to_dev(g)
    v, m, _ = nm.mvue_prune_2of4(d[:, :O], seed=(5 << 32) + 9, stream_id=1)
    ov, om, _ = oracle.prune_2of4(g, (5 << 32) + 9, 1)
    assert np.array_equal(to_host(m), om) and np.array_equal(to_host(v), ov)


def _f32(T, O, seed):
    return synth.make_g(synth.Workload("t", T, O, 8, "f32", "2:4", 0.0, 2.0, 0.3), seed)


# binary32 with a quad to a lane: a wave and less, a partly filled workgroup, a padded stride; either side of its lines (1:2 2 * 2^20 elements, 2:4 40 * 2^20)
@pytest.mark.parametrize("T,O,ld", [(16, 8, 8), (16, 256, 256), (48, 72, 76), (1584, 96, 104), (528, 40, 40), (1024, 2048, 2048), (1040, 2048, 2048)])
@pytest.mark.parametrize("which", ["1of2", "2of4", "approx"])
def test_binary32_matches_the_oracle(oracle, T, O, ld, which):
    import paper_2203_10991_amd as nm
    g = _f32(T, O, T + O)
    g[:4, :8] = np.array([0.0, -0.0, 3e37, 1.5, 2.0 ** -140, 1.5, -1.5, 0.0], dtype=np.float32)
    d = torch.zeros((T, ld), dtype=torch.float32, device=DEV)
    d[:, :O] = to_dev(g)
    seed = (3 << 32) + 5
    if which == "1of2":
        v, m, _ = nm.mvue_prune_1of2(d[:, :O], seed=seed, stream_id=2)
        ov, om, _ = oracle.prune_1of2(g, seed, 2)
    else:
        v, m, _ = nm.mvue_prune_2of4(d[:, :O], seed=seed, stream_id=2, mode=int(which == "approx"))
        ov, om, _ = (oracle.prune_2of4_approx if which == "approx" else oracle.prune_2of4)(g, seed, 2)
    assert np.array_equal(to_host(m), om) and np.array_equal(to_host(v).view(np.uint32), ov.view(np.uint32))


@pytest.mark.parametrize("T", [10240, 10256])
def test_either_side_of_a_binary32_quad_to_a_lane(oracle, T):
    import paper_2203_10991_amd as nm
    O = 4096
    g = _f32(T, O, 4)
    v, m, _ = nm.mvue_prune_2of4(to_dev(g), seed=9, stream_id=1)
    ov, om, _ = oracle.prune_2of4(g, 9, 1)
    assert np.array_equal(to_host(m), om) and np.array_equal(to_host(v).view(np.uint32), ov.view(np.uint32))


@pytest.mark.parametrize("T", [4096, 4112])
def test_either_side_of_a_pair_row_to_a_lane_matches_the_oracle(oracle, T):
    """MVUE 1:2 in bf16 with four lanes to a group up to 4096 x 2560"""
    import paper_2203_10991_amd as nm
    O = 2560
    g = _g(T, O, 8)
    v, m, _ = nm.mvue_prune_1of2(to_dev(g), seed=9, stream_id=1)
    ov, om, _ = oracle.prune_1of2(g, 9, 1)
    assert np.array_equal(to_host(m), om) and np.array_equal(to_host(v), ov)


# beyond the lines of four lanes to a group: a last wave that is not whole
@pytest.mark.parametrize("T,O", [(4112, 2568), (10256, 1032), (16, 655368)])
@pytest.mark.parametrize("which", ["1of2", "2of4", "f32"])
def test_last_wave_partly_filled(oracle, T, O, which):
    import paper_2203_10991_amd as nm
    g = _f32(T, O, 3) if which == "f32" else _g(T, O, 3)
    if which == "2of4":
        (v, m, _), (ov, om, _) = nm.mvue_prune_2of4(to_dev(g), seed=2, stream_id=1), oracle.prune_2of4(g, 2, 1)
    else:
        (v, m, _), (ov, om, _) = nm.mvue_prune_1of2(to_dev(g), seed=2, stream_id=1), oracle.prune_1of2(g, 2, 1)
    u = np.uint32 if which == "f32" else np.uint16
    assert np.array_equal(to_host(m), om) and np.array_equal(to_host(v).view(u), ov.view(u))


# a last wave that is not whole, in each kernel that stores through descriptors: both forms of the one with four columns to a thread, the ones for large tensors of each
# estimator, Greedy and MVUE 1:4 at any size; what lies behind the outputs stays as it is
@pytest.mark.parametrize("which,T,O", [("2of4", 4112, 2568), ("1of2", 10256, 1032), ("2of4", 12208, 1736), ("1of2", 12208, 1736), ("2of4", 16400, 4104), ("approx", 16400, 4104),
                                       ("1of4", 48, 72), ("1of4", 16, 8), ("greedy2of4", 48, 72), ("greedy1of2", 16, 8), ("f32_1of2", 1040, 2056), ("f32_2of4", 10256, 4104),
                                       ("f32_approx", 10256, 4104), ("f32_1of4", 48, 72), ("f32_greedy2of4", 16, 8)])
def test_nothing_behind_the_outputs_is_written(oracle, which, T, O):
    import paper_2203_10991_amd as nm
    f32, form = which.startswith("f32_"), which.split("_")[-1]
    g = _f32(T, O, 3) if f32 else _g(T, O, 3)
    n, dt = T // 2 * O, torch.float32 if f32 else torch.bfloat16
    vb, mb = torch.full((n + 8192,), 7.0, dtype=dt, device=DEV), torch.full((T // 16 * O + 8192,), 0x1234, dtype=torch.int16, device=DEV)
    out = {"vals": vb[:n].view(T // 16, O, 8), "meta": mb[:T // 16 * O].view(T // 16, O)}
    if form.startswith("greedy"):
        k, m = int(form[6]), int(form[-1])
        nm.nm_prune_greedy(to_dev(g), k, m, **out)
        ov, om, _ = oracle.prune_greedy(g, k, m)
    elif form == "approx":
        nm.mvue_prune_2of4(to_dev(g), seed=2, stream_id=1, mode=1, **out)
        ov, om, _ = oracle.prune_2of4_approx(g, 2, 1)
    else:
        {"1of2": nm.mvue_prune_1of2, "2of4": nm.mvue_prune_2of4, "1of4": nm.mvue_prune_1of4}[form](to_dev(g), seed=2, stream_id=1, **out)
        ov, om, _ = {"1of2": oracle.prune_1of2, "2of4": oracle.prune_2of4, "1of4": oracle.prune_1of4}[form](g, 2, 1)
    u = np.uint32 if f32 else np.uint16
    assert np.array_equal(to_host(out["meta"]), om) and np.array_equal(to_host(out["vals"]).view(u), ov.view(u))
    assert bool((vb[n:] == 7.0).all()) and bool((mb[T // 16 * O:] == 0x1234).all())
