"""GPU parity of the 8-bit path (e5m2 neural gradients by stochastic rounding on top of MVUE 2:4, e4m3
activations, 8-bit sparse MFMA) against the CPU oracle, through the C ABI.

  * mvue_prune_2of4_q8: vals8 / meta32 bit for bit, both estimators, bf16 and binary32 inputs, strided input.
  * nm_update_gemm_q8: against the oracle's binary64 sums.  The 8-bit matrix instruction adds the 64 products of a
    step in a fixed-point window below the largest of them before the binary32 accumulation, so small products
    lose low bits next to large ones: tolerance 1e-3 of the sum of absolute products (observed up to 2e-4 on
    lognormal gradients, printed; ten times tighter than the 16-bit path's 1e-2).
"""
import numpy as np
import pytest
import torch

from paper_2203_10991_amd import synth
from gpu_util import DEV, to_dev

pytestmark = pytest.mark.gpu
TOL = 1e-3


@pytest.fixture(scope="module")
def nm():
    import paper_2203_10991_amd as p
    p.load()
    return p


def fit_scale(g_f32: np.ndarray) -> float:
    """power of two that keeps every kept value (at most the sum of a quad's magnitudes) below the largest e5m2"""
    m = float(np.abs(g_f32).max())
    return float(2.0 ** np.floor(np.log2(57344.0 / (4.0 * max(m, 1e-30)))))


def as_f32(g: np.ndarray) -> np.ndarray:
    return g if g.dtype == np.float32 else synth.bf16_to_f32(g)


def h8_codes(T, I, seed, relu=False):
    """e4m3 codes of a scaled normal (or half-normal with zeros) activation tensor: numpy draw, torch's nearest cast"""
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((T, I)).astype(np.float32) * 8.0
    if relu:
        x = np.where(rng.random((T, I)) < 0.5, 0.0, np.abs(x)).astype(np.float32)
    return torch.from_numpy(x).to(torch.float8_e4m3fn).view(torch.uint8).numpy()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("T,O", [(32, 8), (64, 64), (32 * 7, 8 * 13), (32 * 40, 8 * 67), (2048, 1024)])
def test_prune_q8_bit_exact(nm, oracle, dtype, mode, T, O):
    w = synth.Workload(f"q8_{T}x{O}", T, O, 16, dtype, "2:4", 0.0, 2.5, 0.3)
    g = synth.make_g(w, seed=T + O + mode)
    scale = fit_scale(as_f32(g))
    ov, om = oracle.prune_2of4_q8(g, seed=77, stream_id=3, mode=mode, scale=scale)
    v, m = nm.mvue_prune_2of4_q8(to_dev(g), seed=77, stream_id=3, mode=mode, scale=scale)
    torch.cuda.synchronize()
    assert np.array_equal(m.cpu().numpy().view(np.uint32), om)
    assert np.array_equal(v.cpu().numpy(), ov)


# the largest launches with a quad to a lane (approx-MVUE 16384 x 4096, optimal 10240 x 4096, MVUE 1:2 8192 x 4096) and the first ones beyond, a padded stride
@pytest.mark.parametrize("which,T", [("approx", 16384), ("approx", 16416), ("2of4", 10240), ("2of4", 10272), ("1of2", 8192), ("1of2", 8224)])
def test_prune_q8_on_either_side_of_the_lines(nm, oracle, which, T):
    O = 4096
    g = synth.make_g(synth.Workload("q8", T, O, 16, "bf16", "2:4", 0.0, 2.5, 0.3), seed=T)
    scale, seed = fit_scale(as_f32(g)), (1 << 40) + 7
    d = torch.zeros((T, O + 8), dtype=torch.bfloat16, device=DEV)
    d[:, :O] = to_dev(g)
    if which == "1of2":
        (ov, om), (v, m) = oracle.prune_1of2_q8(g, seed, 3, scale), nm.mvue_prune_1of2_q8(d[:, :O], seed=seed, stream_id=3, scale=scale)
    else:
        mode = int(which == "approx")
        (ov, om), (v, m) = oracle.prune_2of4_q8(g, seed, 3, mode, scale), nm.mvue_prune_2of4_q8(d[:, :O], seed=seed, stream_id=3, mode=mode, scale=scale)
    assert np.array_equal(m.cpu().numpy().view(np.uint32), om) and np.array_equal(v.cpu().numpy(), ov)


def test_prune_q8_strided_input_small_and_large_scales(nm, oracle):
    """row stride larger than O; scales that push kept values into the subnormal range and into saturation"""
    T, O = 96, 40
    w = synth.Workload("q8_strided", T, O, 16, "bf16", "2:4", 0.0, 3.0, 0.3)
    g = synth.make_g(w, seed=4)
    wide = torch.zeros((T, O + 24), dtype=torch.bfloat16, device=DEV)
    wide[:, :O] = to_dev(g)
    base = fit_scale(as_f32(g))
    for scale in (base, base * 2.0 ** -22, base * 2.0 ** -30, base * 64.0, 1e30):
        ov, om = oracle.prune_2of4_q8(g, seed=1, stream_id=0, mode=0, scale=scale)
        v, m = nm.mvue_prune_2of4_q8(wide[:, :O], seed=1, stream_id=0, mode=0, scale=scale)
        torch.cuda.synchronize()
        assert np.array_equal(m.cpu().numpy().view(np.uint32), om), scale
        assert np.array_equal(v.cpu().numpy(), ov), scale
    sat = (ov & 0x7F) == 0x7B
    assert sat.any()                                        # the last scale saturates


def test_prune_q8_same_mask_as_the_16_bit_prune(nm):
    """same seed, same stream: the 8-bit prune keeps the positions the 16-bit prune keeps"""
    T, O = 256, 128
    w = synth.Workload("q8_mask", T, O, 16, "bf16", "2:4", 0.0, 2.0, 0.2)
    g = to_dev(synth.make_g(w, seed=8))
    for mode in (0, 1):
        _, m16, _ = nm.mvue_prune_2of4(g, seed=9, stream_id=1, mode=mode)
        _, m32 = nm.mvue_prune_2of4_q8(g, seed=9, stream_id=1, mode=mode, scale=4.0)
        torch.cuda.synchronize()
        m16 = m16.cpu().numpy().view(np.uint16).astype(np.uint32)
        assert np.array_equal(m32.cpu().numpy().view(np.uint32), m16[0::2] | (m16[1::2] << 16))


def gemm_case(nm, oracle, T, O, I, seed, beta=0.0, sample=None, relu=False):
    w = synth.Workload(f"q8_{T}x{O}x{I}", T, O, I, "bf16", "2:4", 0.0, 2.0, 0.3)
    g = synth.make_g(w, seed)
    scale = fit_scale(as_f32(g))
    ov, om = oracle.prune_2of4_q8(g, seed=seed, stream_id=0, mode=0, scale=scale)
    h8 = h8_codes(T, I, seed + 1, relu)
    alpha = 1.0 / (scale * 8.0)
    v, m = nm.mvue_prune_2of4_q8(to_dev(g), seed=seed, stream_id=0, mode=0, scale=scale)
    prior = np.random.default_rng(1).standard_normal((O, I)).astype(np.float32) if beta else None
    dW = torch.from_numpy(prior).to(DEV) if beta else torch.full((O, I), float("nan"), device=DEV)
    nm.nm_update_gemm_q8(v, m, torch.from_numpy(h8).to(DEV), dW=dW, alpha=alpha, beta=beta)
    torch.cuda.synchronize()
    assert np.array_equal(v.cpu().numpy(), ov) and np.array_equal(m.cpu().numpy().view(np.uint32), om)
    got = dW.cpu().numpy().astype(np.float64)
    assert np.isfinite(got).all()
    if sample is None:
        want, wabs = oracle.update_gemm_q8(ov, om, h8, alpha=alpha)
    else:                                   # whole rows and whole columns, chosen at random plus the edges
        rng = np.random.default_rng(seed)
        rows = np.unique(np.concatenate([rng.choice(O, sample, replace=False), [0, O - 1]]))
        cols = np.unique(np.concatenate([rng.choice(I, sample, replace=False), [0, I - 1]]))
        oi = np.concatenate([np.stack(np.meshgrid(rows, np.arange(I), indexing="ij"), -1).reshape(-1, 2),
                             np.stack(np.meshgrid(np.arange(O), cols, indexing="ij"), -1).reshape(-1, 2)])
        want, wabs = oracle.update_gemm_q8(ov, om, h8, alpha=alpha, oi=oi)
        got = got[oi[:, 0], oi[:, 1]]
        prior = prior[oi[:, 0], oi[:, 1]] if beta else None
    if beta:
        want = want + prior
        wabs = wabs + np.abs(prior)
    rel = float((np.abs(got - want) / np.maximum(wabs, 1e-300)).max())
    fro = float(np.linalg.norm(got - want) / max(np.linalg.norm(want), 1e-300))
    print(f"q8 T={T} O={O} I={I} beta={beta}: max |err|/sum|ab| = {rel:.3e}, frobenius = {fro:.3e}", flush=True)
    assert rel <= TOL and fro <= TOL


@pytest.mark.parametrize("T,O,I", [(64, 64, 64), (32, 8, 16), (32 * 11, 8 * 9, 16 * 7), (32 * 33, 64 * 3 + 8, 256 + 48),
                                   (1024, 256, 320), (32 * 13, 128, 256), (2048, 1000, 528)])
def test_update_gemm_q8_matches_fp64_oracle(nm, oracle, T, O, I):
    gemm_case(nm, oracle, T, O, I, seed=T + I)


def test_update_gemm_q8_beta_one_and_relu_activations(nm, oracle):
    gemm_case(nm, oracle, 32 * 9, 200, 272, seed=5, beta=1.0, relu=True)
    gemm_case(nm, oracle, 4096, 64, 576, seed=6, beta=1.0)             # few rows, slabs


# 64 x 64 tiles with the tokens split over the waves: one group, an odd number of groups in one and in many steps, ragged rows and columns, tiles for more
# than one round, slabs (the last one shorter)
@pytest.mark.parametrize("T,O,I,beta", [(32, 8, 16, 0.0), (32, 64, 80, 1.0), (96, 72, 64, 0.0), (544, 200, 112, 1.0), (992, 1016, 1008, 0.0), (1024, 2104, 976, 0.0),
                                        (8224, 512, 512, 0.0), (8192, 264, 528, 1.0)])
def test_update_gemm_q8_small_kernel(nm, oracle, T, O, I, beta):
    from gpu_util import kernels_of
    gemm_case(nm, oracle, T, O, I, seed=T + O, beta=beta)
    v, m = nm.mvue_prune_2of4_q8(torch.randn(T, O, device=DEV).to(torch.bfloat16), seed=1, scale=16.0)
    h8 = torch.from_numpy(h8_codes(T, I, 1)).to(DEV)
    assert any("update_gemm_q8_small_kernel" in n for n in kernels_of(lambda: nm.nm_update_gemm_q8(v, m, h8, alpha=1.0)))


# up to eight rows of those tiles, whose XCDs take runs of all slabs' tiles: numbers of tiles that do not divide by eight, one slab and several; nine rows
@pytest.mark.parametrize("T,O,I,beta", [(96, 72, 144, 0.0), (2080, 72, 720, 1.0), (4128, 120, 464, 0.0), (6016, 200, 336, 1.0), (1056, 456, 1104, 0.0), (8032, 520, 144, 0.0)])
def test_update_gemm_q8_small_kernel_over_the_xcds(nm, oracle, T, O, I, beta):
    test_update_gemm_q8_small_kernel(nm, oracle, T, O, I, beta)


@pytest.mark.parametrize("T,O,I", [(160, 16 * 256, 16 * 256),            # 16 x 16 tiles of 256 x 256: the 2 x 4 XCD grid; odd group count
                                   (96, 50 * 256 - 40, 8 * 256),         # banded map with a short last band, ragged rows
                                   (32 * 14, 33 * 256, 8 * 256 - 16)])   # more than two trips of stages, ragged columns
def test_update_gemm_q8_large_tile_kernel(nm, oracle, T, O, I):
    gemm_case(nm, oracle, T, O, I, seed=T, sample=12)


@pytest.mark.parametrize("T,O,I,slabs,beta", [(4128, 2040, 2000, 2, 0.0), (2080, 2296, 4080, 0, 1.0), (16416, 2040, 2000, 4, 0.0)])
def test_update_gemm_q8_mid_sized_plans(nm, oracle, T, O, I, slabs, beta):
    """mid-sized problems: up to 256 tiles of 128 x 256 run on that tile with the token axis cut into slabs (here 128
    tiles, two slabs, the scale applied in the second pass); beyond that on 256 x 256 tiles in one round (here 144
    tiles), and so do 48 tiles or more under a long reduction (here 64 tiles in four slabs); ragged last tile row and
    column, ragged last slab"""
    assert nm.nm_update_gemm_q8_workspace(T, O, I) == (slabs * O * I * 4 if slabs > 1 else 0)
    gemm_case(nm, oracle, T, O, I, seed=T, beta=beta, sample=10)


# second passes over the partial sums of up to eight slabs of 64 x 64 tiles, and of 140 slabs of the tile kernels (eight threads to a sum); slabs: what the tile
# kernels' plan asks for as workspace (the forms of the second pass that more slabs take: test_update_gemm_q8_tile_kernels)
@pytest.mark.parametrize("T,O,I,slabs", [(32 * 132, 64, 64, 11), (32 * 280, 64, 80, 12), (32 * 552, 72, 272, 46), (32 * 1680, 64, 64, 140), (32 * 280, 296, 256, 12),
                                         (32 * 1680, 296, 256, 70)])
def test_second_pass_over_partial_sums(nm, oracle, T, O, I, slabs):
    from paper_2203_10991_amd import api
    assert api.nm_update_gemm_q8_workspace(T, O, I) == slabs * O * I * 4
    sample = 16 if O > 64 else None
    gemm_case(nm, oracle, T, O, I, seed=5, sample=sample)
    gemm_case(nm, oracle, T, O, I, seed=6, beta=1.0, sample=sample)


def test_update_gemm_q8_beta_one_large_tile(nm, oracle):
    gemm_case(nm, oracle, 128, 16 * 256, 16 * 256, seed=3, beta=1.0, sample=8)


def _random_shapes(n, seed):
    rng = np.random.default_rng(seed)
    return [(int(rng.integers(1, 150)) * 32, int(rng.integers(1, 80)) * 8, int(rng.integers(1, 40)) * 16) for _ in range(n)]


@pytest.mark.parametrize("T,O,I", _random_shapes(12, 77))
def test_update_gemm_q8_random_shapes(nm, oracle, T, O, I):
    """seeded random problem sizes, which all run on 64 x 64 tiles, in one slab and in up to six"""
    gemm_case(nm, oracle, T, O, I, seed=T + O)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T,O", [(32, 8), (64, 64), (32 * 7, 8 * 13), (32 * 40, 8 * 67), (2048, 1024)])
def test_prune_1of2_q8_bit_exact(nm, oracle, dtype, T, O):
    w = synth.Workload(f"q8_12_{T}x{O}", T, O, 16, dtype, "1:2", 0.0, 2.5, 0.3)
    g = synth.make_g(w, seed=T + O + 3)
    scale = fit_scale(as_f32(g)) * 2.0                    # a kept value is at most the sum of TWO magnitudes
    ov, om = oracle.prune_1of2_q8(g, seed=78, stream_id=4, scale=scale)
    v, m = nm.mvue_prune_1of2_q8(to_dev(g), seed=78, stream_id=4, scale=scale)
    torch.cuda.synchronize()
    assert np.array_equal(m.cpu().numpy().view(np.uint32), om)
    assert np.array_equal(v.cpu().numpy(), ov)


def test_prune_1of2_q8_feeds_the_8_bit_gemm(nm, oracle):
    T, O, I = 32 * 12, 136, 144
    w = synth.Workload("q8_12_gemm", T, O, I, "bf16", "1:2", 0.0, 2.0, 0.3)
    g = synth.make_g(w, 5)
    scale = fit_scale(as_f32(g)) * 2.0
    ov, om = oracle.prune_1of2_q8(g, seed=5, stream_id=0, scale=scale)
    h8 = h8_codes(T, I, 6)
    alpha = 1.0 / (scale * 8.0)
    v, m = nm.mvue_prune_1of2_q8(to_dev(g), seed=5, stream_id=0, scale=scale)
    dW = nm.nm_update_gemm_q8(v, m, torch.from_numpy(h8).to(DEV), alpha=alpha)
    torch.cuda.synchronize()
    want, wabs = oracle.update_gemm_q8(ov, om, h8, alpha=alpha)
    got = dW.cpu().numpy().astype(np.float64)
    rel = float((np.abs(got - want) / np.maximum(wabs, 1e-300)).max())
    print(f"1:2 q8 gemm: max |err|/sum|ab| = {rel:.3e}", flush=True)
    assert rel <= TOL


# the tile kernels where the small one leaves them the call: 128 x 256 tiles in one pass, in two, five and ten slabs (one chain to a sum) and in more (eight threads or
# eight chains to a sum), 64 x 256 tiles, of which no plan has a single slab
@pytest.mark.parametrize("T,O,I,beta,tile,second", [
    (32, 1168, 1680, 0.0, "2, 4, 2, 2", None), (32, 1176, 1680, 1.0, "2, 4, 2, 2", None), (768, 2208, 1488, 1.0, "2, 4, 2, 2", "1, 1"), (3104, 800, 1232, 0.0, "2, 4, 2, 2", "1, 1"),
    (10976, 200, 2112, 0.0, "2, 4, 2, 2", "1, 1"), (3584, 176, 6368, 0.0, "2, 4, 2, 2", "1, 1"), (66496, 264, 16, 1.0, "2, 4, 2, 2", "8, 1"), (55296, 72, 16, 0.0, "2, 4, 2, 2", "8, 1"), (28576, 72, 1440, 1.0, "2, 4, 2, 2", "1, 8"),
    (58496, 104, 736, 0.0, "2, 4, 2, 2", "1, 8"), (65888, 8, 528, 0.0, "1, 4, 2, 2", "8, 1"), (53376, 8, 16, 1.0, "1, 4, 2, 2", "8, 1"), (49664, 40, 2144, 0.0, "1, 4, 2, 2", "1, 8")])
def test_update_gemm_q8_tile_kernels(nm, oracle, T, O, I, beta, tile, second):
    from gpu_util import kernels_of
    gemm_case(nm, oracle, T, O, I, seed=T + O, beta=beta)
    v, m = nm.alloc_compressed_q8(T, O, DEV)
    v.zero_(); m.fill_(0x44444444)
    h8, dW = torch.zeros(T, I, dtype=torch.uint8, device=DEV), torch.zeros(O, I, device=DEV)
    names = kernels_of(lambda: nm.nm_update_gemm_q8(v, m, h8, dW=dW, alpha=1.0, beta=beta))
    assert any(f"update_gemm_smfmac_q8_kernel<{tile}, false>" in n for n in names), names
    assert any("splitk_reduce" in n for n in names) == (second is not None) and (second is None or any(f"splitk_reduce_kernel<{second}>" in n for n in names))
