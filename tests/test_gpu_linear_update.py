"""nm_linear_update (one call: prune, update GEMM, conversion, bias gradient) against the oracle on operands padded with zero
rows, at the edges of what it does itself: token counts inside a group (h and g end there; what lies behind them in memory is NaN),
one group, slabs whose last one is short, tiles of every plan, row strides, the ReLU's derivative, 8-bit operands."""
import numpy as np
import pytest
import torch

from paper_2203_10991_amd import synth
from gpu_util import DEV

pytestmark = pytest.mark.gpu


def _bits(t):
    return t.contiguous().view(torch.int16).cpu().numpy().view(np.uint16)


def _behind_nan(t, ld):
    """t as a view of row stride ld with NaN in the padding columns and in 40 rows behind it"""
    wide = torch.full((t.shape[0] + 40, ld), float("nan"), dtype=t.dtype, device=DEV)
    wide[:t.shape[0], :t.shape[1]] = t
    return wide[:t.shape[0], :t.shape[1]]


def _padded(t, m):
    return torch.nn.functional.pad(t, (0, 0, 0, (-t.shape[0]) % m))


# T (ragged and not), O, I: 64x64 tiles with the tokens split over the waves, in one slab and in several, in 8 bits up to two rounds of them; bf16 128x128 tiles in slabs
# and 256x128 ones; 8-bit 128x256 tiles
SHAPES = [(1, 8, 16), (15, 72, 48), (16, 64, 64), (17, 136, 80), (33, 256, 128), (1576, 256, 128), (3001, 128, 64), (2047, 2048, 1024), (3183, 3072, 1536)]


# (the plans are the same for every estimator: the large shapes run once per operand width)
@pytest.mark.parametrize("form,T,O,I", [(f, *s) for f in ("2:4", "1:2", "approx", "q8", "relu") for s in SHAPES
                                        if s[1] * s[2] <= 1 << 20 or f in ("2:4", "q8")])
def test_linear_update_matches_the_oracle(oracle, form, T, O, I):
    from paper_2203_10991_amd import api
    torch.manual_seed(T)
    g = (torch.randn(T, O, device=DEV) * torch.exp(2 * torch.randn(T, O, device=DEV))).to(torch.bfloat16)
    g[torch.rand(T, O, device=DEV) < 0.2] = 0
    h = torch.randn(T, I, device=DEV).to(torch.bfloat16)
    gn, hn = _behind_nan(g, O + 8), _behind_nan(h, I + 24)
    q8, act = form == "q8", None
    if form == "relu":
        act = torch.relu(torch.randn(T, O, device=DEV)).to(torch.bfloat16)
    nm_, mode = ("1:2" if form == "1:2" else "2:4"), int(form == "approx")
    dW, db, g_out = api.nm_linear_update(gn, hn, nm=nm_, mode=mode, q8=q8, seed=13, stream_id=4, bias=True,
                                         act=None if act is None else _behind_nan(act, O + 16))
    torch.cuda.synchronize()
    if act is not None:
        g = g * (act > 0).to(torch.bfloat16)
        assert torch.equal(g_out.view(torch.int16), g.view(torch.int16))
    gp, hp = _bits(_padded(g, 32 if q8 else 16)), _bits(_padded(h, 32 if q8 else 16))
    rows = None                                                            # large cases: a band of dW's rows is enough for the oracle
    if O * I > 1 << 20:
        rows = np.r_[0:8, 248:264, O - 8:O]
    cut = (lambda a: a) if rows is None else (lambda a: np.ascontiguousarray(a[:, rows]))
    if q8:
        sg, sh = oracle.pow2_scale(gp, 57344.0 / 4.0), oracle.pow2_scale(hp, 448.0)
        v, m = oracle.prune_2of4_q8(gp, 13, 4, 0, sg)
        want, wabs = oracle.update_gemm_q8(cut(v), cut(m), oracle.cast_e4m3(hp, sh), alpha=1.0 / (sg * sh))
    else:
        prune = {"1:2": oracle.prune_1of2, "approx": oracle.prune_2of4_approx}.get(form, oracle.prune_2of4)
        v, m, _ = prune(gp, 13, 4)
        want, wabs = oracle.update_gemm(cut(v), cut(m), hp)
    got = dW.double().cpu().numpy()
    got = got if rows is None else got[rows]
    tol = 1e-3 if q8 else 1e-5                                             # the 8-bit instruction's product window; binary32 sums
    assert np.isfinite(got).all()
    assert (np.abs(got - want) <= tol * wabs + 2.0 ** -8 * np.abs(want) + 1e-30).all()      # + the bf16 result's rounding
    assert np.linalg.norm(got - want) <= 3e-3 * np.linalg.norm(want)
    gd = g.double()
    err = (db.double() - gd.sum(0)).abs()
    assert bool((err <= 1e-5 * gd.abs().sum(0) + 2.0 ** -8 * gd.sum(0).abs()).all())


def test_linear_update_large_plan_with_ragged_tokens():
    """enough tiles for the 384-row kernel, whose operands are copied to whole groups: against the separate calls"""
    import paper_2203_10991_amd as nm
    from paper_2203_10991_amd import api
    torch.manual_seed(1)
    T, O, I = 77, 6144, 3072
    g, h = torch.randn(T, O, device=DEV).to(torch.bfloat16), torch.randn(T, I, device=DEV).to(torch.bfloat16)
    dW, db, _ = api.nm_linear_update(_behind_nan(g, O + 8), _behind_nan(h, I + 8), seed=3, stream_id=1, bias=True)
    v, m, _ = nm.mvue_prune_2of4(_padded(g, 16), seed=3, stream_id=1)
    want = nm.nm_update_gemm(v, m, _padded(h, 16)).to(torch.bfloat16)
    assert torch.equal(dW, want)


def test_argument_errors_come_before_any_launch():
    from paper_2203_10991_amd import api, NmError
    lib = api.load()
    g = torch.zeros(64, 64, dtype=torch.bfloat16, device=DEV)
    p = g.data_ptr()
    ok = dict(g=p, ldg=64, act=None, lda=0, h=p + 4096, ldh=64, T=16, O=64, I=64, m=4, mode=0, q8=0, seed=0, stream=0, gout=None, ldgo=0,
              dW=p, db=None, ws=p, wb=1 << 30, st=None)
    def call(**kw):
        return lib.nm_linear_update(*{**ok, **kw}.values())
    assert call(m=3) == 7 and call(mode=2) == 7 and call(m=2, mode=1) == 7 and call(q8=1, act=p, gout=p) == 7
    assert call(O=60) == 2 and call(T=0) == 2 and call(q8=1, I=24) == 2 and call(ldg=32) == 2
    assert call(h=None) == 1 and call(act=p) == 1 and call(dW=None) == 1
    assert call(dW=p + 2) == 4 and call(ldg=68) == 4
    assert call(wb=16) == 6 and call(ws=None) == 6
    assert call() == 5 and lib.nm_linear_update_workspace(16, 60, 64, 0, 0) == 0


def test_views_off_a_16_byte_boundary_are_copied():
    """g, h and act as views that start 2 bytes past a boundary, at row strides the kernels take"""
    from paper_2203_10991_amd import api
    torch.manual_seed(5)
    T, O, I = 40, 64, 48
    make = lambda n: torch.randn(T, n, device=DEV).to(torch.bfloat16)      # noqa: E731
    g, h, act = make(O), make(I), torch.relu(make(O))

    def shifted(t):
        wide = torch.full((T * 80 + 8,), float("nan"), dtype=t.dtype, device=DEV)
        v = wide[1:1 + T * 80].view(T, 80)[:, :t.shape[1]]
        v.copy_(t)
        assert v.data_ptr() % 16
        return v
    want = api.nm_linear_update(g, h, seed=2, act=act, bias=True)
    got = api.nm_linear_update(shifted(g), shifted(h), seed=2, act=shifted(act), bias=True)
    assert all(torch.equal(a, b) for a, b in zip(got, want))


@pytest.mark.parametrize("form,O,T,ld", [("2:4", 8, 2100, 1 << 21),        # 256 threads of four columns span 2048 tokens: 8 GiB at this stride
                                         ("relu", 8, 2100, 1 << 21),
                                         ("q8", 8, 4200, 1 << 20),         # ... 4096 tokens
                                         ("q8", 16, 2100, 1 << 21),        # ... 2048
                                         ("q8", 24, 1500, 1 << 21)])       # ... up to 1408, waves that start inside a row of groups
def test_row_strides_that_put_a_workgroups_rows_beyond_4_gib(form, O, T, ld):
    """g, h, act and g_out as columns of matrices with very long rows: the same bits as from contiguous operands"""
    from paper_2203_10991_amd import api
    torch.manual_seed(O)
    I, q8 = 16, form == "q8"
    wide = torch.empty(T * ld, dtype=torch.bfloat16, device=DEV).view(T, ld)

    def column(t, at):
        v = wide[:, at:at + t.shape[1]]
        v.copy_(t)
        return v
    g = (torch.randn(T, O, device=DEV) * torch.exp(2 * torch.randn(T, O, device=DEV))).to(torch.bfloat16)
    h = torch.randn(T, I, device=DEV).to(torch.bfloat16)
    act = torch.relu(torch.randn(T, O, device=DEV)).to(torch.bfloat16) if form == "relu" else None
    kw = dict(q8=q8, seed=3, stream_id=1, bias=True)
    want = api.nm_linear_update(g, h, act=act, **kw)
    gv, hv, av = column(g, 0), column(h, 64), None if act is None else column(act, 128)
    got = api.nm_linear_update(gv, hv, act=av, **kw)
    assert all(a is None and b is None or torch.equal(a, b) for a, b in zip(got, want))
    if act is None:
        return
    out = torch.empty(T * ld, dtype=torch.bfloat16, device=DEV).view(T, ld)
    for row in (0, 1023, 1024, 2047, T - 1):
        out[row, O:O + 8] = 7.0                                            # (what lies beside the rows stays as it is)
    lib, dW, db = api.load(), torch.empty_like(want[0]), torch.empty_like(want[1])
    ws = torch.empty(lib.nm_linear_update_workspace(T, O, I, 0, 1), dtype=torch.uint8, device=DEV)
    assert lib.nm_linear_update(gv.data_ptr(), ld, av.data_ptr(), ld, hv.data_ptr(), ld, T, O, I, 4, 0, 0, 3, 1, out.data_ptr(), ld, dW.data_ptr(),
                                db.data_ptr(), ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream) == 0
    assert torch.equal(dW, want[0]) and torch.equal(db, want[1]) and torch.equal(out[:, :O], want[2])
    assert bool((out[[0, 1023, 1024, 2047, T - 1], O:O + 8] == 7.0).all())


@pytest.mark.parametrize("cls,precision", [("NMLinear", "native"), ("NMLinear", "q8"), ("NMLinearReLU", "q8")])
def test_the_bias_gradient_stays_differentiable_under_create_graph(cls, precision):
    """db = column sums of the incoming gradient (times the ReLU's derivative): its derivative with respect to that gradient"""
    from paper_2203_10991_amd import autograd
    torch.manual_seed(8)
    layer = getattr(autograd, cls)(64, 32, cfg=autograd.NMConfig(precision=precision), device=DEV, dtype=torch.bfloat16)
    x = torch.randn(40, 64, device=DEV).to(torch.bfloat16)
    gy = torch.randn(40, 32, device=DEV).to(torch.bfloat16).requires_grad_()
    v = torch.randn(32, device=DEV).to(torch.bfloat16)
    y = layer(x)
    dW, db = torch.autograd.grad(y, (layer.weight, layer.bias), gy, create_graph=True)
    (ggy,) = torch.autograd.grad((db * v).sum(), gy)
    want = v.expand(40, 32)
    assert torch.equal(ggy, torch.where(y > 0, want, 0) if cls == "NMLinearReLU" else want)
    plain = torch.autograd.grad(layer(x), (layer.weight, layer.bias), gy.detach())
    assert torch.equal(dW, plain[0])
    g = gy.detach().double() * ((y > 0) if cls == "NMLinearReLU" else 1.0)
    # both sums are in binary32 and rounded once to bf16
    for b in (db, plain[1]):
        assert bool(((b.double() - g.sum(0)).abs() <= 2.0 ** -8 * g.sum(0).abs() + 1e-5 * g.abs().sum(0)).all())


@pytest.mark.parametrize("q8,nmode,mode,relu", [(True, "2:4", 1, False), (True, "1:2", 0, False), (False, "2:4", 1, True), (False, "1:2", 0, True)])
@pytest.mark.parametrize("T,O,I", SHAPES[:7])
def test_linear_update_of_the_other_estimators_matches_the_oracle(oracle, q8, nmode, mode, relu, T, O, I):
    """8-bit approx-MVUE and MVUE 1:2, and both behind a ReLU's derivative: masks through dW, and the bias gradient"""
    from paper_2203_10991_amd import api
    torch.manual_seed(T + 1)
    g = (torch.randn(T, O, device=DEV) * torch.exp(2 * torch.randn(T, O, device=DEV))).to(torch.bfloat16)
    g[torch.rand(T, O, device=DEV) < 0.2] = 0
    h = torch.randn(T, I, device=DEV).to(torch.bfloat16)
    act = torch.relu(torch.randn(T, O, device=DEV)).to(torch.bfloat16) if relu else None
    dW, db, g_out = api.nm_linear_update(_behind_nan(g, O + 8), _behind_nan(h, I + 24), nm=nmode, mode=mode, q8=q8, seed=19, stream_id=5, bias=True,
                                         act=None if act is None else _behind_nan(act, O + 16))
    if relu:
        g = g * (act > 0).to(torch.bfloat16)
        assert torch.equal(g_out.view(torch.int16), g.view(torch.int16))
    gp, hp = _bits(_padded(g, 32 if q8 else 16)), _bits(_padded(h, 32 if q8 else 16))
    if q8:
        sg, sh = oracle.pow2_scale(gp, 57344.0 / (4.0 if nmode == "2:4" else 2.0)), oracle.pow2_scale(hp, 448.0)
        v, m = oracle.prune_1of2_q8(gp, 19, 5, sg) if nmode == "1:2" else oracle.prune_2of4_q8(gp, 19, 5, mode, sg)
        want, wabs = oracle.update_gemm_q8(v, m, oracle.cast_e4m3(hp, sh), alpha=1.0 / (sg * sh))
    else:
        v, m, _ = (oracle.prune_1of2 if nmode == "1:2" else oracle.prune_2of4_approx)(gp, 19, 5)
        want, wabs = oracle.update_gemm(v, m, hp)
    got = dW.double().cpu().numpy()
    # tolerances as in the first test of this file
    assert (np.abs(got - want) <= (1e-3 if q8 else 1e-5) * wabs + 2.0 ** -8 * np.abs(want) + 1e-30).all()
    assert np.linalg.norm(got - want) <= 3e-3 * np.linalg.norm(want)
    gd = g.double()
    assert bool(((db.double() - gd.sum(0)).abs() <= 1e-5 * gd.abs().sum(0) + 2.0 ** -8 * gd.sum(0).abs()).all())


# the layer's scales come from the maxima that each workgroup of the pass over its tensors leaves: 1, 2, a few and nearly all 256 of them a tensor, the
# maximum in the first, in the last and in neither workgroup's share, no maximum (zeros), none that is finite
@pytest.mark.parametrize("T,O,I", [(32, 8, 16), (1056, 64, 144), (4096, 512, 64), (40960, 64, 512)])
def test_layer_scales_are_those_of_the_scale_records(T, O, I):
    from paper_2203_10991_amd import api
    torch.manual_seed(T)
    g0 = torch.randn(T, O, device=DEV).to(torch.bfloat16).clamp(-3, 3)
    h0 = torch.randn(T, I, device=DEV).to(torch.bfloat16).clamp(-3, 3)
    for spot in ("first", "last", "middle", "zeros", "infinite"):
        g, h = g0.clone(), h0.clone()
        if spot == "zeros":
            h.zero_()
        else:
            r = {"first": 0, "last": T - 1, "middle": T // 2, "infinite": T // 3}[spot]
            h[r, -1 if spot == "last" else 0] = -1000.0
            g[r, -1 if spot == "last" else 0] = float("inf") if spot == "infinite" else 3000.0
        rg, rh = api.nm_q8_scale(g, 57344.0 / 4.0), api.nm_q8_scale(h, 448.0)
        v, m = api.mvue_prune_2of4_q8(g, seed=3, stream_id=2, scale=rg)
        want = api.nm_update_gemm_q8(v, m, api.nm_cast_e4m3(h, rh), alpha=float(rg[1] * rh[1]))
        got = api.nm_linear_update(g, h, q8=True, seed=3, stream_id=2)[0]
        # the same operands on the same plan, summed in the same order: one rounding to bf16 apart
        assert torch.equal(got.view(torch.int16), want.to(torch.bfloat16).view(torch.int16)), spot


# the prune with a quad to a lane up to 10 * 2^20 elements (approx-MVUE 16384 * 4096), the one with a token group to a lane beyond it
@pytest.mark.parametrize("form,T,O,I", [("2:4", 4096, 2560, 16), ("2:4", 4097, 2560, 16), ("relu", 4095, 2560, 16), ("relu", 5001, 2104, 16),
                                        ("approx", 16380, 4096, 16), ("approx", 16385, 4104, 16)])
def test_layers_on_either_side_of_the_prunes_lines(oracle, form, T, O, I):
    test_linear_update_matches_the_oracle(oracle, form, T, O, I)


# MVUE 1:2 with four lanes to a group up to 10 * 2^20 elements, the 8-bit prune with eight up to 40 * 2^20; last waves that are not whole
@pytest.mark.parametrize("form,T,O,I", [("1:2", 4095, 2560, 16), ("1:2", 4097, 2568, 16), ("q8", 10239, 4096, 16), ("q8", 10241, 4104, 16), ("q8", 33, 40, 16)])
def test_layers_on_either_side_of_further_lines(oracle, form, T, O, I):
    test_linear_update_matches_the_oracle(oracle, form, T, O, I)


# 128 x 128 tiles with the only, the first few or all stages of their ring ending inside a token group
@pytest.mark.parametrize("form", ["2:4", "relu"])
@pytest.mark.parametrize("T", [1, 17, 33, 200])
def test_ragged_short_reductions_on_128_x_128_tiles(oracle, form, T):
    from gpu_util import kernels_of
    from paper_2203_10991_amd import api
    test_linear_update_matches_the_oracle(oracle, form, T, 2048, 1032)
    g, h = (torch.randn(T, n, device=DEV).to(torch.bfloat16) for n in (2048, 1032))
    assert any("update_gemm_smfmac_kernel<2, 2, 2, 2, false, true>" in n for n in kernels_of(lambda: api.nm_linear_update(g, h)))


# beyond the prunes' small forms, a last wave that is not whole: plain stores up to 20 * 2^20 elements, streaming ones beyond and for whole waves
@pytest.mark.parametrize("form,T,O,cached", [("2:4", 5121, 2056, True), ("relu", 10199, 2056, True), ("1:2", 7085, 1608, True), ("relu", 10201, 2056, False),
                                             ("2:4", 5121, 2048, False)])
def test_the_stores_of_a_last_wave_that_is_not_whole(oracle, form, T, O, cached):
    from gpu_util import kernels_of
    from paper_2203_10991_amd import api
    test_linear_update_matches_the_oracle(oracle, form, T, O, 16)
    g, h = torch.zeros(T, O, dtype=torch.bfloat16, device=DEV), torch.zeros(T, 16, dtype=torch.bfloat16, device=DEV)
    names = kernels_of(lambda: api.nm_linear_update(g, h, nm="1:2" if form == "1:2" else "2:4", act=g if form == "relu" else None))
    assert any(f"prune_layer_kernel<{2 if form == '1:2' else 4}, 0, {2 if form == 'relu' else 0}, {str(cached).lower()}>" in n for n in names)


# sizes at which a layer, whose finishing pass runs either way, is faster on the tile kernels than on 64 x 64 tiles with the tokens split over the waves
@pytest.mark.parametrize("T,O,I", [(3104, 264, 1824), (4076, 1880, 352), (5470, 320, 3120)])
def test_layers_that_stay_on_the_tile_kernels(oracle, T, O, I):
    from gpu_util import kernels_of
    from paper_2203_10991_amd import api
    test_linear_update_matches_the_oracle(oracle, "2:4", T, O, I)
    g, h = (torch.randn(T, n, device=DEV).to(torch.bfloat16) for n in (O, I))
    names = kernels_of(lambda: api.nm_linear_update(g, h))
    assert any("update_gemm" in n for n in names) and not any("small_kernel" in n for n in names)


@pytest.mark.parametrize("T,O,I", [(1152, 2240, 1712), (2979, 760, 2080), (1576, 768, 3072), (12162, 360, 1888)])
def test_8_bit_layers_that_stay_on_the_tile_kernels(oracle, T, O, I):
    from gpu_util import kernels_of
    from paper_2203_10991_amd import api
    test_linear_update_matches_the_oracle(oracle, "q8", T, O, I)
    g, h = (torch.randn(T, n, device=DEV).to(torch.bfloat16) for n in (O, I))
    names = kernels_of(lambda: api.nm_linear_update(g, h, q8=True))
    assert any("update_gemm" in n for n in names) and not any("small_kernel" in n for n in names)
