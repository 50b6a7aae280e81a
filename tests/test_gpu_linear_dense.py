"""nm_linear_forward and nm_linear_input_grad (the dense products of a linear layer) against binary64 sums of the same bf16 operands, at the
edges of their tiles, of a stage of 64 reduction steps and of a chunk of 8, on views whose padding is NaN; the layers that take
them, and those that do not."""
import pytest
import torch

from gpu_util import DEV, kernels_of

pytestmark = pytest.mark.gpu


def _behind_nan(t, ld):
    """t as a view of row stride ld with NaN in the padding columns and in 300 rows behind it"""
    wide = torch.full((t.shape[0] + 300, ld), float("nan"), dtype=t.dtype, device=DEV)
    wide[:t.shape[0], :t.shape[1]] = t
    return wide[:t.shape[0], :t.shape[1]]


def _check(got, x, w, bias=None, relu=False):
    """half a unit in the last place of bf16 (2^-9 of the value, up to 2^-8 where it is just above a power of two) and the binary32
    sums: K additions of at most 2^-24 of the sum of absolute products each, of which 1e-5 is a generous share up to K = 4096"""
    want, wabs = x.double() @ w.double(), x.double().abs() @ w.double().abs()
    if bias is not None:
        want, wabs = want + bias.double(), wabs + bias.double().abs()
    if relu:
        want = want.clamp_min(0)
    assert bool(((got.double() - want).abs() <= 2.0 ** -8 * want.abs() + 1e-5 * wabs + 1e-30).all())


SHAPES = [(1, 8, 8), (33, 40, 72), (64, 64, 64), (65, 72, 56), (197, 264, 256), (300, 136, 120),      # tokens, outputs, inputs: 64 x 64 tiles
          (2047, 1032, 72),                                                                       # 128 x 128 on eight waves
          (7222, 264, 72),                                                                         # 128 x 64
          (1579, 3080, 200),                                                                       # 128 x 128
          (5000, 2056, 264)]                                                                       # 256 x 256


# several tiles to a workgroup: stages that run on from one into the next, stores on their way with them, accumulators cleared in place, a reduction axis that
# ends inside a stage every time
SEVERAL_FORWARD = [(2435, 1608, 1312, "2, 2, 1, 1, false, 4"), (5116, 1568, 416, "2, 2, 2, 1, false, 3"), (9000, 3080, 72, "2, 2, 2, 2, false, 2"),
                   (9000, 4104, 200, "2, 2, 2, 2, false, 2"), (13357, 2016, 736, "2, 4, 4, 2, false, 2")]
SEVERAL_GRAD = [(2435, 856, 1656, "2, 2, 1, 1, true, 4"), (16251, 440, 528, "2, 2, 2, 1, true, 3"), (6390, 264, 2544, "2, 2, 2, 2, true, 2"),
                (13357, 736, 2016, "2, 4, 4, 2, true, 2")]


# 128 x 128 tiles on eight waves, four stages in LDS: fewer stages than that, a whole round of 256 tiles, ragged rows, features and reductions, nearly a round
# of tiles with few stages
EIGHT_WAVES = [(2047, 1032, 72), (2774, 944, 2976), (4096, 1024, 1544), (2040, 1912, 1608), (2130, 1400, 1440), (3886, 720, 864)]


@pytest.mark.parametrize("T,O,I", EIGHT_WAVES)
def test_tiles_on_eight_waves(T, O, I):
    from paper_2203_10991_amd import api
    test_linear_forward(T, O, I)
    test_linear_input_grad(T, I, O)
    x, w, v = (torch.zeros(*s, device=DEV, dtype=torch.bfloat16) for s in ((T, I), (O, I), (I, O)))
    names = kernels_of(lambda: api.nm_linear_forward(x, w)) + kernels_of(lambda: api.nm_linear_input_grad(x, v))
    assert any("dense_gemm_kernel<2, 4, 2, 1, false, 4>" in k for k in names) and any("dense_gemm_kernel<2, 4, 2, 1, true, 4>" in k for k in names)


@pytest.mark.parametrize("T,O,I,kernel", SEVERAL_FORWARD)
def test_linear_forward_of_several_tiles_to_a_workgroup(T, O, I, kernel):
    from paper_2203_10991_amd import api
    test_linear_forward(T, O, I)
    x, w = torch.zeros(T, I, device=DEV, dtype=torch.bfloat16), torch.zeros(O, I, device=DEV, dtype=torch.bfloat16)
    assert any(f"dense_gemm_kernel<{kernel}>" in k for k in kernels_of(lambda: api.nm_linear_forward(x, w)))


@pytest.mark.parametrize("T,O,I,kernel", SEVERAL_GRAD)
def test_linear_input_grad_of_several_tiles_to_a_workgroup(T, O, I, kernel):
    from paper_2203_10991_amd import api
    test_linear_input_grad(T, O, I)
    g, w = torch.zeros(T, O, device=DEV, dtype=torch.bfloat16), torch.zeros(O, I, device=DEV, dtype=torch.bfloat16)
    assert any(f"dense_gemm_kernel<{kernel}>" in k for k in kernels_of(lambda: api.nm_linear_input_grad(g, w)))


@pytest.mark.parametrize("T,O,I", SHAPES)
def test_linear_forward(T, O, I):
    from paper_2203_10991_amd import api
    torch.manual_seed(T + O)
    x, w, b = (torch.randn(*s, device=DEV).to(torch.bfloat16) for s in ((T, I), (O, I), (O,)))
    xn = _behind_nan(x, I + 8)
    _check(api.nm_linear_forward(xn, w), x, w.t())
    _check(api.nm_linear_forward(xn, w, b), x, w.t(), b)
    _check(api.nm_linear_forward(xn, w, b, relu=True), x, w.t(), b, relu=True)


@pytest.mark.parametrize("T,O,I", SHAPES + [(2047, 72, 1032), (1579, 200, 3080), (5000, 264, 2056)])
def test_linear_input_grad(T, O, I):
    from paper_2203_10991_amd import api
    torch.manual_seed(T + I)
    g, w = torch.randn(T, O, device=DEV).to(torch.bfloat16), torch.randn(O, I, device=DEV).to(torch.bfloat16)
    _check(api.nm_linear_input_grad(_behind_nan(g, O + 16), w), g, w)


def test_special_values_stay_where_they_are():
    """an infinity or NaN of x reaches its token's row only, the ReLU keeps a NaN and has no negative zero; the reduction axis ends inside a stage"""
    from paper_2203_10991_amd import api
    torch.manual_seed(1)
    x, w = torch.randn(100, 200, device=DEV).to(torch.bfloat16), torch.rand(72, 200, device=DEV).to(torch.bfloat16) + 0.5
    clean = api.nm_linear_forward(x, w, relu=True)
    x[7, 199], x[40, 3], x[41, 0] = float("nan"), float("inf"), float("-inf")
    y = api.nm_linear_forward(x, w, relu=True)
    assert bool(y[7].isnan().all()) and bool((y[40] == float("inf")).all()) and bool((y[41] == 0).all())
    rest = [r for r in range(100) if r not in (7, 40, 41)]
    assert torch.equal(y[rest], clean[rest]) and not bool(torch.signbit(clean).any())


@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("shape", [(50, 72), (3, 17, 72)])
def test_layers_agree_with_the_framework_products(monkeypatch, relu, shape):
    from paper_2203_10991_amd import api, autograd as ag
    torch.manual_seed(2)
    layer = (ag.NMLinearReLU if relu else ag.NMLinear)(72, 136, cfg=ag.NMConfig(seed=3), device=DEV, dtype=torch.bfloat16)
    x = torch.randn(*shape, device=DEV).to(torch.bfloat16).requires_grad_()
    gy = torch.randn(*shape[:-1], 136, device=DEV).to(torch.bfloat16)
    taken = []
    for name in ("own_linear_forward", "own_linear_input_grad"):
        own = getattr(api, name)
        monkeypatch.setattr(api, name, lambda *a, own=own: (taken.append(own(*a)), taken[-1])[1])
    y = layer(x)
    got = (y,) + torch.autograd.grad(y, (x, layer.weight, layer.bias), gy)
    assert len(taken) == 2 and all(t is not None for t in taken)
    for name in ("own_linear_forward", "own_linear_input_grad"):
        monkeypatch.setattr(api, name, lambda *a: None)
    y = layer(x)
    want = (y,) + torch.autograd.grad(y, (x, layer.weight, layer.bias), gy)
    for a, b in zip(got, want):
        a, b = a.detach(), b.detach()
        assert a.shape == b.shape and a.dtype == b.dtype
        # either side rounds the same sum once: a unit in the last place of bf16 apart
        assert float((a.double() - b.double()).norm()) <= 4e-3 * float(b.double().norm())


def test_what_stays_the_framework_s():
    """autocast regions, operators that are watched, gradients of gradients, views the kernels cannot read, other types, sizes the other library is
    faster at"""
    from paper_2203_10991_amd import api, autograd as ag
    from torch.utils._python_dispatch import TorchDispatchMode
    torch.manual_seed(3)
    w = torch.randn(64, 48, device=DEV).to(torch.bfloat16)
    x = torch.randn(32, 48, device=DEV).to(torch.bfloat16)
    assert api.own_linear_forward(x, w) is not None and api.own_linear_forward(x.view(4, 8, 48), w).shape == (4, 8, 64)
    flat = torch.randn(32 * 48 + 8, device=DEV).to(torch.bfloat16)
    for a in (x.float(), flat[1:1 + 32 * 48].view(32, 48), torch.randn(48, 32, device=DEV).to(torch.bfloat16).t(), x[:0], x[0], x.cpu(), x[:, :40]):
        assert api.own_linear_forward(a, w) is None
    assert api.own_linear_forward(x, w.t().contiguous().t()) is None and api.own_linear_forward(x, w, torch.zeros(64, device=DEV)) is None
    assert api.own_linear_forward(torch.empty(65536, 512, dtype=torch.bfloat16, device=DEV), torch.empty(1024, 512, dtype=torch.bfloat16, device=DEV)) is None
    with torch.autocast("cuda", dtype=torch.float16):
        assert api.own_linear_forward(x, w) is None

    class Watch(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))
    with Watch():
        assert api.own_linear_forward(x, w) is None
    with torch.no_grad():
        assert api.own_linear_input_grad(torch.randn(32, 64, device=DEV).to(torch.bfloat16), w) is not None
    layer = ag.NMLinear(48, 64, bias=False, device=DEV, dtype=torch.bfloat16)
    x.requires_grad_()
    gy = torch.randn(32, 64, device=DEV).to(torch.bfloat16).requires_grad_()
    (dx,) = torch.autograd.grad(layer(x), (x,), gy, create_graph=True)
    (ggy,) = torch.autograd.grad(dx, (gy,), torch.ones_like(dx))
    assert torch.allclose(ggy.float(), torch.ones(32, 48, device=DEV) @ layer.weight.detach().float().t(), rtol=2e-2, atol=1e-2)


def test_the_calls_in_cpp_give_what_the_python_ones_give(monkeypatch):
    """prune, update GEMM and the layer's update through csrc/nm_torch.cpp and without it: same outputs, same exceptions"""
    from paper_2203_10991_amd import api
    torch.manual_seed(4)
    forms = []
    for dt in (torch.bfloat16, torch.float32):
        g, h = (torch.randn(64, n, device=DEV).to(dt) for n in (48, 40))
        wide = torch.randn(64, 56, device=DEV).to(dt)[:, :48]
        for a in (g, wide):
            forms += [lambda a=a: api.mvue_prune_2of4(a, seed=-3, stream_id=2, mode=1), lambda a=a: api.mvue_prune_1of2(a, seed=2 ** 64 + 5)]
        v, m, _ = api.mvue_prune_2of4(g, seed=1)
        forms += [lambda v=v, m=m, h=h: api.nm_update_gemm(v, m, h), lambda v=v, m=m, h=h: api.nm_update_gemm(v, m, h, f32_as_bf16x3=True),
                  lambda v=v, m=m, h=h: api.nm_update_gemm(v, m, h[:48]), lambda v=v, m=m, h=h: api.nm_update_gemm(v, m, h.double()),
                  lambda g=g: api.mvue_prune_2of4(g[:10]), lambda g=g: api.mvue_prune_2of4(g.t()), lambda g=g: api.mvue_prune_2of4(g.half()),
                  lambda g=g: api.mvue_prune_2of4(g.cpu()), lambda g=g: api.mvue_prune_2of4(g, mode=7)]
    g, h = (torch.randn(50, n, device=DEV).to(torch.bfloat16) for n in (48, 32))
    for q8 in (False, True):
        forms += [lambda q8=q8: api.nm_linear_update(g, h, q8=q8, seed=3, bias=True), lambda q8=q8: api.nm_linear_update(g, h, nm="1:2", q8=q8, seed=3),
                  lambda q8=q8: api.nm_linear_update(g, h, q8=q8, act=torch.relu(g)), lambda q8=q8: api.nm_linear_update(g[:, 1:9], h, q8=q8)]
    forms += [lambda: api.nm_linear_update(g, h[:40]), lambda: api.nm_linear_update(g.float(), h)]

    def outcome(f):
        try:
            return f()
        except Exception as e:
            return type(e), str(e)
    native = [outcome(f) for f in forms]

    class Absent:
        def __getattr__(self, name):
            return lambda *a: None
    monkeypatch.setattr(api, "_native", Absent())
    for f, a in zip(forms, native):
        b = outcome(f)
        if isinstance(a, torch.Tensor):
            a, b = (a,), (b,)
        assert len(a) == len(b)
        for s, t in zip(a, b):
            assert torch.equal(s, t) if isinstance(s, torch.Tensor) else s == t


@pytest.mark.parametrize("relu", [False, True])
def test_batches_of_gradients_through_a_layer_that_is_not_trained(relu):
    """torch.autograd.grad(..., is_grads_batched=True): the gradient that reaches the layer has no storage of its own"""
    from paper_2203_10991_amd import autograd as ag
    torch.manual_seed(6)
    layer = (ag.NMLinearReLU if relu else ag.NMLinear)(48, 64, bias=False, device=DEV, dtype=torch.bfloat16).requires_grad_(False)
    x = torch.randn(32, 48, device=DEV).to(torch.bfloat16).requires_grad_()
    g = torch.randn(5, 32, 64, device=DEV).to(torch.bfloat16)
    y = layer(x)
    (got,) = torch.autograd.grad(y, (x,), g, is_grads_batched=True)
    for k in range(5):
        want = (g[k].double() * (y > 0) if relu else g[k].double()) @ layer.weight.double()
        assert float((got[k].double() - want).norm()) <= 4e-3 * float(want.norm())


def test_a_function_mode_sees_the_layers_product():
    from paper_2203_10991_amd import autograd as ag
    from torch.overrides import TorchFunctionMode
    seen = []

    class Watch(TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            seen.append(func)
            return func(*args, **(kwargs or {}))
    layer = ag.NMLinear(48, 64, device=DEV, dtype=torch.bfloat16)
    with Watch():
        layer(torch.randn(32, 48, device=DEV).to(torch.bfloat16))
    assert torch.nn.functional.linear in seen


def test_a_step_that_has_run_once_can_be_captured():
    """in a fresh process: whatever the step uses has been made by then, other libraries' handles too"""
    import os
    import subprocess
    import sys
    code = """
import torch
from paper_2203_10991_amd import autograd as ag
layer = ag.NMLinear(72, 136, cfg=ag.NMConfig(seed=3), device='cuda:0', dtype=torch.bfloat16)
x, gy = (torch.randn(50, n, device='cuda:0').to(torch.bfloat16) for n in (72, 136))
x.requires_grad_()
def step():
    y = layer(x)
    return (y,) + torch.autograd.grad(y, (x, layer.weight, layer.bias), gy)
side = torch.cuda.Stream()
with torch.cuda.stream(side):
    want = step()
torch.cuda.synchronize()
graph = torch.cuda.CUDAGraph()
with torch.cuda.graph(graph, stream=side):
    got = step()
for _ in range(3):
    graph.replay()
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(got, want))
print('replayed')
"""
    r = subprocess.run([sys.executable, "-c", code], cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))), capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "replayed" in r.stdout, r.stdout + r.stderr


def test_reductions_too_long_for_their_tiles_are_the_framework_s():
    """either side of 2048 steps, and of 3584 with 128 tiles of 64 x 64"""
    from paper_2203_10991_amd import api

    def taken(T, O, I):
        x, w, g = (torch.empty(*s, device=DEV, dtype=torch.bfloat16) for s in ((T, I), (O, I), (T, O)))
        with torch.no_grad():
            return api.own_linear_forward(x, w) is not None, api.own_linear_forward(x, w, relu=True) is not None, api.own_linear_input_grad(g, w) is not None
    assert taken(64, 64, 2048) == (True, True, True) and taken(64, 64, 2056) == (False, False, True) and taken(64, 2056, 64) == (True, True, False)
    assert taken(65, 64 * 64, 3584) == (True, True, False) and taken(64, 127 * 64, 3584) == (False, False, False)
    assert taken(65, 3584, 64 * 64) == (False, False, True) and taken(64, 128 * 64, 3592) == (False, False, False)
    assert taken(8, 64, 262144) == (False, False, True)


def test_large_products_the_other_library_is_faster_at():
    """beyond 5e9 multiply-adds: reductions beyond 3072, and from 1024 on 257 to 384 tiles of 128 x 128"""
    from paper_2203_10991_amd import api

    def taken(T, O, I):
        x, w = (torch.empty(*s, device=DEV, dtype=torch.bfloat16) for s in ((T, I), (O, I)))
        return api.own_linear_forward(x, w) is not None
    assert taken(2048, 1024, 3072) and not taken(2048, 1024, 3080) and taken(1024, 1024, 3080)
    assert taken(4096, 1024, 2048) and not taken(4097, 1024, 2048) and taken(5 * 1280, 1024, 1016) and not taken(48 * 128, 1024, 1024) and taken(49 * 128, 1024, 1024)
