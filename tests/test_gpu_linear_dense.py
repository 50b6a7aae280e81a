"""nm_linear_forward and nm_linear_input_grad (the dense products of a linear layer) against binary64 sums of the same bf16 operands, at the
edges of their tiles, of a stage of 64 reduction steps and of a chunk of 8, on views whose padding is NaN."""
import pytest
import torch

from gpu_util import DEV

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
          (2047, 1032, 72),                                                                       # 128 x 64
          (1579, 3080, 200),                                                                       # 128 x 128
          (5000, 2056, 264)]                                                                       # 256 x 256


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
