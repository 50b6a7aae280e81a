"""nm_conv_update (one call: padded grid, prune, update GEMM on shifted views, weight layout) against the oracle on the
materialised grid, at the edges of its tiles: 256 grid rows, 64 channels, image widths that no vector load divides, both tensor
layouts, 16- and 32-token groups, few and many split-K slabs."""
import numpy as np
import pytest
import torch

from paper_2203_10991_amd import synth
from gpu_util import DEV

pytestmark = pytest.mark.gpu


def _grid(t, pad):
    """bf16 bits of the zero-padded channels-last grid of a [N, C, H, W] tensor, flattened to rows"""
    a = t.contiguous().view(torch.int16).cpu().numpy().view(np.uint16).transpose(0, 2, 3, 1)
    return np.pad(a, ((0, 0), (pad, pad), (pad, pad), (0, 0))).reshape(-1, t.shape[1])


@pytest.mark.parametrize("N,C,O,H,W,k", [(1, 16, 8, 5, 3, 3),          # less than a tile of rows, 8 output channels
                                         (2, 16, 72, 7, 7, 3),         # channels past a 64-channel tile
                                         (1, 80, 64, 14, 14, 3),       # exactly one 256-row tile of grid rows
                                         (3, 64, 136, 9, 11, 5),       # 25 taps, odd width
                                         (4, 32, 24, 8, 8, 1),         # no padding
                                         (4, 32, 64, 5, 3, 3),         # the nine-tap kernel: 32 channels, a grid smaller than its ring
                                         (3, 96, 48, 9, 13, 3),        # ... three blocks of 32 channels, output channels short of a tile
                                         (2, 128, 200, 7, 90, 3),      # ... the widest image its ring takes (bf16), a ragged second tile
                                         (2, 64, 64, 3, 96, 3),        # ... an image too wide for it (bf16)
                                         (24, 64, 64, 28, 28, 3)])     # many split-K slabs
@pytest.mark.parametrize("q8", [False, True])
@pytest.mark.parametrize("layouts", [(False, False), (True, True), (True, False)])
def test_conv_update_matches_the_oracle(oracle, N, C, O, H, W, k, q8, layouts):
    import paper_2203_10991_amd as nm
    from paper_2203_10991_amd import api
    torch.manual_seed(N + C + O)
    fmt = [torch.channels_last if cl else torch.contiguous_format for cl in layouts]
    gy = (torch.randn(N, O, H, W, device=DEV) * torch.exp(2 * torch.randn(N, O, H, W, device=DEV))).to(torch.bfloat16).contiguous(memory_format=fmt[0])
    x = torch.relu(torch.randn(N, C, H, W, device=DEV)).to(torch.bfloat16).contiguous(memory_format=fmt[1])
    dW = api.nm_conv_update(gy, x, k, q8=q8, seed=11, stream_id=2)
    pad, wp, gt = k // 2, W + 2 * (k // 2), 32 if q8 else 16
    gg, xg = _grid(gy, pad), _grid(x, pad)
    rows = gg.shape[0]
    T, margin = (rows + gt - 1) // gt * gt, pad * wp + pad
    g2 = np.zeros((T, O), dtype=np.uint16); g2[:rows] = gg
    xf = np.zeros((T + 2 * margin, C), dtype=np.uint16); xf[margin:margin + rows] = xg
    shifts = [(ky - pad) * wp + (kx - pad) for ky in range(k) for kx in range(k)]
    if q8:
        sg, sh = oracle.pow2_scale(g2, 57344.0 / 4.0), oracle.pow2_scale(xf, 448.0)
        v, m = oracle.prune_2of4_q8(g2, 11, 2, 0, sg)
        want, wabs = oracle.update_gemm_q8_shifted(v, m, oracle.cast_e4m3(xf, sh), margin, shifts, alpha=1.0 / (sg * sh))
        tol = 1e-3                                                     # the 8-bit instruction's product window
    else:
        v, m, _ = oracle.prune_2of4(g2, 11, 2)
        want, wabs = oracle.update_gemm_shifted(v, m, xf, margin, shifts)
        tol = 1e-5                                                     # binary32 accumulation
    want, wabs = (a.reshape(O, k, k, C).transpose(0, 3, 1, 2) for a in (want, wabs))
    got = dW.double().cpu().numpy()
    # + half a unit in the last place of the bf16 result
    assert (np.abs(got - want) <= tol * wabs + 2.0 ** -8 * np.abs(want) + 1e-30).all()
    assert np.linalg.norm(got - want) <= 3e-3 * np.linalg.norm(want)   # (a wrong mask in one group would show here)


def test_conv_update_agrees_with_the_separate_calls_at_a_layer_size():
    """approx-MVUE and the optimal estimator, against the library's own prune and GEMM on a grid made with tensor operations"""
    import paper_2203_10991_amd as nm
    from paper_2203_10991_amd import api
    from paper_2203_10991_amd.autograd import padded_rows
    torch.manual_seed(3)
    N, C, O, S = 8, 64, 128, 28
    gy = (torch.randn(N, O, S, S, device=DEV) * torch.exp(2 * torch.randn(N, O, S, S, device=DEV))).to(torch.bfloat16)
    x = torch.relu(torch.randn(N, C, S, S, device=DEV)).to(torch.bfloat16)
    (xr, wp), (gr, _) = padded_rows(x, 1), padded_rows(gy, 1)
    T, margin = (xr.shape[0] + 15) // 16 * 16, wp + 1
    xf = torch.zeros((T + 2 * margin, C), dtype=x.dtype, device=DEV); xf[margin:margin + xr.shape[0]] = xr
    g2 = torch.zeros((T, O), dtype=x.dtype, device=DEV); g2[:gr.shape[0]] = gr
    for mode in (0, 1):
        v, m, _ = nm.mvue_prune_2of4(g2, seed=5, stream_id=1, mode=mode)
        shifts = [(i - 1) * wp + (j - 1) for i in range(3) for j in range(3)]
        want, wabs = (nm.nm_update_gemm_shifted(t, m, xf, margin, shifts).reshape(O, 3, 3, C).permute(0, 3, 1, 2) for t in (v, v.abs()))
        got = api.nm_conv_update(gy, x, 3, mode=mode, seed=5, stream_id=1)
        # same operands (x >= 0, so the sums over |v| are those of the absolute products), sums in another order: each side is
        # within 1e-5 of them; then half a unit in the last place of the bf16 result
        assert bool(((got.float() - want).abs() <= 2.0 ** -8 * want.abs() + 2e-5 * wabs).all())


def test_views_off_a_16_byte_boundary_are_copied():
    from paper_2203_10991_amd import api
    torch.manual_seed(6)
    gy, x = (torch.randn(2, c, 6, 6, device=DEV).to(torch.bfloat16) for c in (16, 32))

    def shifted(t, fmt):
        flat = torch.empty(t.numel() + 8, dtype=t.dtype, device=DEV)[1:1 + t.numel()]
        n, c, h, w = t.shape
        v = flat.view(n, h, w, c).permute(0, 3, 1, 2) if fmt is torch.channels_last else flat.view(n, c, h, w)
        v.copy_(t)
        assert v.data_ptr() % 16 and v.is_contiguous(memory_format=fmt)
        return v
    want = api.nm_conv_update(gy, x, 3, seed=4)
    for fmt in (torch.contiguous_format, torch.channels_last):
        assert torch.equal(api.nm_conv_update(shifted(gy, fmt), shifted(x, fmt), 3, seed=4), want)


def test_a_binary32_weight_gets_unrounded_sums():
    """autocast: bf16 tensors, binary32 weight -- its gradient keeps the binary32 sums"""
    from paper_2203_10991_amd.autograd import NMConfig, _conv_update_shifted
    torch.manual_seed(7)
    gy, x = (torch.randn(2, c, 6, 6, device=DEV).to(torch.bfloat16) for c in (16, 32))
    a = _conv_update_shifted(gy, x, 3, NMConfig(seed=4), torch.float32)
    b = _conv_update_shifted(gy, x, 3, NMConfig(seed=4), torch.bfloat16)
    assert a.dtype == torch.float32 and b.dtype == torch.bfloat16
    assert torch.equal(a.to(torch.bfloat16), b) and not torch.equal(a.to(torch.bfloat16).float(), a)


@pytest.mark.parametrize("N,C,O,H,W,k", [(1, 16, 8, 5, 3, 3), (2, 16, 72, 7, 7, 3), (1, 80, 64, 14, 14, 3), (3, 64, 136, 9, 11, 5), (4, 32, 24, 8, 8, 1),
                                         (3, 96, 48, 9, 13, 3), (24, 64, 64, 28, 28, 3)])
@pytest.mark.parametrize("q8", [False, True])
@pytest.mark.parametrize("channels_last", [False, True])
def test_conv_update_with_the_approximate_estimator_matches_the_oracle(oracle, N, C, O, H, W, k, q8, channels_last):
    """approx-MVUE: two selection words per block, in the 8-bit form dealt to the two lanes of a pair in another way than the
    optimal estimator's"""
    from paper_2203_10991_amd import api
    torch.manual_seed(N + C + O)
    fmt = torch.channels_last if channels_last else torch.contiguous_format
    gy = (torch.randn(N, O, H, W, device=DEV) * torch.exp(2 * torch.randn(N, O, H, W, device=DEV))).to(torch.bfloat16).contiguous(memory_format=fmt)
    x = torch.relu(torch.randn(N, C, H, W, device=DEV)).to(torch.bfloat16).contiguous(memory_format=fmt)
    got = api.nm_conv_update(gy, x, k, q8=q8, mode=1, seed=17, stream_id=3).double().cpu().numpy()
    pad, wp, gt = k // 2, W + 2 * (k // 2), 32 if q8 else 16
    gg, xg = _grid(gy, pad), _grid(x, pad)
    rows, margin = gg.shape[0], pad * wp + pad
    T = (rows + gt - 1) // gt * gt
    g2, xf = np.pad(gg, ((0, T - rows), (0, 0))), np.pad(xg, ((margin, margin + T - rows), (0, 0)))
    shifts = [(ky - pad) * wp + (kx - pad) for ky in range(k) for kx in range(k)]
    if q8:
        sg, sh = oracle.pow2_scale(g2, 57344.0 / 4.0), oracle.pow2_scale(xf, 448.0)
        v, m = oracle.prune_2of4_q8(g2, 17, 3, 1, sg)
        want, wabs = oracle.update_gemm_q8_shifted(v, m, oracle.cast_e4m3(xf, sh), margin, shifts, alpha=1.0 / (sg * sh))
    else:
        v, m, _ = oracle.prune_2of4_approx(g2, 17, 3)
        want, wabs = oracle.update_gemm_shifted(v, m, xf, margin, shifts)
    want, wabs = (a.reshape(O, k, k, C).transpose(0, 3, 1, 2) for a in (want, wabs))
    # the sums' tolerances as above, half a unit in the last place of the bf16 result, a wrong mask in one group
    assert (np.abs(got - want) <= (1e-3 if q8 else 1e-5) * wabs + 2.0 ** -8 * np.abs(want) + 1e-30).all()
    assert np.linalg.norm(got - want) <= 3e-3 * np.linalg.norm(want)


@pytest.mark.parametrize("N,C,O,H,W,k", [(2, 16, 8, 5, 1, 3),          # images one pixel wide: no pixel pairs
                                         (2, 24, 16, 1, 1, 3),
                                         (3, 16, 24, 5, 3, 1),         # no border and an odd number of pixels: pairs would straddle images
                                         (3, 48, 40, 7, 5, 1),         # ... with 32 channels in flight
                                         (5, 16, 24, 3, 2, 1),         # ... an even number, the grid's end inside a tile
                                         (2, 40, 72, 4, 2, 3),         # every pair of an image row is border beside a pixel
                                         (1, 48, 40, 65, 3, 5)])       # pairs that start on the row's last pixel, odd and even rows in turn
@pytest.mark.parametrize("q8", [False, True])
def test_conv_update_pixel_pairs_at_the_edges(oracle, N, C, O, H, W, k, q8):
    if q8 and C % 16:
        C += 8
    test_conv_update_matches_the_oracle(oracle, N, C, O, H, W, k, q8, (False, False))


@pytest.mark.parametrize("N,C,O,H,W,k,form", [(16, 144, 144, 14, 14, 3, "1, 1, 64, 256"),          # up to eleven slabs
                                              (12, 48, 24, 28, 28, 3, "8, 1, 32, 576"),            # up to 63: a thread to a chain
                                              (40, 272, 272, 14, 14, 1, "1, 8, 64, 256"),          # ... large: a thread to a sum
                                              (24, 48, 376, 28, 28, 3, "1, 8, 64, 256"),
                                              (32, 48, 24, 28, 28, 3, "16, 1, 16, 576"),           # 64 and more
                                              (128, 128, 512, 56, 56, 1, "1, 16, 64, 256")])       # ... large
def test_conv_update_second_pass_forms(N, C, O, H, W, k, form):
    """against the same sums by separate calls, unrounded: what is left is the rounding to bf16, 2^-9 of a value at most"""
    from gpu_util import kernels_of
    from paper_2203_10991_amd import api, autograd as ag
    torch.manual_seed(C)
    x, gy = torch.randn(N, C, H, W, device=DEV).to(torch.bfloat16), torch.randn(N, O, H, W, device=DEV).to(torch.bfloat16)
    got = api.nm_conv_update(gy, x, k, seed=3).double()
    want = ag._conv_update_shifted(gy, x, k, ag.NMConfig(seed=3), torch.float32).double()
    assert float((got - want).norm()) <= 2.0 ** -9 * float(want.norm()) * 1.01
    assert any(f"finish_conv_kernel<{form}>" in name for name in kernels_of(lambda: api.nm_conv_update(gy, x, k, seed=3)))
