"""nm_q8_scale over the shapes at which its launch changes form: one row per workgroup, several workgroups per row, more
rows than workgroups, a contiguous tensor taken as one row, sizes around a workgroup's trip.  The record has to hold the
bit pattern of the maximum wherever in the tensor it sits, with larger values in the padding that a row stride skips."""
import numpy as np
import pytest
import torch

from gpu_util import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("R,C,ld", [(1, 8, 8), (1, 16, 16), (3, 8, 24), (511, 16, 24), (512, 16, 24), (513, 16, 16), (700, 8, 16), (1300, 40, 48),
                                    (2, 8192 * 4 + 8, 8192 * 4 + 16), (7, 8192 * 9, 8192 * 9 + 8), (1, 8 * 8192 * 8 + 8, 8 * 8192 * 8 + 8), (3, 8 * 8192 * 8, 8 * 8192 * 8 + 16), (300, 8192 + 8, 8192 + 16), (4096, 1032, 1032)])
def test_scale_record_over_the_launch_forms(oracle, dtype, R, C, ld):
    import paper_2203_10991_amd as nm
    rng = np.random.default_rng(R * 131 + C)
    wide = torch.full((R, ld), 1e6, dtype=dtype, device=DEV)
    wide[:, :C] = torch.from_numpy(rng.standard_normal((R, C)).astype(np.float32)).to(DEV).to(dtype).clamp(-4, 4)
    spots = [(0, 0), (R - 1, C - 1), (R - 1, 0), (0, C - 1)] + [(int(rng.integers(R)), int(rng.integers(C))) for _ in range(6)]
    for k, (r, c) in enumerate(spots):
        t = wide.clone()
        t[r, c] = -(16.0 + k)                                   # (exact in bf16)
        rec = nm.nm_q8_scale(t[:, :C], 448.0).cpu().numpy()
        s = np.float32(oracle.pow2_scale(np.full((1, 8), -(16.0 + k), dtype=np.float32), 448.0))
        assert rec.view(np.uint32)[2] == np.float32(16.0 + k).view(np.uint32), (r, c)
        assert rec[0] == s and rec[1] == np.float32(1.0) / s and rec.view(np.uint32)[3] == 0


# strided rows of at most 1024 16-byte pieces: several rows to a trip of a workgroup.  Pieces that no power of two divides, the longest
# row (1024 pieces, bf16 8192 and binary32 4096 columns) and one piece more, row counts around whole trips and four trips in flight
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("R,C,ld", [(40001, 24, 40), (2, 8, 24), (65537, 8, 16), (16383, 72, 80), (2100, 4096, 4104), (2100, 8192, 8200), (1030, 4104, 4112),
                                    (1030, 8200, 8208)])
def test_scale_record_of_short_strided_rows(oracle, dtype, R, C, ld):
    test_scale_record_over_the_launch_forms(oracle, dtype, R, C, ld)


def test_short_strided_rows_are_not_walked_one_by_one():
    """a narrow view takes about as long as a contiguous tensor of the same size (a row per trip was 45 times as long)"""
    import paper_2203_10991_amd as nm
    wide = torch.randn(802816, 128, device=DEV).to(torch.bfloat16)
    narrow, packed = wide[:, :64], wide[:, :64].contiguous()

    def least_ms(t):
        best = float("inf")
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            nm.nm_q8_scale(t, 448.0)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        return best
    assert least_ms(narrow) < 6.0 * least_ms(packed)
