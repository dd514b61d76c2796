"""The planner's segmentation without a hint (host only): whole chunks, at most
16 segments, no empty segment, and aggregates that outgrow the static scratch
only where a single segment per sequence already does."""

import pytest

import paper_2609_34174_amd as gl


@pytest.mark.parametrize("dtype", [gl.BF16, gl.F32])
@pytest.mark.parametrize("d,m", [(64, 64), (64, 128), (128, 64), (128, 128)])
@pytest.mark.parametrize("BH", [1, 7, 8, 33, 128, 257, 4096])
def test_automatic_segments(dtype, d, m, BH):
    for T in (1, 63, 64, 65, 1000, 8192, 100003):
        s = gl.make_shape(B=BH, H=1, T=T, d_in=d, d_out=m, dtype=dtype)
        p = gl.plan(s)
        for C, seg, n in ((p.fwd_chunk, p.fwd_segment, p.fwd_nseg), (p.bwd_chunk, p.bwd_segment, p.bwd_nseg)):
            assert seg % C == 0 and 1 <= n <= 16 and (n - 1) * seg < T <= n * seg
        one = 3 * BH * d * m * 4  # aggregates of one segment per sequence, and dW0's sums
        assert p.workspace_bytes <= max(gl.STATIC_SCRATCH_BYTES, one) + 3 * 256
