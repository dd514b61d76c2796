"""The planner's segmentation without a hint (host only): whole chunks, at most
16 segments, no empty segment, aggregates that outgrow the static scratch only
where a single segment per sequence already does, and the reset pair's choices
beside measured times."""

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


@pytest.mark.parametrize("dtype", [gl.BF16, gl.F32])
@pytest.mark.parametrize("d,m", [(64, 64), (64, 128), (128, 128)])
@pytest.mark.parametrize("BH", [1, 8, 33, 257, 4096])
def test_workspace_of_every_plan(dtype, d, m, BH):
    """Saved, gated and gated saved plans: aggregates of parallel segments within
    the scratch each, chunk-start states and a single segment's sums beside them."""
    for T in (64, 1000, 8192, 60000):
        s = gl.make_shape(B=BH, H=1, T=T, d_in=d, d_out=m, dtype=dtype)
        md, gates, slack = BH * d * m * 4, BH * 16 * 4, 8 * 256
        agg = max(gl.STATIC_SCRATCH_BYTES, 3 * md)  # A, B per segment and one sum per sequence
        saved, ws = gl.saved_bytes(s)
        assert ws <= agg + slack and saved <= agg
        states = md * ((T + 31) // 32)  # 32- or 64-token tiles
        gated_saved, gated_ws = gl.gated_saved_bytes(s)
        assert gated_saved <= states and gated_ws <= 1.5 * agg + gates + slack
        assert gl.gated_workspace_bytes(s) <= 1.5 * agg + states + gates + slack


# Forward + backward of the bf16 reset pair, us by segments per sequence (64 x 64,
# scalar eta, documents of mean length 200), measured on an MI355X.
RESET_US = {
    (1, 2000): {4: 107, 5: 94, 6: 89, 8: 71, 11: 62, 16: 54},
    (8, 2000): {4: 108, 5: 96, 6: 90, 8: 73, 11: 64, 16: 57},
    (16, 2000): {4: 110, 5: 97, 6: 91, 8: 75, 11: 66, 16: 63},
    (24, 4000): {4: 184, 5: 165, 6: 144, 8: 119, 11: 104, 16: 102},
    (40, 2000): {4: 114, 5: 107, 6: 99, 8: 94, 11: 91, 16: 103},
    (40, 4000): {4: 191, 5: 162, 6: 147, 8: 147, 11: 126, 16: 143},
    (64, 1000): {2: 116, 3: 97, 4: 81, 6: 89, 8: 79, 16: 111},
    (128, 2000): {2: 196, 3: 186, 4: 160, 5: 193, 6: 196, 8: 179, 11: 201, 16: 221},
}


@pytest.mark.parametrize("BH,T", sorted(RESET_US))
def test_reset_pair_segments(BH, T):
    """The backward's count, from the saved buffer's size: segment-end weights and chunk-start states."""
    saved, _ = gl.reset_saved_bytes(gl.make_shape(B=BH, H=1, T=T, d_in=64, d_out=64, dtype=gl.BF16))
    n = saved // (BH * 64 * 64 * 4) - (T + 63) // 64
    us = RESET_US[BH, T]
    assert us.get(n, 1e9) <= 1.05 * min(us.values()), (n, us)
