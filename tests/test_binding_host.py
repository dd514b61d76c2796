"""Host-side checks of the binding's own argument handling (no GPU, no library call)."""

import pytest

import paper_2609_34174_amd as gl

torch = pytest.importorskip("torch")

DIMS = gl._Dims()
DIMS.B, DIMS.H, DIMS.T, DIMS.d_in, DIMS.d_out = 1, 2, 8, 64, 64


@pytest.mark.parametrize("known", [gl.BWD_OUTPUTS, gl.GATED_OUTPUTS])
def test_supplied_outputs_are_checked_whether_requested_or_not(known):
    """Every known entry of `out` reaches the kernel, which writes it at the full size."""
    for k in known:
        for bad in (torch.empty(1, 2, 8, 64), torch.empty(3), torch.empty(3, dtype=torch.int32)):
            with pytest.raises((TypeError, ValueError)):
                gl._grads(DIMS, (), {k: bad}, known, "cpu")
        with pytest.raises(TypeError):
            gl._grads(DIMS, (k,), {k: None}, known, "cpu")
        assert gl._grads(DIMS, (), {k: None}, known, "cpu") == {k: None}
    assert gl._grads(DIMS, (), {"note": 3}, known, "cpu") == {"note": 3}  # not an output: not passed on
    with pytest.raises(ValueError):
        gl._grads(DIMS, ("note",), None, known, "cpu")


def test_workspace_is_checked():
    with pytest.raises(ValueError):  # host memory
        gl._workspace(64, "cpu", torch.empty(64, dtype=torch.uint8))
    with pytest.raises(ValueError):
        gl._workspace(64, "cpu", torch.empty(63, dtype=torch.uint8))
    with pytest.raises(ValueError, match="too small"):  # 64 elements over one byte of storage
        gl._workspace(64, "cpu", torch.empty(1, dtype=torch.uint8).expand(64))
    assert gl._workspace(0, "cpu", None) == (None, 0)
    ws, n = gl._workspace(64, "cpu", None)
    assert n == ws.numel() == 64
