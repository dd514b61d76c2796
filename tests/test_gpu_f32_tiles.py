"""fp32 64 x 64 backward: 32-token tiles by default, 64 on the hint, against the
oracle at the edges of both, for the plain calls and the saved pair."""

import pytest

from parity_util import check, log, to_host
from test_gpu_parity import KEYS, oracle_all, small_inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2609_34174_amd as gl  # noqa: E402
from parity_util import to_dev  # noqa: E402


@pytest.mark.parametrize("prefix", ["exclusive", "inclusive"])
@pytest.mark.parametrize("chunk,tile", [(0, 32), (64, 64)])
@pytest.mark.parametrize("T,segment", [(31, 0), (33, 0), (64, 0), (65, 64), (191, 64)])
def test_f32_backward_tiles(T, segment, chunk, tile, prefix):
    log(f"f32 tiles T={T} segment={segment} chunk={chunk} {prefix}")
    s = gl.make_shape(B=1, H=3, T=T, d_in=64, d_out=64, dtype=gl.F32, prefix=prefix, chunk=chunk, segment=segment)
    assert gl.plan(s).bwd_chunk == tile
    inp = small_inputs(1, 3, T, 64, 64, "f32", seed=T, eta_kind="token")
    W0, X, G, dY, eta = (to_dev(inp[k], "f32", torch) for k in ("W0", "X", "G", "dY", "eta"))
    kw = dict(prefix=prefix, chunk=chunk, segment=segment)
    y = gl.scan_fwd(W0, X, G, eta, **kw)
    plain = gl.scan_bwd(W0, X, G, dY, eta, **kw)
    ys, saved = gl.scan_fwd_save(W0, X, G, eta, **kw)
    pair = gl.scan_bwd_saved(W0, X, G, dY, saved, eta, **kw)
    ref = oracle_all(inp, prefix)
    for k in KEYS:
        check(k, to_host(y if k == "y" else plain[k]), ref[k], "f32")
        check(k, to_host(ys if k == "y" else pair[k]), ref[k], "f32")
