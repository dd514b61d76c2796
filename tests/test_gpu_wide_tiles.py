"""Wide maps with enough sequences for the 128-wide output tiles (512 of them),
for the anti-causal tiles of grids between and for dW0's long walks, which the
smaller cases leave to narrower tiles and shorter walks.  The oracle takes
sampled sequences (each is an independent problem); dW0, which sums over all,
is dY^T X in float64."""

import numpy as np
import pytest

from oracle import gradlev_oracle as orc
from parity_util import check, log, to_host
from test_gpu_wide import WIDE_BWD, dev_inputs, inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2609_34174_amd as gl  # noqa: E402


# Output tiles are 128 tokens x 128 columns: B * H * 2 * (width / 128) of them here.
@pytest.mark.parametrize("B,H", [
    (8, 16),  # 512: 128-wide tiles; dW0 64 tiles of 24 steps
    (5, 16),  # 320: 64-wide ones, 640 workgroups; dW0 64 tiles of 15 steps
    (4, 8),   # 128: 64-wide ones, 256 workgroups
])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_wide_tiles(dtype, B, H):
    T = 130
    log(f"wide tiles dtype={dtype} B={B} H={H} T={T}")
    inp = inputs(B, H, T, 256, 256, dtype, seed=B + H, alpha_kind="family", eta_kind="token", with_reset=True)
    W0, X, G, dY, e, a, r = dev_inputs(inp, dtype)
    y = gl.scan_fwd_gated(W0, X, G, e, a, r)
    out = gl.scan_bwd_gated(W0, X, G, dY, e, a, r, outputs=WIDE_BWD)
    out = {"y": y, **out}
    x, dy = (np.asarray(inp[k], np.float64) for k in ("X", "dY"))
    check("dw0", to_host(out.pop("dw0")), sum(np.swapaxes(dy[b], 1, 2) @ x[b] for b in range(B)), dtype)
    for b, h in ((0, 0), (1, H - 1), (B - 1, H // 2)):
        at = {k: inp[k][b:b + 1, h:h + 1] for k in ("X", "G", "dY", "eta", "alpha")}
        args, kw = (inp["W0"][h:h + 1], at["X"], at["G"], at["eta"]), dict(alpha=at["alpha"], reset=inp["reset"][b:b + 1])
        ref = {"y": orc.scan_fwd(*args, **kw), **orc.scan_bwd(*args, at["dY"], **kw)}
        for k in out:
            check(k, to_host(out[k])[b:b + 1, h:h + 1], ref[k], dtype)
