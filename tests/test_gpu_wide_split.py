"""Wide backward with split score contractions: the gate gradients take dY G^T
from the read's finish and X X^T from the split's partials, whichever other
outputs are asked for.  Widths with one and with both contractions split."""

import numpy as np
import pytest

from oracle import gradlev_oracle as orc
from parity_util import check, log, to_host
from test_gpu_wide import WIDE_BWD, dev_inputs, inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2609_34174_amd as gl  # noqa: E402


@pytest.mark.parametrize("dtype,d,m", [("bf16", 512, 1024), ("bf16", 256, 1024), ("f32", 1024, 256)])
def test_wide_split_gate_gradients(dtype, d, m):
    log(f"wide split dtype={dtype} d={d} m={m}")
    inp = inputs(1, 1, 193, d, m, dtype, seed=6, alpha_kind="family", eta_kind="token", with_reset=True)
    W0, X, G, dY, e, a, r = dev_inputs(inp, dtype)
    full = {k: to_host(v) for k, v in gl.scan_bwd_gated(W0, X, G, dY, e, a, r, outputs=WIDE_BWD).items()}
    ref = orc.scan_bwd(inp["W0"], inp["X"], inp["G"], inp["eta"], inp["dY"], alpha=inp["alpha"], reset=inp["reset"])
    for k in WIDE_BWD:
        check(k, full[k], ref[k], dtype)
    for subset in (("deta",), ("dalpha",), ("deta", "dg"), ("gtilde", "deta"), ("dx", "dg", "dalpha")):
        log(f"  subset {subset}")
        part = gl.scan_bwd_gated(W0, X, G, dY, e, a, r, outputs=subset)
        for k in subset:
            np.testing.assert_array_equal(to_host(part[k]), full[k], err_msg=str(subset))


@pytest.mark.parametrize("T", [129, 200])
def test_wide_unread_step_size(T):
    """No token reads the last one's write: its step size may be anything."""
    log(f"wide unread step size T={T}")
    inp = inputs(1, 1, T, 256, 128, "f32", seed=9, alpha_kind="family", eta_kind="token", with_reset=False)
    W0, X, G, dY, e, a, r = dev_inputs(inp, "f32")
    ref = gl.scan_bwd_gated(W0, X, G, dY, e, a, r, outputs=WIDE_BWD)
    e = e.clone()
    e[..., -1] = float("inf")
    got = gl.scan_bwd_gated(W0, X, G, dY, e, a, r, outputs=WIDE_BWD)
    for k in WIDE_BWD:
        np.testing.assert_array_equal(to_host(got[k]), to_host(ref[k]), err_msg=k)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T", [1, 129, 300])
@pytest.mark.parametrize("alpha_kind,with_reset", [("1", False), ("1", True), ("signed", True)])
def test_wide_deta_alone(dtype, T, alpha_kind, with_reset):
    """Without a read: one workgroup per tile contracts both products (narrow maps)."""
    log(f"wide deta alone dtype={dtype} T={T} alpha={alpha_kind} reset={with_reset}")
    inp = inputs(2, 2, T, 128, 256, dtype, seed=T, alpha_kind=alpha_kind, eta_kind="token", with_reset=with_reset)
    W0, X, G, dY, e, a, r = dev_inputs(inp, dtype)
    ref = orc.scan_bwd(inp["W0"], inp["X"], inp["G"], inp["eta"], inp["dY"], alpha=inp["alpha"], reset=inp["reset"])
    got = {k: gl.scan_bwd_gated(W0, X, G, dY, e, a, r, outputs=o) for k, o in (("deta", ("deta",)), ("dg", ("deta", "dg")))}
    check("deta", to_host(got["deta"]["deta"]), ref["deta"], dtype)
    check("dg", to_host(got["dg"]["dg"]), ref["dg"], dtype)
    np.testing.assert_array_equal(to_host(got["dg"]["deta"]), to_host(got["deta"]["deta"]))
    e = e.clone()
    e[..., -1] = float("inf")  # no token reads the last one's write
    again = gl.scan_bwd_gated(W0, X, G, dY, e, a, r, outputs=("deta",))["deta"]
    np.testing.assert_array_equal(to_host(again), to_host(got["deta"]["deta"]))
