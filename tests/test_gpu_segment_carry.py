"""GPU parity of the gated scans over segment counts: the carry into a segment
sums the others' aggregates in batches of four (64-wide) or two (128-wide), so
the counts cover none, less than a batch, whole batches and remainders up to
the limit of 16 segments."""

import pytest

from parity_util import check, log
from test_gpu_gated import KEYS, inputs, oracle_all, run_gpu

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width,dtype", [(64, "bf16"), (128, "bf16"), (128, "f32")])
@pytest.mark.parametrize("nseg", [1, 2, 4, 5, 6, 16])
def test_gated_carry(width, dtype, nseg):
    T = 64 * nseg - 13
    log(f"gated carry width={width} dtype={dtype} nseg={nseg} T={T}")
    inp = inputs(1, 2, T, width, width, dtype, seed=90 + nseg, alpha_kind="0.99", eta_kind="token", with_reset=False)
    out = run_gpu(inp, dtype, segment=64)
    ref = oracle_all(inp)
    for k in KEYS:
        check(k, out[k], ref[k], dtype)
