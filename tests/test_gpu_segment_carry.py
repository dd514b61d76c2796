"""GPU parity of the scans over segment counts: the carry into a segment sums
the others' aggregates in batches of four or two, so the counts cover none,
less than a batch, whole batches and remainders up to the limit of 16 segments."""

import pytest

from parity_util import check, log
from test_gpu_gated import KEYS, inputs, oracle_all, run_gpu
import test_gpu_parity as unit

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


@pytest.mark.parametrize("d,m,dtype", [(64, 64, "bf16"), (64, 128, "bf16"), (128, 64, "f32"), (128, 128, "bf16")])
@pytest.mark.parametrize("nseg", [1, 2, 3, 4, 5, 7, 16])
def test_unit_carry(d, m, dtype, nseg):
    T = 64 * nseg - 13
    log(f"unit carry {d}x{m} dtype={dtype} nseg={nseg} T={T}")
    inp = unit.small_inputs(1, 2, T, d, m, dtype, seed=70 + nseg, eta_kind="scalar")
    out = unit.run_gpu(inp, dtype, "exclusive", segment=64)
    ref = unit.oracle_all(inp, "exclusive")
    for k in unit.KEYS:
        check(k, out[k], ref[k], dtype)
