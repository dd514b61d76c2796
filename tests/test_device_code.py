"""What the compiler made of the kernels, where a change of source has lost it before (host only)."""

import os

import pytest

import device_code
import paper_2609_34174_amd as gl

pytestmark = pytest.mark.skipif(not os.path.exists(gl.LIB_PATH) or not all(map(device_code.tool, (
    "llvm-readelf", "llvm-objdump", "c++filt"))), reason="needs the built library and LLVM's tools")


def serial_loads(code):
    """Longest run of 16-byte loads that are each waited for before the next is issued."""
    run = best = 0
    last = None
    for line in code:
        if line.startswith("global_load_dwordx4"):
            if last == "load":
                run = 0
            last = "load"
        elif line.startswith("s_waitcnt") and "vmcnt(0)" in line:
            if last == "load":
                run += 1
                best = max(best, run)
            last = "wait"
    return best


@pytest.mark.parametrize("kernel", ["fwd_main_kernel", "bwd_main_kernel", "bwd_split_kernel"])
def test_segment_sums_keep_their_loads_in_flight(kernel):
    """The prologues sum up to 16 segments' aggregates: a wait per load is most of a short segment's time."""
    found = {k: serial_loads(v) for k, v in device_code.listing().items() if k.startswith(kernel + "<")}
    assert found
    assert {k: n for k, n in found.items() if n >= 4} == {}


@pytest.mark.parametrize("kernel", ["agg_kernel<OpF32", "fwd_main_kernel<OpF32, 128, 128", "wide_"])
def test_streaming_kernels_do_not_spill(kernel):
    """fp32 tiles take twice bf16's registers: a second set of them, or a second
    buffer's addresses, has spilled up to 67 registers in these loops."""
    found = {k: n for k, n in device_code.spills().items() if k.startswith(kernel)}
    assert found
    assert {k: n for k, n in found.items() if n > 4} == {}
