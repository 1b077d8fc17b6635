"""The library's host side on a stand-in for the HIP runtime (no GPU): what it allocates, builds and launches, and what a call
leaves behind when one of its allocations fails."""
import ctypes as C
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import _host_hip

ENOTREADY, ENOMEM = -6, -3


def _linear(rt, e, T, split=None, reduce=1):
    rt.lib.pipe_forward.argtypes = [C.c_void_p] * 2 + [C.c_int, C.c_float, C.c_void_p, C.c_int, C.c_void_p, C.c_int] + [C.c_void_p] * 2
    arr = (C.c_int * len(split))(*split) if split else None
    return rt.lib.pipe_forward(e, 1 << 40, T, 0.0, arr, len(split or ()), None, reduce, 1 << 44, None)


def failed_allocation_is_reported_once(rt):
    """A call whose scratch cannot be allocated says so; the next one, for which it can, succeeds."""
    e = rt.expand(64, 64, 4, 2, 1.0, 16)
    rt.host.host_fail(1)
    assert _linear(rt, e, 200) == ENOMEM
    rt.host.host_fail(0)
    assert not any("kernel" in n for n in rt.names())
    assert _linear(rt, e, 200) == 0


def control_words_start_at_zero(rt):
    """The stream's control words (among them the slots that kernels only ever raise) are cleared when they are allocated, also
    by a call that then fails for want of another buffer."""
    e = rt.expand(64, 64, 4, 2, 1.0, 16)
    rt.host.host_fail(1)
    assert _linear(rt, e, 200) == ENOMEM
    rt.host.host_fail(0)
    assert _linear(rt, e, 200) == 0
    assert rt.names().count("hipMemset") == 1


@pytest.mark.parametrize("scenario", ["failed_allocation_is_reported_once", "control_words_start_at_zero"])
def test_host(scenario, tmp_path):
    _host_hip.run(__file__, scenario, tmp_path)


if __name__ == "__main__":
    globals()[sys.argv[1]](_host_hip.Runtime(sys.argv[2]))
