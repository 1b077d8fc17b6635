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


def _depthwise(rt, e, N=2, Ch=32, H=6, W=6, k=3, nhwc=0, x=1 << 40, y=1 << 44):
    rt.lib.pipe_forward_depthwise2d.argtypes = ([C.c_void_p] * 2 + [C.c_int] * 9 + [C.c_float, C.c_void_p, C.c_int, C.c_void_p, C.c_int] +
                                                [C.c_void_p] * 2)
    return rt.lib.pipe_forward_depthwise2d(e, x, N, Ch, H, W, k, k, 1, k // 2, nhwc, 0.0, None, 0, None, 1, y, None)


def failed_preparation_starts_over(rt):
    """Whichever allocation of the preparation fails, the call after it builds every table before the layer reads them."""
    for k in (3, 5):
        whole = ["dense_order_kernel"] * 2 + (["pack_columns_kernel"] if k == 3 else [])
        nth, failures = 1, 0
        while True:
            e = rt.expand(32, k * k, 4, 2, 1.0, 16)
            rt.host.host_fail(nth)
            rc = _depthwise(rt, e, k=k)
            rt.host.host_fail(0)
            names = rt.names()
            if rc == 0:
                break
            failures += 1
            assert not any("depthwise" in n for n in names)
            assert _depthwise(rt, e, k=k) == 0
            built = [w for n in rt.names() for w in ("dense_order_kernel", "pack_columns_kernel") if w in n]
            assert built == whole, (k, nth, built)
            assert _depthwise(rt, e, k=k) == 0
            assert not any(w in n for n in rt.names() for w in whole)      # built once
            nth += 1
        assert failures >= (3 if k == 3 else 2)


def capture_builds_nothing(rt):
    """Under capture an unprepared layer is refused before anything is allocated; afterwards it is prepared as if never called."""
    e = rt.expand(32, 9, 4, 2, 1.0, 16)
    rt.host.host_capture(1)
    rt.host.host_fail(0)
    assert _depthwise(rt, e) == ENOTREADY
    assert rt.host.host_mallocs() == 0 and rt.names() == []
    rt.host.host_capture(0)
    assert _depthwise(rt, e) == 0
    assert sum("dense_order_kernel" in n for n in rt.names()) == 2


def wide_layers_quantize_once(rt):
    """Few tokens: the streaming kernel quantizes them itself unless too many of its workgroups would repeat the work."""
    for rows, one_launch in ((65536, True), (65552, False)):     # 1024 and 1025 bins
        e = rt.expand(rows, 64, 8, 1, 1.0, 16)
        assert _linear(rt, e, 2) == 0
        assert not any("quantize_small" in n for n in rt.names()) == one_launch
        assert _linear(rt, e, 1) == 0                              # a single token: always
        assert not any("quantize_small" in n for n in rt.names())


def any_number_of_images_is_served(rt):
    """Many small maps: more images than a launch of one workgroup each can hold, and numbers where two steps are quicker."""
    e = {c: rt.expand(c, 9, 4, 2, 1.0, 16) for c in (16, 32, 64)}

    def fused(C, N, H, nhwc, x=1 << 40):
        assert _depthwise(rt, e[C], N=N, Ch=C, H=H, W=H, nhwc=nhwc, x=x) == 0, (C, N, H, nhwc)
        names = rt.names()
        one = any("depthwise3_kernel" in n for n in names)
        assert one != any("depthwise_kernel" in n for n in names)
        return one

    assert not fused(16, 1 << 24, 1, 1)      # more workgroups than a launch can hold
    assert not fused(16, 1 << 22, 7, 1)
    assert not fused(16, 100000, 1, 0)       # (channels first: more images than a grid has rows)
    assert not fused(64, 65536, 1, 1)        # few outputs a workgroup
    assert not fused(16, 5349, 7, 0)
    assert not fused(32, 14563, 3, 0)
    assert fused(16, 100, 1, 1)              # few workgroups: one launch less
    for nhwc in (0, 1):
        assert fused(64, 512, 28, nhwc)
        assert fused(32, 600, 28, nhwc, x=(1 << 40) + 4)


@pytest.mark.parametrize("scenario", ["failed_allocation_is_reported_once", "control_words_start_at_zero",
                                      "failed_preparation_starts_over", "capture_builds_nothing",
                                      "any_number_of_images_is_served", "wide_layers_quantize_once"])
def test_host(scenario, tmp_path):
    _host_hip.run(__file__, scenario, tmp_path)


if __name__ == "__main__":
    globals()[sys.argv[1]](_host_hip.Runtime(sys.argv[2]))
