"""The library's host side on a stand-in for the HIP runtime (no GPU): what it allocates, builds and launches, and what a call
leaves behind when one of its allocations fails."""
import ctypes as C
import os
import re
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import _host_hip

ENOTREADY, EDEVICE, ENOMEM = -6, -4, -3


class Layer(C.Structure):   # pipe_chain_layer
    _fields_ = [("e", C.c_void_p), ("bias", C.c_void_p), ("act", C.c_int), ("skip", C.c_int), ("pre_act", C.c_int), ("conv", C.c_int * 4), ("s_in", C.c_void_p)]


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


def single_pass_tables_hold_no_needless_items(rt):
    """The bins of the single-pass kernel: every order of every row block once, adjacent and ascending; and the items that its tiles
    multiply (four bins, each as many as the fullest) exceed the stored row blocks only where a pair or a row block of three
    orders leaves no other choice -- not by the row blocks that a member pruned."""
    import random
    rng = random.Random(5)
    #         rows  K  kept of the groups, split, gated, items multiplied per stored row block at most
    for rows, K, part, split, gated, most in ((4096, 4, 4, [2, 2], 0, 1.01), (4096, 8, 8, [2, 2, 2, 2], 0, 1.01), (4096, 2, 4, [1, 1], 0, 1.01),
                                              (4096, 3, 1, [3], 0, 1.01), (2048, 4, 2, [4], 0, 1.05), (4096, 8, 4, [3, 3, 2], 0, 1.01),
                                              (4096, 4, 4, [2, 2], 1, 1.2), (4096, 8, 8, [2, 2, 2, 2], 1, 1.35), (48, 4, 3, [1, 3], 0, 9)):
        n_rb = rows // 16
        kept = [sorted(rng.sample(range(n_rb), n_rb // part)) if part > 1 else list(range(n_rb)) for _ in range(K - 1)]
        e = rt.expand(rows, 64, 4, K, 1.0 / part, 16, kept=kept if part > 1 else ())
        rt.copied.clear()
        rt.lib.pipe_prepare.argtypes = [C.c_void_p, C.c_void_p, C.c_int, C.c_int, C.c_void_p]
        rt.lib.pipe_prepare_mlp.argtypes = [C.c_void_p, C.c_void_p, C.c_int, C.c_void_p, C.c_int, C.c_int, C.c_void_p]
        arr = (C.c_int * len(split))(*split)
        if gated:
            l2 = rt.expand(64, rows // 2, 4, K, 1.0, 16)
            rt.copied.clear()
            assert rt.lib.pipe_prepare_mlp(e, l2, 2, arr, len(split), 200, None) == 0
        else:
            assert rt.lib.pipe_prepare(e, arr, len(split), 200, None) == 0
        raw = (C.c_int32 * (len(rt.copied[0]) // 4)).from_buffer_copy(rt.copied[0])
        bins = [raw[i:i + 16] for i in range(0, len(raw), 16)]          # pos, scale pos, row block, {member, ends, ups, live | items << 1}
        orders_of = [[0] + [k + 1 for k in range(K - 1) if part == 1 or rb in kept[k]] for rb in range(n_rb)]
        first = [sum(split[:m]) for m in range(len(split))]
        seen, stored, multiplied = {}, 0, 0
        assert len(bins) % 4 == 0
        zero = max(p for b in bins for p in b[4:8])                      # the all-zero position is the last
        for c in range(0, len(bins), 4):
            tile = bins[c:c + 4]
            items = tile[0][15] >> 1
            assert items in (0, 3, 4) and all(b[15] >> 1 == items for b in tile)
            multiplied += 4 * items
            for b in tile:
                scaled = [q for q in range(4) if b[4 + q] != zero]
                assert (b[15] & 1) == (len(scaled) > 0) and all(q < items for q in scaled)
                assert all(b[q] == b[4 + q] for q in scaled)             # an item's codes and scales
                run = []
                for q in range(4):
                    if b[4 + q] != zero:
                        run.append(b[4 + q])
                    if (b[13] >> q) & 1:
                        key = (b[12], b[8 + q], (b[14] >> q) & 1)
                        assert key not in seen
                        seen[key] = run
                        stored += len(run)
                        run = []
                assert run == []
        for m, size in enumerate(split):
            for rb in range(n_rb):
                u, up = (rb % (n_rb // 2), rb // (n_rb // 2)) if gated else (rb, 0)
                want = [k for k in orders_of[rb] if first[m] <= k < first[m] + size]
                got = seen.pop((m, u, up))
                assert len(got) == len(want) == len(set(got)), (rows, m, rb)
        assert seen == {}
        assert stored == sum(len(o) for o in orders_of)
        assert multiplied <= most * stored, (rows, K, part, split, gated, multiplied, stored)


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


def _tile(names):
    """(bits, blocks of 16 tokens, groups along k, stages ahead) of the one single-pass launch among `names`."""
    found = [re.search(r"gemm_bins_kernelILi(\d)ELi(\d)ELi\dELi\dELb[01]ELi(\d)ELi(\d)E", n) for n in names]
    (m,) = [f for f in found if f]
    return tuple(int(g) for g in m.groups())


def tiles_follow_the_units_they_leave(rt):
    """Height, groups and loads ahead of the single-pass kernel by the tiles that 256 compute units in 8 dies are dealt (each of these
    sizes was slower another way)."""
    for rows, inp, bits, K, T, want in (
            (768, 3072, 8, 2, 600, (8, 1, 1, 2)), (768, 3072, 8, 2, 1000, (8, 2, 1, 2)), (768, 3072, 8, 2, 1800, (8, 4, 1, 2)),
            (768, 3072, 8, 2, 2600, (8, 4, 1, 1)),                                        # one die is dealt more tiles than it has units
            (4096, 4096, 8, 2, 200, (8, 2, 1, 2)), (4096, 4096, 8, 2, 500, (8, 4, 1, 2)), (4096, 4096, 8, 2, 600, (8, 4, 1, 1)),
            (11008, 4096, 8, 2, 160, (8, 2, 1, 1)), (11008, 4096, 8, 2, 190, (8, 4, 1, 1)), (2304, 768, 8, 2, 700, (8, 4, 1, 1)),
            (768, 3072, 4, 2, 250, (4, 1, 1, 2)), (4096, 11008, 4, 2, 200, (4, 2, 2, 2)), (4096, 4096, 4, 2, 400, (4, 4, 2, 2)),
            (4096, 4096, 4, 2, 600, (4, 4, 1, 2)), (4096, 4096, 4, 2, 4096, (4, 4, 1, 1)), (3072, 768, 4, 2, 300, (4, 2, 1, 2)), (3072, 512, 4, 2, 300, (4, 2, 1, 1)),
            (768, 3072, 2, 2, 250, (2, 1, 1, 2)), (4096, 4096, 2, 2, 200, (2, 2, 2, 2)), (4096, 4096, 2, 2, 600, (2, 4, 1, 2)),
            (4096, 11008, 2, 2, 500, (2, 4, 1, 2)), (6144, 4096, 2, 2, 322, (2, 4, 1, 2)), (5632, 4096, 2, 2, 322, (2, 2, 2, 2)), (5632, 3072, 2, 2, 322, (2, 4, 1, 2))):
        e = rt.expand(rows, inp, bits, K, 1.0, 16)
        assert _linear(rt, e, T) == 0
        assert _tile(rt.names()) == want, (rows, inp, bits, T)
    rt.lib.pipe_expand_conv2d.argtypes = [C.c_void_p] + [C.c_int] * 6 + [C.c_float, C.c_int, C.c_void_p, C.POINTER(C.c_void_p)]
    rt.lib.pipe_forward_conv2d.argtypes = [C.c_void_p] * 2 + [C.c_int] * 9 + [C.c_float, C.c_void_p, C.c_int, C.c_void_p, C.c_int] + [C.c_void_p] * 2
    for rows, Ch, H, N, bits, want in ((512, 256, 14, 5, 8, (8, 1, 1, 2)), (512, 256, 14, 10, 8, (8, 2, 1, 2)), (512, 512, 7, 32, 8, (8, 2, 1, 2)),
                                       (256, 256, 14, 5, 2, (2, 1, 1, 1)), (128, 64, 56, 8, 2, (2, 4, 1, 1)), (512, 512, 7, 60, 2, (2, 4, 1, 2)), (256, 256, 14, 5, 4, (4, 1, 1, 2))):
        W, e = (C.c_float * (rows * Ch * 9))(), C.c_void_p()
        assert rt.lib.pipe_expand_conv2d(W, rows, Ch, 3, 3, bits, 2, 1.0, 16, None, C.byref(e)) == 0
        rt.names()
        assert rt.lib.pipe_forward_conv2d(e, 1 << 40, N, Ch, H, H, 3, 3, 1, 1, 0, 0.0, None, 0, None, 1, 1 << 44, None) == 0
        assert _tile(rt.names()) == want, (rows, Ch, N, bits)

    rt.lib.pipe_chain_forward.argtypes = [C.c_void_p, C.c_int, C.c_void_p, C.c_int, C.c_float, C.c_void_p, C.c_int] + [C.c_void_p] * 3
    for width, T, want in ((1024, 1000, (4, 4, 1, 2)), (1024, 1100, (4, 4, 1, 1)), (1536, 700, (4, 4, 1, 2))):   # 256, 288 and 264 tiles of 64
        e = rt.expand(width, width, 4, 4, 1.0, 16)
        arr = (Layer * 2)(Layer(e, None, 3, -1), Layer(e, None, 0, -1))
        rt.names()
        assert rt.lib.pipe_chain_forward(arr, 2, 1 << 40, T, 0.0, (C.c_int * 1)(4), 1, None, 1 << 44, None) == 0
        names = [n for n in rt.names() if "gemm_bins_kernel" in n]
        assert _tile(names[:1]) == want, (width, T, names)


def a_sum_over_two_members_is_a_launch_each(rt):
    """The second layer of an MLP: a launch of the single-pass kernel per member where the walk is long and a member of a single order
    has 192 tiles; else one launch, pass by pass."""
    mlp = rt.lib.pipe_mlp_forward
    mlp.argtypes = [C.c_void_p] * 2 + [C.c_int, C.c_void_p, C.c_int, C.c_float, C.c_void_p, C.c_int] + [C.c_void_p] * 5

    def launches(rows, hidden, K, split, T, kept):
        l1, l2 = rt.expand(hidden, 64, 4, K, 1.0, 16), rt.expand(rows, hidden, 4, K, 0.5 if kept else 1.0, 16, kept=kept)
        arr = (C.c_int * len(split))(*split)
        rt.names()
        assert mlp(l1, l2, 1, 1 << 40, T, 0.0, arr, len(split), None, None, None, 1 << 44, None) == 0
        names = rt.names()
        modes = [int(m.group(1)) for m in (re.search(r"gemm_bins_kernelILi\dELi\dELi\dELi(\d)E", n) for n in names) if m]
        return modes, sum("gemm_tiled_kernel" in n for n in names)

    half = [list(range(0, 256, 2)), list(range(1, 256, 2))]
    assert launches(4096, 3072, 3, [2, 1], 1540, half) == ([2, 0, 6], 0)      # GELU, first member, the other's on top: 8 x 25 tiles
    assert launches(4096, 3072, 3, [2, 1], 1500, half) == ([2, 0, 6], 0)      # 8 x 24
    assert launches(4096, 3072, 3, [2, 1], 1470, half) == ([2], 1)            # 8 x 23
    assert launches(1040, 3072, 4, [2, 2], 300, ()) == ([2, 0, 6], 0)
    assert launches(1040, 2816, 4, [2, 2], 300, ()) == ([2], 1)               # 44 steps


def unprepared_batches_stream(rt):
    """17 to 128 tokens of a layer that the tiled kernel serves by rule: where an allocation of its schedule fails, or under capture without
    one, the streaming kernel runs, once; a prepared layer is captured tiled."""
    def kernels():
        names = rt.names()
        return sum("gemm_stream_kernel" in n for n in names), sum("gemm_bins_kernel" in n for n in names)

    e = rt.expand(8192, 320, 4, 2, 1.0, 16)
    assert _linear(rt, e, 16) == 0 and kernels() == (1, 0)
    assert _linear(rt, e, 200) == 0 and kernels() == (0, 1)                       # this stream's scratch is there
    for nth in range(1, 9):
        e = rt.expand(8192, 320, 4, 2, 1.0, 16)
        rt.names()
        rt.host.host_fail(nth)
        assert _linear(rt, e, 64) == 0
        rt.host.host_fail(0)
        first = kernels()
        assert first in ((1, 0), (0, 1))
        assert _linear(rt, e, 64) == 0 and kernels() == (0, 1)
        if first == (0, 1):
            break
    assert 2 <= nth < 8
    e = rt.expand(8192, 320, 4, 2, 1.0, 16)
    rt.names()
    rt.host.host_capture(1)
    assert _linear(rt, e, 64) == 0 and kernels() == (1, 0)
    assert _linear(rt, e, 200) == ENOTREADY and kernels() == (0, 0)
    rt.host.host_capture(0)
    rt.lib.pipe_prepare.argtypes = [C.c_void_p] * 2 + [C.c_int] * 2 + [C.c_void_p]
    assert rt.lib.pipe_prepare(e, None, 0, 128, None) == 0 and kernels() == (0, 0)
    rt.host.host_capture(1)
    assert _linear(rt, e, 64) == 0 and kernels() == (0, 1)
    rt.host.host_capture(0)


def prepared_calls_allocate_nothing(rt):
    """After a preparation for T_max tokens every call of no more is served under capture: tiled, streamed (a gated layer's raw outputs
    have a buffer of their own there), in one resident launch, and from inputs that the resident launch does not take."""
    mlp, chain, prep_mlp, prep_chain = (getattr(rt.lib, "pipe_" + n) for n in ("mlp_forward", "chain_forward", "prepare_mlp", "prepare_chain"))
    mlp.argtypes = [C.c_void_p] * 2 + [C.c_int, C.c_void_p, C.c_int, C.c_float, C.c_void_p, C.c_int] + [C.c_void_p] * 5
    prep_mlp.argtypes = [C.c_void_p] * 2 + [C.c_int, C.c_void_p, C.c_int, C.c_int, C.c_void_p]
    chain.argtypes = [C.c_void_p, C.c_int, C.c_void_p, C.c_int, C.c_float, C.c_void_p, C.c_int] + [C.c_void_p] * 3
    prep_chain.argtypes = [C.c_void_p] + [C.c_int] * 4 + [C.c_void_p, C.c_int, C.c_void_p]

    def captured(call, t_max, stream, what):
        for T in sorted({1, 8, 9, 16, 17, 33, 64, 65, 100, 112, 113, 128, 129, 200, t_max}):
            if T > t_max:
                break
            for x in (1 << 40, (1 << 40) + 4):
                rt.host.host_fail(0)
                rt.host.host_capture(1)
                rc = call(T, x, stream)
                rt.host.host_capture(0)
                assert (rc, rt.host.host_mallocs()) == (0, 0), (what, t_max, T, x & 15, rc)

    stream = 0
    for t_max in (6, 16, 40, 100, 128, 129, 130, 300):
        for act, split in ((2, (2, 2)), (2, (3, 1)), (2, None), (1, (2, 2)), (1, None)):
            K = sum(split) if split else 3
            l1, l2 = rt.expand((2 if act == 2 else 1) * 512, 320, 4, K, 1.0, 16), rt.expand(320, 512, 4, K, 1.0, 16)
            arr, M = ((C.c_int * len(split))(*split), len(split)) if split else (None, 0)
            stream += 4096                        # one that nobody has used
            assert prep_mlp(l1, l2, act, arr, M, t_max, stream) == 0
            captured(lambda T, x, st: mlp(l1, l2, act, x, T, 0.0, arr, M, None, None, None, 1 << 44, st), t_max, stream, (act, split))
        for K, split in ((4, (2, 2)), (3, None), (8, (4, 4))):
            arr, M = ((C.c_int * len(split))(*split), len(split)) if split else (None, 0)
            es = [rt.expand(320, 320, 4, K, 1.0, 16) for _ in range(3)]
            layers = (Layer * 3)(*[Layer(e, None, 0, -1) for e in es])
            stream += 4096
            assert prep_chain(layers, 3, t_max, 1, 1, arr, M, stream) == 0
            captured(lambda T, x, st: chain(layers, 3, x, T, 0.0, arr, M, None, 1 << 44, st), t_max, stream, ("chain", split))


def failed_launches_are_reported(rt):
    """A launch that fails in the middle of a call of 17 to 128 tokens on the tiled kernels ends the call with its error: no kernel is sent
    behind it, and the next call starts with the maxima cleared."""
    mlp, chain = rt.lib.pipe_mlp_forward, rt.lib.pipe_chain_forward
    mlp.argtypes = [C.c_void_p] * 2 + [C.c_int, C.c_void_p, C.c_int, C.c_float, C.c_void_p, C.c_int] + [C.c_void_p] * 5
    chain.argtypes = [C.c_void_p, C.c_int, C.c_void_p, C.c_int, C.c_float, C.c_void_p, C.c_int] + [C.c_void_p] * 3
    rt.lib.pipe_forward_asymmetric.argtypes = [C.c_void_p] * 2 + [C.c_int, C.c_void_p, C.c_int] + [C.c_void_p] * 3
    wide = rt.expand(8192, 320, 4, 2, 1.0, 16)
    l1, l2 = rt.expand(22016, 320, 4, 4, 1.0, 16), rt.expand(320, 11008, 4, 4, 1.0, 16)
    es = [rt.expand(1536, 1536, 4, 4, 1.0, 16) for _ in range(3)]
    layers, one = (Layer * 3)(*[Layer(e, None, 0, -1) for e in es]), (C.c_int * 1)(4)
    calls = {"linear": lambda: _linear(rt, wide, 100),
             "asymmetric": lambda: rt.lib.pipe_forward_asymmetric(wide, 1 << 40, 100, None, 0, None, 1 << 44, None),
             "mlp": lambda: mlp(l1, l2, 2, 1 << 40, 100, 0.0, None, 0, None, None, None, 1 << 44, None),
             "chain": lambda: chain(layers, 3, 1 << 40, 100, 0.0, one, 1, None, 1 << 44, None)}
    for what, call in calls.items():
        assert call() == 0
        rt.names()
        assert call() == 0
        whole = [n for n in rt.names() if "kernel" in n]
        assert any("gemm_bins_kernel" in n for n in whole) and not any("gemm_stream" in n for n in whole), whole
        for nth in range(1, len(whole) + 1):
            rt.host.host_fail_launch(nth)
            assert call() == EDEVICE, (what, nth)
            assert rt.names() == whole[:nth - 1], (what, nth)
            rt.host.host_fail_launch(0)
            assert call() == 0
            assert [n for n in rt.names() if "zero_u32" not in n] == whole, (what, nth)


def batches_take_the_kernel_of_their_size(rt):
    """Layers, MLPs and chains of 17 to 128 tokens, on both sides of each line between the kernels: the last batch that is streamed and the first that is
    tiled.  Where a schedule of the tiled route cannot be built, or under capture, the whole call is streamed."""
    mlp, chain = rt.lib.pipe_mlp_forward, rt.lib.pipe_chain_forward
    mlp.argtypes = [C.c_void_p] * 2 + [C.c_int, C.c_void_p, C.c_int, C.c_float, C.c_void_p, C.c_int] + [C.c_void_p] * 5
    chain.argtypes = [C.c_void_p, C.c_int, C.c_void_p, C.c_int, C.c_float, C.c_void_p, C.c_int] + [C.c_void_p] * 3

    def route():
        names = rt.names()
        tiled = ["gemm_stream" not in n for n in names if "gemm_" in n]
        assert tiled and len(set(tiled)) == 1, names
        return tiled[0]

    def members(split):
        return ((C.c_int * len(split))(*split), len(split)) if split else (None, 0)

    def an_mlp(act, width, hidden, bits, K, split):
        l1, l2 = rt.expand((2 if act == 2 else 1) * hidden, width, bits, K, 1.0, 16), rt.expand(width, hidden, bits, K, 1.0, 16)
        arr, M = members(split)
        return lambda T: mlp(l1, l2, act, 1 << 40, T, 0.0, arr, M, None, None, None, 1 << 44, None)

    def a_chain(width, L, bits, K, split):
        es = [rt.expand(width, width, bits, K, 1.0, 16) for _ in range(L)]
        layers, (arr, M) = (Layer * L)(*[Layer(e, None, 0, -1) for e in es]), members(split)
        return lambda T: chain(layers, L, 1 << 40, T, 0.0, arr, M, None, 1 << 44, None)

    def a_layer(out, width, bits, K):
        e = rt.expand(out, width, bits, K, 1.0, 16)
        return lambda T: _linear(rt, e, T)

    GELU, GATED = 1, 2
    lines = ((a_layer, (1024, 5120, 4, 4), 112), (a_layer, (1024, 1024, 4, 4), 96), (a_layer, (1024, 1024, 2, 4), 96), (a_layer, (2048, 1024, 8, 2), 96), (a_layer, (768, 3072, 4, 4), 128),
             (an_mlp, (GELU, 320, 1088, 4, 3, None), 64), (an_mlp, (GELU, 768, 3072, 4, 2, None), 96), (an_mlp, (GELU, 768, 3072, 4, 3, None), 80),
             (an_mlp, (GELU, 320, 1088, 4, 2, (1, 1)), 128), (an_mlp, (GELU, 320, 1088, 8, 2, None), 128),
             (an_mlp, (GATED, 320, 1088, 4, 3, None), 64), (an_mlp, (GATED, 320, 480, 4, 4, (2, 2)), 64), (an_mlp, (GATED, 320, 1088, 4, 4, (2, 2)), 128),
             (an_mlp, (GATED, 1024, 3072, 4, 4, (2, 2)), 96), (an_mlp, (GATED, 320, 1088, 2, 4, (2, 2)), 96), (an_mlp, (GATED, 320, 3072, 2, 4, (2, 2)), 64),
             (an_mlp, (GATED, 320, 1088, 4, 4, (3, 1)), 112), (an_mlp, (GATED, 512, 3072, 4, 4, (3, 1)), 128), (an_mlp, (GATED, 1024, 3072, 4, 4, (3, 1)), 112),
             (a_chain, (1536, 3, 4, 4, None), 80), (a_chain, (1536, 3, 4, 4, (2, 2)), 96), (a_chain, (1536, 3, 2, 4, (2, 2)), 112), (a_chain, (320, 3, 4, 4, None), 128),
             (a_chain, (320, 3, 4, 8, (4, 4)), 128), (a_chain, (320, 6, 4, 8, (4, 4)), 64), (a_chain, (2880, 3, 4, 8, (4, 4)), 64), (a_chain, (320, 3, 4, 8, None), 128))
    for make, args, last in lines:
        call = make(*args)
        for T in (17, last, last + 1) if last < 128 else (17, 65, 97, last):
            assert call(T) == 0
            assert route() == (T > last), (args, T)
    for make, args, T in ((an_mlp, (GATED, 320, 480, 4, 4, (2, 2)), 100), (an_mlp, (GELU, 320, 1088, 4, 3, None), 100), (a_chain, (320, 6, 4, 8, (4, 4)), 100)):
        assert make(*args)(200) == 0                     # this stream's scratch is there
        assert make(*args)(64) == 0                      # (and the streamed gated layer's)
        streamed = 0
        for nth in range(1, 30):
            call = make(*args)
            rt.names()
            rt.host.host_fail(nth)
            assert call(T) == 0
            rt.host.host_fail(0)
            if route():
                break
            streamed += 1
            assert call(T) == 0 and route()
        assert 2 <= streamed < 29, (args, streamed)      # each layer's schedules
        call = make(*args)
        rt.host.host_capture(1)
        assert call(T) == 0 and not route()
        rt.host.host_capture(0)


def streamed_8_bit_walks_ask_for_two_tiles(rt):
    """The instance of the streaming kernel that an 8-bit layer takes, on both sides of each line: token blocks, steps of k, bins; an input for
    each member takes one tile at a time."""
    mlp = rt.lib.pipe_mlp_forward
    mlp.argtypes = [C.c_void_p] * 2 + [C.c_int, C.c_void_p, C.c_int, C.c_float, C.c_void_p, C.c_int] + [C.c_void_p] * 5

    def tiles():
        return [int(m.group(1)) for m in (re.search(r"gemm_stream_kernelILi\d.*?Stream(?:Params|Plain)ELi(\d)E", n) for n in rt.names()) if m]

    for out, width, bits, K, T, want in ((256, 256, 8, 2, 33, 2), (256, 4096, 8, 2, 16, 1), (256, 320, 4, 2, 33, 1), (256, 320, 2, 4, 33, 1),
                                         (16384, 512, 8, 4, 16, 2), (16368, 512, 8, 4, 16, 1),                                   # 1024 bins
                                         (2048, 4352, 8, 4, 1, 2), (2032, 4352, 8, 4, 1, 1), (2048, 4096, 8, 4, 1, 1),           # quantized by the launch: 128 bins, 68 steps
                                         (20496, 256, 8, 4, 1, 2), (20480, 256, 8, 4, 1, 1),                                     # ... 1281 bins
                                         (8192, 8192, 8, 4, 16, 2), (8176, 8192, 8, 4, 16, 1), (8192, 7936, 8, 4, 16, 1)):       # 512 bins, 128 steps
        e = rt.expand(out, width, bits, K, 1.0, 16)
        rt.names()
        assert _linear(rt, e, T) == 0
        assert tiles() == [want], (out, width, bits, K, T)
    l1, l2 = rt.expand(512, 320, 8, 4, 1.0, 16), rt.expand(320, 512, 8, 4, 1.0, 16)
    two = (C.c_int * 2)(2, 2)
    rt.names()
    assert mlp(l1, l2, 1, 1 << 40, 40, 0.0, two, 2, None, None, None, 1 << 44, None) == 0
    assert tiles() == [2, 1]


@pytest.mark.parametrize("scenario", ["failed_allocation_is_reported_once", "control_words_start_at_zero",
                                      "failed_preparation_starts_over", "capture_builds_nothing",
                                      "any_number_of_images_is_served", "wide_layers_quantize_once",
                                      "single_pass_tables_hold_no_needless_items", "tiles_follow_the_units_they_leave",
                                      "a_sum_over_two_members_is_a_launch_each", "unprepared_batches_stream",
                                      "prepared_calls_allocate_nothing", "failed_launches_are_reported",
                                      "batches_take_the_kernel_of_their_size", "streamed_8_bit_walks_ask_for_two_tiles"])
def test_host(scenario, tmp_path):
    _host_hip.run(__file__, scenario, tmp_path)


if __name__ == "__main__":
    globals()[sys.argv[1]](_host_hip.Runtime(sys.argv[2]))
