"""The activation quantizers' quotient (a correctly rounded division by corrections, IEEE division outside its range) and the
reduction in front of it: the codes are those of numpy's fp32 division for values on, next to and far from the edges
between two codes, for every size of scale, for infinities and NaN, at every alignment of the input."""
import numpy as np
import pytest
import torch

from _parity import dev

pytestmark = pytest.mark.gpu

f32 = np.float32


@pytest.fixture(scope="module")
def pipe():
    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_2311_15806_amd.binding as b
    return b


def _codes(x, s):
    with np.errstate(all="ignore"):
        q = np.rint((x / f32(s)).astype(f32))
    q = np.where(np.isnan(q), -127, q)          # max(NaN, -127) is -127
    return np.clip(q, -127, 127).astype(np.int8)


def _edges(s, n, seed):
    """Values within a few ulp of (k + 1/2) s, others spread over many binades, and the special ones."""
    rng = np.random.default_rng(seed)
    mid = ((rng.integers(-130, 130, n // 2) + 0.5) * np.float64(f32(s))).astype(f32)
    mid = (mid.view(np.int32) + rng.integers(-3, 4, mid.size)).view(f32)
    wide = (rng.standard_normal(n - mid.size) * np.exp2(rng.uniform(-20, 8, n - mid.size)) * s).astype(f32)
    x = np.concatenate([mid, wide])
    x[:6] = [np.inf, -np.inf, np.nan, 0.0, -0.0, f32(1e-45)]
    x[6:8] = [f32(3e38), f32(-3e38)]
    return x


@pytest.mark.parametrize("s", [0.03, 1.0, 0.0123456789, 3.3e-5, 7.7e8, 1.1e-26, 0.9e-27, 1e-38, 2e27, 1e36])
def test_codes_are_those_of_the_division(pipe, s):
    T, I = 200, 512
    e = pipe.pipe_expand(dev(np.random.default_rng(1).standard_normal((16, I)).astype(f32)), 8, 1, 1.0, 16)
    x = _edges(s, T * I, int(1000 * np.log2(s)) & 0xffff).reshape(T, I)
    _, qx, sx = pipe.pipe_forward_acc(e, dev(x), s_x=s)
    ref = _codes(x, s)
    assert np.array_equal(qx.cpu().numpy(), ref)
    assert float(sx.item()) == float(f32(s))
    # the wide path (no row-major copy): the layer on these codes is exact in integers, one order, one scale
    gids, scales, codes = e.order(1)
    acc = ref.astype(np.int64) @ codes.astype(np.int64).T
    y = pipe.pipe_forward(e, dev(x), s_x=s).cpu().numpy()
    with np.errstate(all="ignore"):
        exact = np.float64(f32(s)) * (scales.astype(np.float64) * acc)
    ok = np.isfinite(exact.astype(f32)) & (np.abs(exact) > 1e-30)
    assert np.all(np.abs(y[ok] - exact[ok]) <= 3e-7 * np.abs(exact[ok]))     # two fp32 products
    e.free()


@pytest.mark.parametrize("T,I", [(33, 1028), (129, 4), (140, 68), (300, 516), (1000, 4100)])
@pytest.mark.parametrize("shift", [0, 1])
def test_dynamic_scale_over_the_parts_of_the_reduction(pipe, T, I, shift):
    """The largest magnitude in the first, a middle and the last element; inputs that are not 16-byte aligned."""
    e = pipe.pipe_expand(dev(np.random.default_rng(2).standard_normal((16, I)).astype(f32)), 8, 1, 1.0, 16)
    for at in (0, T * I // 2, T * I - 1):
        x = np.random.default_rng(at + I).standard_normal(T * I).astype(f32)
        x[at] = -37.5
        buf = torch.empty(T * I + 4, dtype=torch.float32, device="cuda")
        xd = buf[shift:shift + T * I].view(T, I)
        xd.copy_(dev(x.reshape(T, I)))
        _, qx, sx = pipe.pipe_forward_acc(e, xd)
        s = f32(37.5) / f32(127)
        assert float(sx.item()) == float(s)
        assert np.array_equal(qx.cpu().numpy(), _codes(x, s).reshape(T, I))
        y, ys = pipe.pipe_forward(e, xd), pipe.pipe_forward(e, xd, s_x=float(s))
        assert torch.equal(y, ys)
        lo = float(max(0.0, float(-x.min())))
        hi = float(max(0.0, float(x.max())))
        _, qa, sa, z = pipe.pipe_forward_acc_asymmetric(e, xd)
        sar = f32(f32(hi) + f32(lo)) / f32(255)
        zr = int(np.clip(np.rint(f32(lo) / sar), 0, 255))
        assert sa == float(sar) and z == zr
        assert np.array_equal(qa.cpu().numpy(), np.clip(np.rint(x / sar) + f32(zr), 0, 255).astype(np.uint8).reshape(T, I))
    e.free()


@pytest.mark.parametrize("C,H,W,N", [(64, 1, 3, 2), (64, 9, 7, 3), (128, 7, 7, 2), (192, 4, 17, 2), (256, 6, 6, 1),
                                       (64, 57, 59, 5), (128, 48, 44, 4), (64, 113, 115, 21)])   # two and four loads a lane
@pytest.mark.parametrize("shift", [0, 1])
def test_channels_last_codes_and_sums(pipe, C, H, W, N, shift):
    """Codes and per-pixel sums of a convolution's input at the edges of its tiles of 1024 to 4096 elements, both layouts, inputs that are not
    16-byte aligned: a pointwise layer's accumulators and outputs (bit for bit) against the codes."""
    rng = np.random.default_rng(C + H + W)
    x = rng.standard_normal((N, C, H, W)).astype(f32)
    e = pipe.pipe_expand_conv2d(dev(rng.standard_normal((32, C)).astype(f32)), C, 1, 1, 4, 1, 1.0, 16)
    _, _, codes = e.order(1)
    s = f32(f32(np.abs(x).max()) / f32(127))
    q = _codes(x.reshape(-1), s).reshape(x.shape).astype(np.int64)
    want = q.transpose(0, 2, 3, 1).reshape(-1, C).astype(np.float64) @ codes.T.astype(np.float64)    # (whole numbers below 2^53)
    ys = []
    for nhwc in (False, True):
        xl = np.ascontiguousarray(x.transpose(0, 2, 3, 1)) if nhwc else x
        buf = torch.empty(x.size + 4, dtype=torch.float32, device="cuda")
        xd = buf[shift:shift + x.size].view(*xl.shape)
        xd.copy_(dev(xl))
        acc, _, sx = pipe.pipe_forward_conv2d_acc(e, xd, 1, 1, 1, 0, nhwc=nhwc)
        assert float(sx.item()) == float(s)
        assert np.array_equal(acc.cpu().numpy()[0], want)
        ys.append(pipe.pipe_forward_conv2d(e, xd, 1, 1, 1, 0, nhwc=nhwc))
    assert torch.equal(ys[0], ys[1])
    e.free()
