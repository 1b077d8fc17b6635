"""The single-pass tiled kernel (batches above 128 tokens, members of at most 4 orders) where its tiles have edges:
one token more than the streaming kernel takes, token tiles of one token, all token-tile heights, column tiles with
empty waves, row blocks that a member pruned, bins of every composition, one stage of k and many.  With a given scale
every token is independent of its batch, and both kernels fold the orders with the same fp32 operations in the same
order: a batch must equal its parts of at most 128 tokens, which the streaming kernel serves, bit for bit."""
import numpy as np
import pytest
import torch

from _parity import dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pipe():
    assert torch.cuda.is_available(), "these tests need the GPU"
    import paper_2311_15806_amd.binding as b
    return b


def _weight(seed, O, I):
    rng = np.random.default_rng(seed)
    return (rng.standard_t(3, size=(O, I)) * 0.02).astype(np.float32)


def _parts(T):
    return [(a, min(a + 128, T)) for a in range(0, T, 128)]


#            O     I     bits K gamma group split   T
LAYERS = [(16, 100, 4, 1, 1.0, 16, [1], 129),
          (48, 256, 2, 4, 0.34, 16, [4], 193),       # counts 1 to 4: every kind of bin; n_bins no multiple of 4
          (1040, 300, 2, 4, 0.25, 16, [1, 3], 150),  # members: most row blocks of the second are pruned
          (320, 1030, 4, 3, 0.5, 32, [2, 1], 257),
          (256, 700, 8, 2, 1.0, 16, [1, 1], 191),
          (2048, 512, 3, 4, 0.5, 64, [2, 2], 400),   # 64-token tiles
          (4096, 260, 2, 3, 0.5, 64, [3], 321),
          (4096, 1000, 2, 4, 0.5, 64, [4], 381),     # ternary, loads between the multiplies two stages ahead
          (48, 1500, 4, 3, 0.5, 16, [3], 129),       # the same with tiles of 16 tokens: six stages ...
          (320, 1700, 4, 4, 0.5, 16, [2, 2], 150),   # ... seven
          (2048, 1800, 4, 4, 0.5, 16, [4], 501),     # two groups along k, tiles of 64 tokens
          (2048, 1700, 2, 4, 0.5, 16, [4], 200),     # ... of 32
          (1024, 1800, 8, 2, 1.0, 16, [2], 502),
          (48, 2000, 2, 4, 0.34, 16, [4], 193),      # 16 tokens, two stages ahead, eight of them
          (2048, 1700, 4, 4, 0.5, 16, [4], 300),     # two groups, 32 tokens, seven stages: four and three
          (4096, 2000, 4, 4, 0.5, 16, [4], 390),     # 64 tokens, two stages ahead, 16 of them ...
          (4096, 1700, 4, 3, 0.5, 16, [2, 1], 420),  # ... 14
          (2048, 1100, 8, 2, 1.0, 16, [2], 400),     # 8 bits, two ahead: 32 tokens ...
          (4096, 700, 8, 2, 1.0, 16, [1, 1], 257),   # ... 64
          (11008, 300, 8, 2, 1.0, 16, [2], 130),     # 8 bits, two low tiles a compute unit
          (3072, 768, 4, 3, 0.5, 16, [3], 333),      # 4 bits, 32 tokens, two ahead: six stages ...
          (2048, 1000, 4, 4, 0.5, 16, [1, 3], 280)]  # ... eight


@pytest.mark.parametrize("O,I,bits,K,gamma,group,split,T", LAYERS)
@pytest.mark.parametrize("reduce", [True, False])
def test_batch_equals_its_parts(pipe, O, I, bits, K, gamma, group, split, T, reduce):
    rng = np.random.default_rng(O + I + T)
    e = pipe.pipe_expand(dev(_weight(O * 7 + I, O, I)), bits, K, gamma, group)
    x = dev(rng.standard_normal((T, I)).astype(np.float32))
    b = dev(rng.standard_normal(O).astype(np.float32))
    for tile in (0, 16, 32, 64):
        pipe.pipe_set_token_tile(tile)
        try:
            y = pipe.pipe_forward(e, x, s_x=0.03, split=split, bias=b, reduce_members=reduce)
        finally:
            pipe.pipe_set_token_tile(0)
        ref = torch.cat([pipe.pipe_forward(e, x[a:z].contiguous(), s_x=0.03, split=split, bias=b, reduce_members=reduce)
                         for a, z in _parts(T)], dim=0 if reduce else 1)
        assert torch.equal(y, ref), "token tile %d" % tile
    e.free()


@pytest.mark.parametrize("H,I,bits,K,gamma,split,T", [(48, 200, 4, 2, 0.5, [2], 129), (336, 260, 2, 4, 0.25, [2, 2], 321),
                                                      (2752, 300, 4, 4, 0.5, [2, 2], 200)])
def test_gated_batch_equals_its_parts(pipe, H, I, bits, K, gamma, split, T):
    rng = np.random.default_rng(H + T)
    l1 = pipe.pipe_expand(dev(_weight(H, 2 * H, I)), bits, K, gamma, 16)
    l2 = pipe.pipe_expand(dev(_weight(H + 1, 64, H)), bits, K, gamma, 16)
    x = dev(rng.standard_normal((T, I)).astype(np.float32))
    b1 = dev(rng.standard_normal(2 * H).astype(np.float32))
    call = lambda v: pipe.pipe_mlp_forward_given_scales(l1, l2, pipe.PIPE_ACT_SILU_GATED, v, 0.03, [0.02] * len(split), split=split,
                                                        bias1=b1, return_hidden=True)
    y, h = call(x)
    parts = [call(x[a:z].contiguous()) for a, z in _parts(T)]
    # SiLU(gate)*up is evaluated by another kernel at 128 tokens and less: the same fp32 formula, a few ulp apart at most
    ref = torch.cat([p[1] for p in parts], dim=1)
    assert (h - ref).abs().max() <= 4e-7 * ref.abs().max()
    # one code of Q(h) may fall the other way for it: one step of the hidden scale times a weight
    yr = torch.cat([p[0] for p in parts], dim=0)
    assert (y - yr).abs().max() <= 1e-5 * yr.abs().max() + 0.02 * float(pipe.pipe_expansion_reconstruct(l2).abs().max())
    l1.free(), l2.free()


#            N  C    H   W   stride pad bits K
DEPTHWISE = [(2, 16, 1, 1, 1, 1, 8, 1), (3, 80, 7, 7, 1, 1, 4, 2), (1, 64, 13, 36, 1, 0, 2, 4), (2, 144, 28, 28, 2, 1, 4, 3),
             (1, 32, 9, 70, 2, 2, 3, 4), (1, 208, 6, 33, 1, 2, 4, 3)]


@pytest.mark.parametrize("N,C,H,W,stride,pad,bits,K", DEPTHWISE)
def test_fused_depthwise_at_its_tile_edges(pipe, N, C, H, W, stride, pad, bits, K):
    """Partial channel groups, row bands and column tiles, windows wholly in the padding, all four ways the input is read (16 bytes
    at a time or element by element, channels first or last); an output that overlaps the input, which takes two steps."""
    from oracle import pipe_oracle as po
    rng = np.random.default_rng(C + W)
    Wt = rng.standard_normal((C, 9)).astype(np.float32)
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    b = rng.standard_normal(C).astype(np.float32)
    e = pipe.pipe_expand(dev(Wt), bits, K, 0.5, 16)
    ora = po.expand(Wt, bits, K, 0.5, 16)
    for s_x in (0.0, 0.02):
        ref = po.forward_depthwise2d(ora, x, 3, 3, stride, pad, s_x=s_x if s_x > 0 else None, bias=b)["y"]
        y = pipe.pipe_forward_depthwise2d(e, dev(x), 3, 3, stride, pad, s_x=s_x, bias=dev(b))
        # exact integer sums, at most K + 1 rounded fp32 operations of terms no larger than the layer's largest output
        assert np.abs(y.cpu().numpy() - ref).max() <= (K + 1) * 1.2e-7 * 4 * np.abs(ref).max()
        yl = pipe.pipe_forward_depthwise2d(e, dev(x.transpose(0, 2, 3, 1)), 3, 3, stride, pad, nhwc=True, s_x=s_x, bias=dev(b))
        assert torch.equal(y, yl)
        buf = torch.empty(x.size + 1, dtype=torch.float32, device="cuda")   # not 16-byte aligned: element by element
        xs = buf[1:].view(N, C, H, W)
        xs.copy_(dev(x))
        assert torch.equal(y, pipe.pipe_forward_depthwise2d(e, xs, 3, 3, stride, pad, s_x=s_x, bias=dev(b)))
        xs = buf[1:].view(N, H, W, C)
        xs.copy_(dev(x.transpose(0, 2, 3, 1)))
        assert torch.equal(y, pipe.pipe_forward_depthwise2d(e, xs, 3, 3, stride, pad, nhwc=True, s_x=s_x, bias=dev(b)))
        both = torch.empty(max(x.size, y.numel()), dtype=torch.float32, device="cuda")
        both[:x.size].view(N, H, W, C).copy_(dev(x.transpose(0, 2, 3, 1)))
        bias = dev(b)
        assert pipe._lib.pipe_forward_depthwise2d(e.handle, both.data_ptr(), N, C, H, W, 3, 3, stride, pad, 1, float(s_x), None, 0,
                                                  bias.data_ptr(), 1, both.data_ptr(), pipe._stream()) == 0
        assert torch.equal(y, both[:y.numel()].view_as(y))
    e.free()


@pytest.mark.parametrize("N,C,H,W", [(5000, 48, 3, 3), (70000, 16, 1, 1), (9, 80, 20, 33), (300, 32, 30, 41)])
@pytest.mark.parametrize("s_x", [0.0, 0.02])
def test_many_maps_channels_first(pipe, N, C, H, W, s_x):
    """More tiles than the turning quantizer has workgroups, more images than a grid has rows, partial tiles: the layer on a
    channels-first input equals the one on the same input channels last, which no tile turns."""
    e = pipe.pipe_expand(dev(np.random.default_rng(C).standard_normal((C, 9)).astype(np.float32)), 4, 2, 0.5, 16)
    x = torch.randn((N, H, W, C), generator=torch.Generator().manual_seed(N))
    kw = dict(s_x=s_x, split=[1, 1], reduce_members=False)   # (two members: never the fused kernel)
    last = pipe.pipe_forward_depthwise2d(e, x.cuda(), 3, 3, 1, 1, nhwc=True, **kw)
    first = pipe.pipe_forward_depthwise2d(e, x.permute(0, 3, 1, 2).contiguous().cuda(), 3, 3, 1, 1, **kw)
    assert torch.equal(first, last)
    e.free()


@pytest.mark.parametrize("T,I,bits,s_x", [(16, 256, 8, 0.0), (15, 200, 4, 0.0), (5, 768, 2, 0.02), (2, 1020, 4, 0.0), (1, 4096, 2, 0.0),
                                          (1, 8192, 4, 0.0), (1, 68, 4, 0.0), (16, 4, 8, 0.0), (4, 1024, 3, 0.0)])
def test_quantizing_in_the_streaming_kernel_changes_nothing(pipe, T, I, bits, s_x):
    """Few codes: one launch instead of two, bit for bit (rows whose quads fill a wave and rows that do not)."""
    e = pipe.pipe_expand(dev(_weight(T * I, 112, I)), bits, 2, 1.0, 16)
    x = dev(np.random.default_rng(I + T).standard_normal((T, I)).astype(np.float32))
    y = pipe.pipe_forward(e, x, s_x=s_x)
    pipe.pipe_set_decode_fusion(False)
    try:
        ref = pipe.pipe_forward(e, x, s_x=s_x)
    finally:
        pipe.pipe_set_decode_fusion(True)
    assert torch.equal(y, ref)
    e.free()


@pytest.mark.parametrize("T", [9, 100, 700])
def test_hidden_maximum_wherever_it_lies(pipe, T):
    """The hidden tensor's largest value in the first, a middle and the last tokens and channels (another workgroup and line of its
    slot each time): the scale is that of the tensor, and the next call finds the slots cleared, also one of the other quantizer."""
    I, H = 256, 1040
    rng = np.random.default_rng(T)
    W1 = _weight(T + 1, H, I)
    l1, l2 = pipe.pipe_expand(dev(W1), 4, 4, 0.5, 16), pipe.pipe_expand(dev(_weight(T + 2, 64, H)), 4, 4, 0.5, 16)
    x0 = rng.standard_normal((T, I)).astype(np.float32)
    split, act = [2, 2], pipe.PIPE_ACT_GELU
    asym = lambda: pipe.pipe_mlp_forward_asymmetric(l1, l2, act, dev(x0), split=split)
    pipe.pipe_set_decode_resident(0)
    try:
        before = asym()
        for t, c in ((0, 0), (T // 2, 517), (T - 1, H - 1), (T // 3, 300), (T - 1, 16)):
            x = x0.copy()
            x[t] = 4 * W1[c] / np.abs(W1[c]).max()      # the row of W1 it meets answers loudest or nearly so
            y, h = pipe.pipe_mlp_forward(l1, l2, act, dev(x), s_x=0.05, split=split, return_hidden=True)
            sh = [float(np.float32(h[m].abs().max().item()) / np.float32(127)) for m in range(2)]
            assert torch.equal(y, pipe.pipe_mlp_forward_given_scales(l1, l2, act, dev(x), 0.05, sh, split=split))
            assert torch.equal(before, asym())
    finally:
        pipe.pipe_set_decode_resident(1)
    l1.free(), l2.free()


#            O     I    bits K gamma split   T  act: three or four workgroups of 64-token tiles share a compute unit (256 of them assumed)
OCCUPANCY = [(4096, 256, 2, 1, 1.0, [1], 4096, "plain"),     # 1024 tiles: one round of four
             (4096, 64, 4, 1, 1.0, [1], 4095, "plain"),      # an odd number of stages, a ragged last tile
             (4096, 320, 4, 1, 1.0, [1], 3072, "plain"),     # 768: one round of three
             (4096, 200, 2, 2, 0.5, [1, 1], 3000, "plain"),  # members apart, pruned row blocks
             (4112, 260, 4, 1, 1.0, [1], 4000, "gelu"), (4096, 260, 2, 1, 1.0, [1], 3100, "gelu"), (4128, 130, 4, 2, 0.5, [2], 4095, "gated")]


@pytest.mark.parametrize("O,I,bits,K,gamma,split,T,act", OCCUPANCY)
def test_workgroups_per_unit_change_nothing(pipe, O, I, bits, K, gamma, split, T, act):
    """Many 64-token tiles, served by the variant with one register set of fragments or by the one with two: 32-token tiles (other
    loops) give the same bits."""
    rng = np.random.default_rng(O + T)
    l1, l2 = pipe.pipe_expand(dev(_weight(O + I, O, I)), bits, K, gamma, 16), None
    x = dev(rng.standard_normal((T, I)).astype(np.float32))
    b = dev(rng.standard_normal(O).astype(np.float32))
    if act == "plain":
        call = lambda: pipe.pipe_forward(l1, x, s_x=0.03, split=split, bias=b, reduce_members=len(split) == 1)
    else:
        l2 = pipe.pipe_expand(dev(_weight(O, 16, O if act == "gelu" else O // 2)), bits, K, gamma, 16)
        kind = pipe.PIPE_ACT_GELU if act == "gelu" else pipe.PIPE_ACT_SILU_GATED
        call = lambda: pipe.pipe_mlp_forward(l1, l2, kind, x, s_x=0.03, split=split, bias1=b, return_hidden=True)[1]
    got = {}
    for tile in (0, 32, 64):
        pipe.pipe_set_token_tile(tile)
        try:
            got[tile] = call()
        finally:
            pipe.pipe_set_token_tile(0)
    assert torch.equal(got[0], got[32]) and torch.equal(got[64], got[32])
    l1.free()
    if l2 is not None:
        l2.free()


@pytest.mark.parametrize("scale", [0.05, 1.0, 2.0, 6.0])
def test_gelu_values(pipe, scale):
    """GELU of every size of argument, as the hidden tensor of an MLP whose first layer is an identity (codes of one order, their
    scale a power of two): against 64 bits, within the approximation's error of 1.8e-8 in erfc and the roundings on the way to it -- four in the
    exponent, v Q(v) = -log2 erfc, and two in its power -- times |a| / 2, and one of the result.  (0.5 a (1 + erff) leaves this
    bound in the negative tail, where it cancels.)"""
    T, I = 200, 256
    l1 = pipe.pipe_expand(dev(np.eye(I, dtype=np.float32) * np.float32(127)), 8, 1, 1.0, 16)   # weights 127 = code 127 x scale 1
    l2 = pipe.pipe_expand(dev(_weight(1, 16, I)), 8, 1, 1.0, 16)
    s = 2.0 ** np.round(np.log2(scale / 40)) / 127
    codes = np.random.default_rng(7).integers(-127, 128, size=(T, I)).astype(np.float64)
    x = dev((codes * np.float32(s)).astype(np.float32))
    y, h = pipe.pipe_mlp_forward(l1, l2, pipe.PIPE_ACT_GELU, x, s_x=float(np.float32(s)), split=[1], return_hidden=True)
    a = torch.from_numpy((codes * 127 * np.float64(np.float32(s))).astype(np.float32)).double()
    erfc = torch.special.erfc(a.abs() / 2 ** 0.5)
    ref = 0.5 * a * torch.special.erfc(-a / 2 ** 0.5)
    bound = 0.5 * a.abs() * (1.8e-8 + erfc * (2.0 ** -22 * -erfc.log().clamp(min=-700.) + 2.0 ** -23)) + 2.0 ** -24 * ref.abs() + 5e-15
    err = (h.view(T, I).cpu().double() - ref).abs()
    print("scale", scale, "largest error over its bound", float((err / bound).max()))
    assert bool((err <= bound).all()), float((err / bound).max())
    l1.free(), l2.free()


@pytest.mark.parametrize("T", [40, 200])   # the streaming kernel, the single-pass one
def test_gelu_of_infinities(pipe, T):
    I = 256
    l1, l2 = pipe.pipe_expand(dev(_weight(2, I, 64)), 8, 1, 1.0, 16), pipe.pipe_expand(dev(_weight(1, 16, I)), 8, 1, 1.0, 16)
    b = np.zeros(I, dtype=np.float32)
    b[3], b[70], b[200], b[201], b[202] = np.inf, -np.inf, np.nan, 3e38, -3e38
    x = dev(np.random.default_rng(T).standard_normal((T, 64)).astype(np.float32))
    y, h = pipe.pipe_mlp_forward(l1, l2, pipe.PIPE_ACT_GELU, x, s_x=0.03, split=[1], bias1=dev(b), return_hidden=True)
    h = h.view(T, I)
    assert bool((h[:, 3] == np.inf).all()) and bool(torch.isnan(h[:, [70, 200]]).all())    # (minus infinity times zero, as in the direct form)
    assert bool((h[:, 201] == np.float32(3e38)).all()) and bool((h[:, 202].abs() <= 5e-15).all())
    rest = [c for c in range(I) if c not in (3, 70, 200)]
    assert bool(torch.isfinite(h[:, rest]).all())
    l1.free(), l2.free()


# Two groups along k and two stages ahead in the other epilogues and for convolutions: the sums are exact integers, so the height that is set by
# hand, which runs with one of each, gives the same bits.  nks = 28 and 36 steps; the convolutions have one tap a stage or several.
@pytest.mark.parametrize("kind,T,C,k", [("gelu", 300, 1696, 0), ("gated", 300, 1696, 0), ("chain", 300, 1696, 0), ("chain", 1100, 1696, 0), ("chain", 13000, 512, 0), ("chain2", 13000, 512, 0),
                                        ("conv", 3, 256, 3), ("conv", 30, 256, 3), ("conv", 3, 64, 5), ("conv8", 40, 256, 3), ("conv2", 3, 256, 3),
                                        ("conv", 12, 256, 3), ("conv", 30, 192, 3), ("conv", 60, 256, 3), ("conv", 60, 64, 5), ("conv8", 3, 256, 3), ("conv8", 12, 64, 5), ("conv8", 40, 192, 3),
                                        ("conv2", 12, 256, 3), ("conv2", 30, 64, 5), ("conv2", 60, 512, 3), ("gated", 500, 1696, 0)])
def test_two_groups_equal_one(pipe, kind, T, C, k):
    rng = np.random.default_rng(T + C)
    made = []

    def expand(O, I, bits=4):
        made.append(pipe.pipe_expand(dev(_weight(O + I, O, I)), bits, 3, 0.5, 16))
        return made[-1]

    if kind in ("gelu", "gated"):
        act = pipe.PIPE_ACT_GELU if kind == "gelu" else pipe.PIPE_ACT_SILU_GATED
        l1, l2 = expand(512 if kind == "gelu" else 3200, C), expand(1008, 512 if kind == "gelu" else 1600)
        x = dev(rng.standard_normal((T, C)).astype(np.float32))
        call = lambda: pipe.pipe_mlp_forward(l1, l2, act, x, split=[2, 1], bias1=None, bias2=None, return_hidden=True)
    elif kind in ("chain", "chain2"):   # (816 to 1020 tiles of 64 tokens: four workgroups per compute unit)
        R = pipe.PIPE_ACT_RELU
        bits = 4 if kind == "chain" else 2
        layers = [(expand(C, C, bits), None, R, -1, True), (expand(C, C, bits), None, R, 0, True), (expand(304, C, bits), None, pipe.PIPE_ACT_NONE, -1, True)]
        x = dev(rng.standard_normal((T, C)).astype(np.float32))
        call = lambda: (pipe.pipe_chain_forward(layers, x, split=[2, 1]),)
    else:
        bits = {"conv": 4, "conv8": 8, "conv2": 2}[kind]
        e = pipe.pipe_expand_conv2d(dev(_weight(C, 256, C * k * k)), C, k, k, bits, 3, 0.5, 16)
        made.append(e)
        x = dev(rng.standard_normal((T, C, 14, 13)).astype(np.float32))
        call = lambda: (pipe.pipe_forward_conv2d(e, x, k, k, 1, k // 2, split=[3]),)
    got = call()
    for tile in (16, 32, 64):
        pipe.pipe_set_token_tile(tile)
        try:
            one = call()
        finally:
            pipe.pipe_set_token_tile(0)
        for a, b in zip(got, one):
            assert torch.equal(a, b), "token tile %d" % tile
    for e in made:
        e.free()


# The sum over two members with inputs of their own, a launch per member: second layers of 48 steps and more, in every height and with one and two
# groups, with row blocks that the second member pruned.  Both kernels add the same exact integers in the same order.
@pytest.mark.parametrize("bits,out,hidden,K,gamma,split,T,bias",
                         [(4, 48, 3072, 4, 0.34, [2, 2], 129, True), (4, 1040, 3100, 4, 0.1, [2, 2], 300, False),
                          (4, 1040, 3100, 3, 0.25, [2, 1], 300, True), (4, 4096, 3100, 4, 0.5, [2, 2], 500, True),
                          (4, 2048, 3080, 4, 0.1, [2, 2], 1000, True), (4, 4096, 3080, 2, 1.0, [1, 1], 800, False),
                          (2, 512, 3072, 4, 0.25, [2, 2], 200, True), (2, 4096, 3072, 4, 0.5, [2, 2], 700, False),
                          (8, 1024, 3072, 4, 0.5, [2, 2], 150, True), (8, 2048, 3072, 4, 0.25, [2, 2], 900, False),
                          # (the one of three orders above stays pass by pass; these have 200 tiles and more of the single order)
                          (4, 4096, 3080, 3, 0.5, [2, 1], 1540, True), (2, 4096, 3072, 3, 0.5, [2, 1], 1540, False), (8, 4096, 3072, 3, 0.5, [2, 1], 1540, True)])
def test_sum_over_members_equals_its_parts(pipe, bits, out, hidden, K, gamma, split, T, bias):
    rng = np.random.default_rng(out + T)
    hidden -= hidden % 16
    l1 = pipe.pipe_expand(dev(_weight(out, hidden, 64)), bits, K, 1.0, 16)
    l2 = pipe.pipe_expand(dev(_weight(out + 1, out, hidden)), bits, K, gamma, 16)
    x = dev(rng.standard_normal((T, 64)).astype(np.float32))
    b2 = dev(rng.standard_normal(out).astype(np.float32)) if bias else None
    call = lambda v: pipe.pipe_mlp_forward_given_scales(l1, l2, pipe.PIPE_ACT_GELU, v, 0.03, [0.01, 0.003], split=split, bias2=b2,
                                                        return_hidden=True)
    y, h = call(x)
    parts = [call(x[a:z].contiguous()) for a, z in _parts(T)]
    assert torch.equal(h, torch.cat([p[1] for p in parts], dim=1))
    assert torch.equal(y, torch.cat([p[0] for p in parts], dim=0))
    l1.free(), l2.free()


# A member's infinite scale reaches only the row blocks that it has orders of: those that the second member pruned keep the first one's sum, in a
# tile of their own (with a bias) or beside others' items.  One and two groups along k.
@pytest.mark.parametrize("bias", [False, True])
@pytest.mark.parametrize("bits,out,hidden,T", [(4, 1040, 3104, 300), (2, 4096, 3072, 700), (8, 2048, 3072, 900)])
def test_infinite_member_scale_leaves_pruned_row_blocks(pipe, bits, out, hidden, T, bias):
    rng = np.random.default_rng(out + T)
    l1 = pipe.pipe_expand(dev(_weight(out, hidden, 64)), bits, 4, 1.0, 16)
    l2 = pipe.pipe_expand(dev(_weight(out + 1, out, hidden)), bits, 4, 0.25, 16)
    x = dev(rng.standard_normal((T, 64)).astype(np.float32))
    b2 = dev(rng.standard_normal(out).astype(np.float32)) if bias else None
    call = lambda s_h: pipe.pipe_mlp_forward_given_scales(l1, l2, pipe.PIPE_ACT_GELU, x, 0.03, s_h, split=[2, 2], bias2=b2)
    kept = np.zeros(out // 16, dtype=bool)
    for k in (3, 4):
        kept[l2.order(k)[0]] = True
    rows = torch.from_numpy(np.repeat(~kept, 16)).to("cuda:0")
    assert 0 < int(rows.sum()) < out
    finite, infinite = call([0.01, 0.003]), call([0.01, float("inf")])
    assert bool(torch.isfinite(finite).all())
    assert torch.equal(infinite[:, rows], finite[:, rows])
    assert not bool(torch.isfinite(infinite[:, ~rows]).any())      # (codes of zero times infinity)
    l1.free(), l2.free()


@pytest.mark.parametrize("kind,T", [("linear", 17), ("linear", 64), ("linear", 65), ("linear", 128), ("asymmetric", 40), ("gelu", 64), ("gelu", 65),
                                    ("gated", 64), ("gated", 65), ("narrow", 65), ("gated21", 113), ("chain", 65), ("chain4", 128), ("chain8", 65), ("deep8", 65)])
def test_batches_of_17_to_128_tokens_by_either_kernel(pipe, kind, T):
    """Calls on either side of the lines between the tiled kernels and the streaming kernel, against the latter, bit for bit; and captured where only
    the streaming kernel is ready (its scratch, no tile schedules), replayed with other inputs."""
    g = torch.Generator(device="cuda")
    g.manual_seed(T)
    mk = lambda o, i, bits, K, group=16: pipe.pipe_expand(torch.randn(o, i, generator=g, device="cuda") * (1.5 / i ** 0.5), bits, K, 0.5, group)
    wide = 1552 if kind in ("chain", "chain4") else 320
    xs = [torch.randn(T, wide, generator=g, device="cuda") * s for s in (1.0, 3.0)]
    x = xs[0].clone()
    if kind in ("linear", "asymmetric"):
        es = [mk(8192, 320, 4, 4)]          # 320 bins: 17 tokens are past the line
        call = (lambda: pipe.pipe_forward(es[0], x)) if kind == "linear" else (lambda: pipe.pipe_forward_asymmetric(es[0], x))
    elif kind in ("gelu", "gated", "narrow", "gated21"):
        up = 2 if kind != "gelu" else 1
        K, split = {"gelu": (3, None), "gated": (4, [2, 2]), "narrow": (4, [2, 2]), "gated21": (3, [2, 1])}[kind]
        hidden = 480 if kind == "narrow" else 1088
        es = [mk(up * hidden, 320, 4, K), mk(320, hidden, 4, K)]
        act = pipe.PIPE_ACT_GELU if kind == "gelu" else pipe.PIPE_ACT_SILU_GATED
        call = lambda: pipe.pipe_mlp_forward(es[0], es[1], act, x, split=split)
    else:
        K, split, L = {"chain": (4, [2, 2], 3), "chain4": (4, None, 3), "chain8": (8, [4, 4], 3), "deep8": (8, [4, 4], 4)}[kind]
        es = [mk(wide, wide, 2, K) for _ in range(L)]
        layers = [(e, None, 0 if l == L - 1 else 3, 1 if l == 1 else -1, True) for l, e in enumerate(es)]
        call = lambda: pipe.pipe_chain_forward(layers, x, split=split)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    pipe.pipe_set_kernel(2)
    try:
        with torch.cuda.stream(side):       # sizes the streaming kernel's scratch there
            streamed = []
            for v in xs:
                x.copy_(v)
                streamed.append(call().clone())
    finally:
        pipe.pipe_set_kernel(0)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        out = call()
    for rep in range(4):
        x.copy_(xs[rep % 2])
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, streamed[rep % 2]), rep
    for v, want in zip(xs, streamed):       # eager: the rule's route
        x.copy_(v)
        assert torch.equal(call(), want)
    for e in es:
        e.free()


@pytest.mark.parametrize("T,n_in,out,K", [(17, 60, 48, 2), (33, 700, 336, 3), (128, 768, 1008, 4), (20, 1100, 64, 1), (64, 1536, 320, 2), (97, 1540, 176, 4),
                                          (40, 2300, 96, 3), (100, 11008, 64, 2), (16, 520, 16384, 4), (7, 8192, 12288, 4), (1, 8192, 2048, 4), (1, 4100, 2064, 4),
                                          (1, 252, 20512, 4), (1, 5000, 2064, 4), (100, 2300, 96, 6), (3, 5000, 160, 12), (17, 60, 48, 16)])
def test_streamed_8_bit_walks_by_two_tiles(pipe, T, n_in, out, K):
    """8-bit layers whose waves walk no tile, one, an odd or an even number of them, by two at a time: outputs and accumulators bit for bit those of
    the tiled kernels, accumulators the whole numbers of the codes."""
    g = torch.Generator(device="cuda")
    g.manual_seed(T + n_in)
    e = pipe.pipe_expand(torch.randn(out, n_in, generator=g, device="cuda") / n_in ** 0.5, 8, K, 1.0, 16)
    x = torch.randn(T, n_in, generator=g, device="cuda")
    got = []
    try:
        for which in (2, 1):
            pipe.pipe_set_kernel(which)
            got.append((pipe.pipe_forward(e, x),) + tuple(pipe.pipe_forward_acc(e, x)))
    finally:
        pipe.pipe_set_kernel(0)
    for a, b in zip(*got):
        assert torch.equal(a, b)
    acc, qx = got[0][1], got[0][2]
    if n_in * out <= 1 << 20:
        for k in range(K):
            codes = np.asarray(e.order(k + 1)[2]).astype(np.float64)
            assert np.array_equal(acc[k].cpu().numpy(), qx.cpu().numpy().astype(np.float64) @ codes.T)    # (whole numbers below 2^53)
    e.free()


@pytest.mark.parametrize("bits,T,n_in,scale,static", [(2, 1, 8192, 1.0, 0.0), (4, 1, 8188, 1.0, 0.0), (8, 1, 4, 1.0, 0.02), (4, 16, 252, 1.0, 0.0), (2, 3, 1028, 1.0, 0.0),
                                                      (8, 4, 1024, 1.0, 0.01), (4, 15, 20, 1.0, 0.0), (4, 2, 2048, 1e-30, 0.0), (2, 5, 516, 1e30, 0.0), (8, 16, 256, 0.0, 0.0)])
def test_streaming_kernel_quantizes_its_tokens(pipe, bits, T, n_in, scale, static):
    """Codes from the streaming kernel's own quantizer against the launch of its own, bit for bit: the largest input, quads that end a row or the
    batch inside a wave, one quad, scales beyond the short division's range, NaN and infinities under a given scale."""
    g = torch.Generator(device="cuda")
    g.manual_seed(T + n_in)
    e = pipe.pipe_expand(torch.randn(176, n_in, generator=g, device="cuda") / n_in ** 0.5, bits, 2, 0.5, 16)   # bins past a group of eight
    x = torch.randn(T, n_in, generator=g, device="cuda") * scale
    if static > 0:
        x[0, 0], x[-1, -1], x[0, 1] = float("nan"), float("inf"), -float("inf")
    try:
        pipe.pipe_set_decode_fusion(False)
        want = pipe.pipe_forward(e, x, s_x=static)
    finally:
        pipe.pipe_set_decode_fusion(True)
    assert torch.equal(pipe.pipe_forward(e, x, s_x=static), want)
    assert bool(torch.isfinite(want).all())
    e.free()
