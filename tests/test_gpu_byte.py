"""GPU parity of the byte kernel (tables that are an exact product plus an error of one byte) against the CPU oracle: every
sum bit-exact, at the edges of its tiles, runs and slices, and of what counts as such a table."""
import numpy as np
import pytest
import torch

import oracle as orc
from paper_2203_04071_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2203_04071_amd import binding
    binding.load()
    assert torch.cuda.is_available()
    return binding


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    return t.detach().cpu().numpy()


def table(kind, bits, rng):
    """A table with a byte form (the whole byte in use), or one that misses it by one."""
    h = 1 << (bits - 1)
    v = np.arange(-h, h, dtype=np.int64)
    n = 2 * h
    if kind == "product":           # exact product + an error that spans 255
        t = v[:, None] * v[None, :] + rng.integers(-77, 179, size=(n, n))
        t[0, 0], t[-1, -1] = h * h - 77, (h - 1) ** 2 + 178
    elif kind == "dropped":         # both operands lose low bits
        d = min(2, bits - 1)
        t = ((v >> d) << d)[:, None] * ((v >> d) << d)[None, :] + rng.integers(-9, 10, size=(n, n))
    elif kind == "one_side":        # only the activation loses bits
        t = ((v >> 1) << 1)[:, None] * v[None, :] + rng.integers(-100, 101, size=(n, n))
    elif kind in ("bare", "bare_activation"):       # dropped bits change no entry: activations that differ in them share a table line
        d = 2 if bits > 3 else 1
        t = ((v >> d) << d)[:, None] * (((v >> d) << d) if kind == "bare" else v)[None, :] + rng.integers(-100, 101, size=(n, n))[(np.arange(n) >> d) << d]
    elif kind.startswith("share"):  # 2^d activations share a line, and no product that keeps more of an activation leaves a byte
        d = int(kind[-1])
        t = rng.integers(-77, 179, size=(n, n))[(np.arange(n) >> d) << d]
        t[:1 << d, 0], t[:1 << d, h] = 178, -77     # (it would add up to h times the lost bits to the first and nothing to the second: beyond 255)
        t = ((v >> d) << d)[:, None] * v[None, :] + t
    else:                           # spans 256: no byte form
        t = v[:, None] * v[None, :] + rng.integers(-128, 128, size=(n, n))
        t[0, 0], t[-1, -1] = h * h - 128, (h - 1) ** 2 + 128
    return np.ascontiguousarray(np.clip(t, -32768, 32767).astype(np.int32))


CONVS = [
    # N, Cin, H, W, Cout, kh, kw, sh, sw, ph, pw, dh, dw
    (1, 1, 1, 1, 1, 1, 1, 1, 1, 0, 0, 1, 1),            # one lookup
    (2, 3, 9, 9, 15, 3, 3, 1, 1, 1, 1, 1, 1),           # one channel group per tap, packed over taps; one tile less one channel
    (3, 5, 8, 13, 17, 3, 3, 2, 2, 1, 1, 1, 1),          # two groups per tap, odd width, stride 2, one tile and one channel
    (2, 13, 10, 7, 33, 5, 3, 1, 3, 2, 1, 1, 1),         # horizontal stride 3
    (2, 20, 12, 14, 16, 3, 3, 1, 2, 2, 2, 2, 2),        # dilation with stride 2
    (1, 64, 8, 8, 64, 3, 3, 1, 1, 1, 1, 1, 1),          # few pixels: slices of the inner dimension
    (1, 100, 7, 7, 40, 3, 3, 1, 1, 1, 1, 1, 1),         # the same with a ragged last step
    (9, 16, 32, 33, 32, 1, 1, 1, 1, 0, 0, 1, 1),        # one step, several row tiles
    (40, 24, 28, 30, 48, 3, 3, 1, 1, 1, 1, 1, 1),       # many pixels, runs that end inside a row
]


@pytest.mark.parametrize("bits,kind", [(8, "product"), (8, "dropped"), (8, "beyond"), (7, "product"), (6, "one_side"), (5, "product"),
                                       (4, "product"), (3, "product"), (2, "product")])
@pytest.mark.parametrize("case", CONVS)
def test_convolution(B, bits, kind, case):
    N, Cin, H, W, Cout, kh, kw, sh, sw, ph, pw, dh, dw = case
    rng = np.random.default_rng(1000 * bits + sum(case))
    lut = table(kind, bits, rng)
    L = B.Lut(lut, bits)
    x = wl.random_i8(rng, (N, Cin, H, W), bits)         # uniform over all codes, the most negative included
    w = wl.random_i8(rng, (Cout, Cin, kh, kw), bits)
    pw_ = B.adapt_weights_pack_conv2d(L, dev(w))
    want = orc.approx_conv2d(lut, bits, x, w, (sh, sw), (ph, pw), (dh, dw), threads=4)
    for _ in range(2):              # (the second call finds the arrival counters as the first left them)
        got = host(B.adapt_approx_conv2d_packed(pw_, dev(x), (sh, sw), (ph, pw), (dh, dw)))
        assert got.shape == want.shape and (got == want).all()
    plain = host(B.adapt_approx_conv2d(L, dev(x), dev(w), (sh, sw), (ph, pw), (dh, dw)))
    assert (plain == want).all()


@pytest.mark.parametrize("bits,kind", [(8, "product"), (8, "dropped"), (7, "product"), (6, "one_side")])
@pytest.mark.parametrize("images,hw,steps", [(1, 12, range(1, 10)), (9, 64, range(1, 6)), (8, 256, (1, 2, 3, 5))])
def test_every_remainder_of_a_group_of_steps(B, bits, kind, images, hw, steps):
    """1 x 1 layers of 1, 2, .. steps of 16 inner indices (the last one ragged): the exact product takes them in pairs, copies and
    activations in groups of four; few, more and many pixels, so that all numbers of pixels per row slot occur."""
    rng = np.random.default_rng(17 * bits + images)
    h = 1 << (bits - 1)
    t = table(kind, bits, rng)
    lut = B.Lut(t, bits)
    for s in steps:
        cin = 16 * s - 3 * (s % 2)
        x = rng.integers(-h, h, size=(images, cin, hw, hw)).astype(np.int8)
        w = rng.integers(-h, h, size=(16, cin, 1, 1)).astype(np.int8)
        pw = B.adapt_weights_pack_conv2d(lut, dev(w))
        got = host(B.adapt_approx_conv2d_packed(pw, dev(x), (1, 1), (0, 0)))
        assert np.array_equal(got, orc.approx_conv2d(t, bits, x, w, (1, 1), (0, 0))), s


@pytest.mark.parametrize("bits", [6, 8])
@pytest.mark.parametrize("shape", [(4096, 1, 1), (4097, 15, 17), (4099, 130, 33), (9000, 64, 16), (5000, 517, 100)])
def test_linear(B, bits, shape):
    M, K, N = shape
    rng = np.random.default_rng(bits + sum(shape))
    lut = table("product", bits, rng)
    L = B.Lut(lut, bits)
    a, w = wl.random_i8(rng, (M, K), bits), wl.random_i8(rng, (N, K), bits)
    want = orc.approx_linear(lut, bits, a, w, threads=4)
    pw = B.adapt_weights_pack_linear(L, dev(w))
    assert (host(B.adapt_approx_linear_packed(pw, dev(a))) == want).all()
    assert (host(B.adapt_approx_linear(L, dev(a), dev(w))) == want).all()


@pytest.mark.parametrize("bits", [6, 8])
@pytest.mark.parametrize("case", [(3, 7, 5, 6, 9, 4, 2, 1), (2, 20, 4, 4, 33, 2, 2, 0), (1, 33, 3, 7, 16, 3, 3, 0), (2, 16, 9, 5, 17, 3, 1, 1)])
def test_transposed_convolution(B, bits, case):
    N, Cin, H, W, Cout, k, st, pad = case
    rng = np.random.default_rng(bits + sum(case))
    lut = table("product", bits, rng)
    L = B.Lut(lut, bits)
    x, w = wl.random_i8(rng, (N, Cin, H, W), bits), wl.random_i8(rng, (Cin, Cout, k, k), bits)
    pw = B.adapt_weights_pack_conv_transpose2d(L, dev(w), st)
    want = orc.approx_conv_transpose2d(lut, bits, x, w, st, pad, threads=4)
    assert (host(B.adapt_approx_conv_transpose2d_packed(pw, dev(x), pad)) == want).all()


@pytest.mark.parametrize("bits", [6, 8])
@pytest.mark.parametrize("stride,kind", [(1, "product"), (2, "product"), (2, "beyond")])
def test_chain_into_a_strided_layer(B, bits, stride, kind):
    """The copy a producer writes for a layer that moves by `stride` pixels, behind a ReLU (half of every table) and without,
    between handles with and without a byte form."""
    rng = np.random.default_rng(bits + stride)
    lut1, lut2 = table("product", bits, rng), table(kind, bits, rng)
    L1, L2 = B.Lut(lut1, bits), B.Lut(lut2, bits)
    x = dev(rng.standard_normal((3, 6, 11, 13)).astype(np.float32))
    w1, w2 = wl.random_i8(rng, (18, 6, 3, 3), bits), wl.random_i8(rng, (21, 18, 3, 3), bits)
    p1, p2 = B.adapt_weights_pack_conv2d(L1, dev(w1)), B.adapt_weights_pack_conv2d(L2, dev(w2))
    s_x, s_1, s_2, s_o = 0.05, 1e-3, 0.3, 1e-3
    B.adapt_conv2d_chain_prepare(p2, 3, 11, 13, (stride, stride), (1, 1))
    for act in (B.ACT_RELU, B.ACT_NONE, B.ACT_RELU):
        y1 = B.adapt_conv2d_layer_f32(p1, x, s_x, s_1, (1, 1), (1, 1), act=act)
        want = B.adapt_dequant_i32(B.adapt_approx_conv2d(L2, B.adapt_quantize_f32(y1, s_2, bits), dev(w2), (stride, stride), (1, 1)), s_o, 1, 1, 3 * 21 * (-(-11 // stride)) * (-(-13 // stride)))
        out1, out2 = torch.empty_like(y1), torch.empty_like(want)
        B.adapt_conv2d_layer_chain_f32(p1, x, s_x, s_1, out1, (1, 1), (1, 1), act=act, next_pw=p2, s_next=s_2)
        B.adapt_conv2d_layer_chain_f32(p2, None, s_2, s_o, out2, (stride, stride), (1, 1), in_shape=(3, 11, 13))
        assert torch.equal(out1, y1) and torch.equal(out2, want)


@pytest.mark.parametrize("M,K,N,bits", [(512, 777, 37, 8), (1111, 130, 999, 8), (16, 4096, 17, 7), (4095, 33, 48, 6), (4095, 40, 250, 5)])
def test_linear_layers_below_4096_rows(B, M, K, N, bits):
    """Whichever kernel the estimate picks: sums of packed and plain weights, and the fused layer, bit-exact; a recorded first
    call (which may not allocate) too."""
    rng = np.random.default_rng(M + K)
    t = table("product", bits, rng)
    L = B.Lut(t, bits)
    h = 1 << (bits - 1)
    a, w = rng.integers(-h, h, size=(M, K)).astype(np.int8), rng.integers(-h, h, size=(N, K)).astype(np.int8)
    want = orc.approx_linear(t, bits, a, w)
    ad, wd = dev(a), dev(w)
    assert (host(B.adapt_approx_linear(L, ad, wd)) == want).all()
    pw = B.adapt_weights_pack_linear(L, wd)
    out = torch.zeros((M, N), dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        B.adapt_approx_linear_packed(pw, ad, out=out)
    for _ in range(3):
        out.zero_()
        g.replay()
        assert (host(out) == want).all()
    assert (host(B.adapt_approx_linear_packed(pw, ad)) == want).all()
    x = (a.astype(np.float32) * np.float32(0.25))
    y = B.adapt_linear_layer_f32(pw, dev(x), 0.25, 0.5)
    q = orc.quantize(x, np.float32(0.25), bits)
    assert np.array_equal(host(y).view(np.uint32), orc.dequant(orc.approx_linear(t, bits, q, w), np.float32(0.5), M, N, 1).reshape(M, N).view(np.uint32))


@pytest.mark.parametrize("bits", [8, 7])
@pytest.mark.parametrize("images,cin,cout,hw,stride", [(50, 20, 200, 27, 2), (24, 36, 140, 20, 1), (40, 33, 72, 14, 1),
                                                       (8, 36, 140, 20, 1), (6, 33, 72, 14, 1), (4, 17, 40, 14, 1), (9, 5, 523, 28, 1)])
def test_channel_tiles_that_no_power_of_two_divides(B, bits, images, cin, cout, hw, stride):
    """13, 9, 5, 3 and 33 channel tiles with several row tiles: where these are few, or the channel tiles many, workgroups are dealt to the XCDs by
    the tables they read (some XCDs have none), elsewhere in the usual order."""
    rng = np.random.default_rng(bits + cout)
    t = table("product", bits, rng)
    x, w = wl.random_i8(rng, (images, cin, hw, hw), bits), wl.random_i8(rng, (cout, cin, 3, 3), bits)
    pw = B.adapt_weights_pack_conv2d(B.Lut(t, bits), dev(w))
    want = orc.approx_conv2d(t, bits, x, w, (stride, stride), (1, 1), threads=4)
    for _ in range(2):
        assert (host(B.adapt_approx_conv2d_packed(pw, dev(x), (stride, stride), (1, 1))) == want).all()


@pytest.mark.parametrize("K", [32640, 32641])
def test_longest_inner_dimension(B, K):
    """The last length whose group offsets fit, and the first that takes the other tables."""
    rng = np.random.default_rng(K)
    t = table("product", 6, rng)
    L = B.Lut(t, 6)
    a, w = wl.random_i8(rng, (4100, K), 6), wl.random_i8(rng, (3, K), 6)
    pw = B.adapt_weights_pack_linear(L, dev(w))
    assert (host(B.adapt_approx_linear_packed(pw, dev(a))) == orc.approx_linear(t, 6, a, w, threads=4)).all()


@pytest.mark.parametrize("sw", [7, 1 << 26, (1 << 31) - 1])
def test_one_output_column_under_any_stride(B, sw):
    """The horizontal stride does not matter where the window never moves: packed and plain weights, and a chained input."""
    rng = np.random.default_rng(sw)
    t = table("product", 7, rng)
    L = B.Lut(t, 7)
    x, w = wl.random_i8(rng, (64, 5, 66, 6), 7), wl.random_i8(rng, (9, 5, 3, 5), 7)
    want = orc.approx_conv2d(t, 7, x, w, (1, 7), (0, 0), (1, 1), threads=4)
    assert want.shape == (64, 9, 64, 1)
    pw = B.adapt_weights_pack_conv2d(L, dev(w))
    assert (host(B.adapt_approx_conv2d_packed(pw, dev(x), (1, sw), (0, 0))) == want).all()
    assert (host(B.adapt_approx_conv2d(L, dev(x), dev(w), (1, sw), (0, 0))) == want).all()
    w1 = wl.random_i8(rng, (5, 5, 1, 1), 7)
    p1 = B.adapt_weights_pack_conv2d(L, dev(w1))
    B.adapt_conv2d_chain_prepare(pw, 64, 66, 6, (1, sw), (0, 0))
    xf = dev(x.astype(np.float32))
    y1 = B.adapt_conv2d_layer_f32(p1, xf, 1.0, 0.01)
    ref = B.adapt_conv2d_layer_f32(pw, y1, 0.5, 0.1, (1, sw))
    out1, out2 = torch.empty_like(y1), torch.empty_like(ref)
    B.adapt_conv2d_layer_chain_f32(p1, xf, 1.0, 0.01, out1, next_pw=pw, s_next=0.5)
    B.adapt_conv2d_layer_chain_f32(pw, None, 0.5, 0.1, out2, (1, sw), in_shape=(64, 66, 6))
    assert torch.equal(out1, y1) and torch.equal(out2, ref)


def test_activation_copy_beyond_two_gigabytes(B):
    """8 channels under stride 2 on three columns: an input of just under 2^31 elements, whose copy takes four words per row and
    channel group.  Compared with the same layer on parts of the batch; the copy a producer writes, too."""
    N, H = 8000, 11180
    assert N * H * 3 * 8 < 0x7fffff00 < N * H * 4 * 8
    gen = torch.Generator(device="cuda").manual_seed(1)
    x = torch.randint(-128, 128, (N, 8, H, 3), generator=gen, device="cuda", dtype=torch.int8)
    w = torch.randint(-128, 128, (1, 8, 1, 1), generator=gen, device="cuda", dtype=torch.int8)
    L = B.Lut(table("product", 8, np.random.default_rng(1)), 8)
    pw = B.adapt_weights_pack_conv2d(L, w)
    got = B.adapt_approx_conv2d_packed(pw, x, (1, 2))
    for n in (0, 3999, N - 500):
        assert torch.equal(got[n:n + 500], B.adapt_approx_conv2d(L, x[n:n + 500], w, (1, 2)))
    # the input as a layer's output: 1 channel -> 8 channels, written into the copy alone
    del x, got
    p1 = B.adapt_weights_pack_conv2d(L, torch.randint(-128, 128, (8, 1, 1, 1), generator=gen, device="cuda", dtype=torch.int8))
    xf = torch.randn((N, 1, H, 3), generator=gen, device="cuda")
    B.adapt_conv2d_chain_prepare(pw, N, H, 3, (1, 2))
    B.adapt_conv2d_layer_chain_f32(p1, xf, 0.02, 1e-3, None, next_pw=pw, s_next=0.1)
    out = torch.empty((N, 1, H, 2), dtype=torch.float32, device="cuda")
    B.adapt_conv2d_layer_chain_f32(pw, None, 0.1, 1e-3, out, (1, 2), in_shape=(N, H, 3))
    for n in (0, 3999, N - 500):
        y = B.adapt_conv2d_layer_f32(p1, xf[n:n + 500], 0.02, 1e-3)
        assert torch.equal(out[n:n + 500], B.adapt_conv2d_layer_f32(pw, y, 0.1, 1e-3, (1, 2)))


@pytest.mark.parametrize("bits,kind", [(8, "product"), (7, "dropped"), (8, "beyond")])
def test_ordinary_call_between_a_relu_producer_and_a_chained_call(B, bits, kind):
    """A prepared handle that ran on its own input holds codes of both signs, whatever the producer before had said."""
    rng = np.random.default_rng(bits)
    t = table(kind, bits, rng)
    L = B.Lut(t, bits)
    p1 = B.adapt_weights_pack_conv2d(L, dev(wl.random_i8(rng, (16, 16, 1, 1), bits)))
    p2 = B.adapt_weights_pack_conv2d(L, dev(wl.random_i8(rng, (16, 16, 3, 3), bits)))
    x, x2 = (dev(rng.standard_normal((8, 16, 16, 16)).astype(np.float32)) for _ in range(2))
    out = torch.empty((8, 16, 16, 16), dtype=torch.float32, device="cuda")
    B.adapt_conv2d_chain_prepare(p2, 8, 16, 16, (1, 1), (1, 1))
    B.adapt_conv2d_layer_chain_f32(p1, x, 0.05, 1e-3, torch.empty_like(out), act=B.ACT_RELU, next_pw=p2, s_next=0.1)
    want = B.adapt_conv2d_layer_f32(p2, x2, 0.05, 1e-3, (1, 1), (1, 1))
    B.adapt_conv2d_layer_chain_f32(p2, None, 0.05, 1e-3, out, (1, 1), (1, 1), in_shape=(8, 16, 16))
    assert torch.equal(out, want)


def bits_equal(a, b):
    return np.array_equal(np.ascontiguousarray(a).view(np.uint32), np.ascontiguousarray(b).view(np.uint32))


FORMS = [(8, "product"), (8, "dropped"), (7, "dropped"), (8, "one_side"), (6, "one_side")]


def finish(acc, s_out, bias, resid, act):
    n, c, hw = acc.shape[0], acc.shape[1], int(np.prod(acc.shape[2:], dtype=np.int64))
    y = orc.dequant(acc, s_out, n, c, hw, bias).reshape(acc.shape)
    if resid is not None:
        y = orc.add(y, resid).reshape(acc.shape)
    return (orc.relu(y) if act == 1 else orc.tanh(y) if act == 2 else y).reshape(acc.shape)


@pytest.mark.parametrize("bits,kind", FORMS)
@pytest.mark.parametrize("act", [0, 1, 2])
def test_fused_layers_on_every_form(B, bits, kind, act):
    """Bias, residual, ReLU and tanh in the epilogue, tables whose exact product drops operand bits among them: a convolution with
    few pixels (slices) and one with ragged runs, a linear layer, a transposed convolution with border terms."""
    rng = np.random.default_rng(bits + act)
    t = table(kind, bits, rng)
    L = B.Lut(t, bits)
    s_x, s_out = np.float32(0.02), np.float32(2e-4)
    for N, Cin, H, W, Cout, k, st in ((1, 40, 8, 8, 24, 3, 1), (5, 7, 11, 13, 18, 3, 2), (40, 6, 20, 20, 16, 1, 1)):
        x, w = rng.standard_normal((N, Cin, H, W)).astype(np.float32), wl.random_i8(rng, (Cout, Cin, k, k), bits)
        acc = orc.approx_conv2d(t, bits, orc.quantize(x, s_x, bits), w, (st, st), (k // 2, k // 2), threads=4)
        bias, resid = rng.standard_normal(Cout).astype(np.float32), rng.standard_normal(acc.shape).astype(np.float32)
        pw = B.adapt_weights_pack_conv2d(L, dev(w))
        got = B.adapt_conv2d_layer_f32(pw, dev(x), s_x, s_out, (st, st), (k // 2, k // 2), bias=dev(bias), act=act, residual=dev(resid))
        assert bits_equal(host(got), finish(acc, s_out, bias, resid, act)), (Cin, Cout)
    x, w = rng.standard_normal((4097, 33)).astype(np.float32), wl.random_i8(rng, (21, 33), bits)
    acc, bias = orc.approx_linear(t, bits, orc.quantize(x, s_x, bits), w, threads=4), rng.standard_normal(21).astype(np.float32)
    got = B.adapt_linear_layer_f32(B.adapt_weights_pack_linear(L, dev(w)), dev(x), s_x, s_out, dev(bias), act)
    assert bits_equal(host(got), finish(acc, s_out, bias, None, act))
    assert (host(B.adapt_approx_linear(L, dev(orc.quantize(x, s_x, bits)), dev(w))) == acc).all()
    for N, Cin, H, W, Cout, k, st, pad in ((3, 7, 5, 6, 9, 4, 2, 1), (9, 20, 9, 13, 33, 4, 2, 0), (2, 5, 7, 7, 8, 6, 3, 0)):
        x, w = rng.standard_normal((N, Cin, H, W)).astype(np.float32), wl.random_i8(rng, (Cin, Cout, k, k), bits)
        q = orc.quantize(x, s_x, bits)
        acc, bias = orc.approx_conv_transpose2d(t, bits, q, w, st, pad, threads=4), rng.standard_normal(Cout).astype(np.float32)
        pw = B.adapt_weights_pack_conv_transpose2d(L, dev(w), st)
        assert (host(B.adapt_approx_conv_transpose2d_packed(pw, dev(q), pad)) == acc).all()
        got = B.adapt_conv_transpose2d_layer_f32(pw, dev(x), s_x, s_out, pad, dev(bias), act)
        assert bits_equal(host(got), finish(acc, s_out, bias, None, act)), (k, st, pad)


@pytest.mark.parametrize("bits,kind", [(8, "product"), (7, "product"), (8, "dropped")])
@pytest.mark.parametrize("act", [0, 2])
@pytest.mark.parametrize("case", [
    # N, Cin, H, W, Cout, k, stride, padding
    (600, 3, 16, 16, 3, 4, 2, 1),           # at most four channels of a tile, many pixels per row slot
    (40, 5, 9, 13, 20, 4, 2, 0),            # the same in the last tile, runs that end inside a row
    (60, 4, 12, 10, 4, 6, 2, 2),            # three taps: 25 classes of border positions
    (2, 6, 1, 9, 7, 6, 2, 0),               # fewer rows than taps: no classes
    (3, 2, 1, 2, 5, 4, 2, 1),               # every position at a border
    (2, 3, 5, 4, 6, 24, 2, 11)])            # more classes than LDS has room for
def test_border_terms_and_narrow_tiles_of_transposed_layers(B, bits, kind, act, case):
    N, Cin, H, W, Cout, k, st, pad = case
    rng = np.random.default_rng(bits + act + sum(case))
    t = table(kind, bits, rng)
    x, w = rng.standard_normal((N, Cin, H, W)).astype(np.float32), wl.random_i8(rng, (Cin, Cout, k, k), bits)
    s_x, s_out = np.float32(0.02), np.float32(2e-4)
    q, bias = orc.quantize(x, s_x, bits), rng.standard_normal(Cout).astype(np.float32)
    acc = orc.approx_conv_transpose2d(t, bits, q, w, st, pad, threads=4)
    pw = B.adapt_weights_pack_conv_transpose2d(B.Lut(t, bits), dev(w), st)
    assert (host(B.adapt_approx_conv_transpose2d_packed(pw, dev(q), pad)) == acc).all()
    assert bits_equal(host(B.adapt_conv_transpose2d_layer_f32(pw, dev(x), s_x, s_out, pad, dev(bias), act)), finish(acc, s_out, bias, None, act))


@pytest.mark.parametrize("bits,kind", FORMS)
@pytest.mark.parametrize("first", ["conv", "transposed", "depthwise", "grouped"])
def test_chains_between_forms(B, bits, kind, first):
    """The copy that each kind of producer writes for a convolution that moves by 1 to 3 pixels (a transposed one: for such a
    one too), behind a ReLU (half of every table) and without; 8 and 18 channels (whole words of the copy, and a last one that is not)."""
    rng = np.random.default_rng(bits)
    t = table(kind, bits, rng)
    L = B.Lut(t, bits)
    s_x, s_1, s_2, s_o = np.float32(0.03), np.float32(1e-3), np.float32(0.2), np.float32(1e-3)
    for C in (8, 18):
        x = rng.standard_normal((3, C, 11, 13)).astype(np.float32)
        if first == "transposed":
            x = x[:, :, :6, :7]
        q = orc.quantize(x, s_x, bits)
        if first == "conv":
            w1 = wl.random_i8(rng, (C, C, 3, 3), bits)
            p1, acc1 = B.adapt_weights_pack_conv2d(L, dev(w1)), orc.approx_conv2d(t, bits, q, w1, (1, 1), (1, 1), threads=4)
            run = lambda out, act, p2: B.adapt_conv2d_layer_chain_f32(p1, dev(x), s_x, s_1, out, (1, 1), (1, 1), act=act, next_pw=p2, s_next=s_2)
        elif first == "transposed":
            w1 = wl.random_i8(rng, (C, C, 4, 4), bits)
            p1, acc1 = B.adapt_weights_pack_conv_transpose2d(L, dev(w1), 2), orc.approx_conv_transpose2d(t, bits, q, w1, 2, 1, threads=4)
            run = lambda out, act, p2: B.adapt_conv_transpose2d_layer_chain_f32(p1, dev(x), s_x, s_1, out, 1, act=act, next_pw=p2, s_next=s_2)
        else:
            g = C if first == "depthwise" else C // 2
            w1 = wl.random_i8(rng, (C, C // g, 3, 3), bits)
            acc1 = orc.approx_conv2d(t, bits, q, w1, (1, 1), (1, 1), (1, 1), g, threads=4)
            run = lambda out, act, p2: out.copy_(B.adapt_conv2d_grouped_layer_f32(L, dev(x), dev(w1), s_x, s_1, (1, 1), (1, 1), groups=g, act=act,
                                                                                  next_pw=p2, s_next=s_2))
        _, _, H, W = acc1.shape
        for st in (1, 2, 3) + ((0,) if first == "transposed" else ()):          # (0: the consumer is a transposed convolution, too)
            w2 = wl.random_i8(rng, (C, 19, 4, 4) if st == 0 else (19, C, 3, 3), bits)
            p2 = B.adapt_weights_pack_conv_transpose2d(L, dev(w2), 2) if st == 0 else B.adapt_weights_pack_conv2d(L, dev(w2))
            if st == 0:
                B.adapt_conv_transpose2d_chain_prepare(p2, 3, H, W, 1)
            else:
                B.adapt_conv2d_chain_prepare(p2, 3, H, W, (st, st), (1, 1))
            for act in (1, 0, 1):
                y = finish(acc1, s_1, None, None, act)
                q2 = orc.quantize(y, s_2, bits)
                acc2 = orc.approx_conv_transpose2d(t, bits, q2, w2, 2, 1, threads=4) if st == 0 else orc.approx_conv2d(t, bits, q2, w2, (st, st), (1, 1), threads=4)
                out1 = torch.empty(acc1.shape, dtype=torch.float32, device="cuda")
                out2 = torch.empty(acc2.shape, dtype=torch.float32, device="cuda")
                run(out1, act, p2)
                if st == 0:
                    B.adapt_conv_transpose2d_layer_chain_f32(p2, None, s_2, s_o, out2, 1, in_shape=(3, H, W))
                else:
                    B.adapt_conv2d_layer_chain_f32(p2, None, s_2, s_o, out2, (st, st), (1, 1), in_shape=(3, H, W))
                assert bits_equal(host(out1), y), (C, st, act)
                assert bits_equal(host(out2), finish(acc2, s_o, None, None, 0)), (C, st, act)


@pytest.mark.parametrize("bits,kind", [(8, "product"), (8, "dropped"), (7, "product"), (7, "one_side"), (6, "product"), (2, "product")])
@pytest.mark.parametrize("rows,Hs", [(1, 64), (65, 128), (7, 192), (64, 576), (50, 320), (33, 448), (70, 832), (17, 1088)])
def test_time_steps_on_one_byte_entries(B, bits, kind, rows, Hs):
    """The three recurrent steps on either side of the rule that takes one-byte entries (8 bits: nearly all of these; fewer: from 32 or 48 rows and
    192 or 256 units on; several rounds of workgroups: all): asymmetric tables, slices of 4 to 68 inner indices, of which up to three groups of four are
    no block of 16, codes beyond the operand's range (which wrap), activations that are word-aligned only, or not even that
    (which take the 16-bit entries)."""
    rng = np.random.default_rng(bits + rows + Hs)
    t = table(kind, bits, rng)
    L = B.Lut(t, bits)
    s_ih, s_hh, s_h = np.float32(3e-5), np.float32(2e-5), np.float32(1.0) / np.float32(max(1, (1 << (bits - 1)) - 1))
    h = 1 << (bits - 1)
    qh = rng.integers(-128, 128, size=(rows, Hs)).astype(np.int8)
    wrapped = ((((qh.astype(np.int32) + h) & (2 * h - 1)) - h)).astype(np.int8)
    shifted = [torch.empty(rows * Hs + by, dtype=torch.int8, device="cuda")[by:].view(rows, Hs) for by in (1, 4)]
    for q in shifted:
        q.copy_(dev(qh))
    new = lambda dt: torch.empty((rows, Hs), dtype=dt, device="cuda")
    for gates in (4, 3, 1):
        w = wl.random_i8(rng, (gates * Hs, Hs), bits)
        acc_ih = rng.integers(-40000, 40000, size=(rows, gates * Hs)).astype(np.int32)
        acc_hh = orc.approx_linear(t, bits, wrapped, w, threads=4)
        pw = B.adapt_weights_pack_linear(L, dev(w))
        c0, h0, bias = (rng.standard_normal(s).astype(np.float32) for s in ((rows, Hs), (rows, Hs), gates * Hs))
        for q in (dev(qh), *shifted):
            hd, qn = new(torch.float32), new(torch.int8)
            if gates == 4:
                cd = dev(c0)
                B.adapt_lstm_step_f32(pw, q, dev(acc_ih), s_ih, s_hh, s_h, dev(bias), cd, hd, qn)
                want, c_want = orc.lstm_cell(acc_ih, acc_hh, s_ih, s_hh, bias, c0)
                assert bits_equal(host(cd), c_want)
            elif gates == 3:
                B.adapt_gru_step_f32(pw, q, dev(acc_ih), s_ih, s_hh, s_h, dev(bias), None, dev(h0), hd, qn)
                want = orc.gru_cell(acc_ih, acc_hh, s_ih, s_hh, bias, None, h0)
            else:
                B.adapt_rnn_step_f32(pw, q, dev(acc_ih), s_ih, s_hh, s_h, dev(bias), hd, qn)
                want = orc.rnn_cell(acc_ih, acc_hh, s_ih, s_hh, bias)
            assert bits_equal(host(hd), want), (gates, q.data_ptr() % 4)
            assert (host(qn) == orc.quantize(want, s_h, bits)).all()


# Tables of which several activations share a line, so that a step copies 4 to 128 of them, half as many behind a ReLU (that each table is
# taken as one of these is checked on the host, in test_byte_form_host.py)
BARE = [(8, "bare"), (8, "bare_activation"), (7, "bare"), (8, "share1"), (8, "share3"), (6, "share3"), (5, "share2"), (4, "share1"), (4, "share2"), (3, "share1")]


@pytest.mark.parametrize("bits,kind", BARE)
@pytest.mark.parametrize("case", CONVS)
def test_convolution_where_activations_share_lines(B, bits, kind, case):
    test_convolution(B, bits, kind, case)


@pytest.mark.parametrize("bits,kind", BARE)
@pytest.mark.parametrize("act", [0, 1, 2])
def test_fused_layers_where_activations_share_lines(B, bits, kind, act):
    test_fused_layers_on_every_form(B, bits, kind, act)


@pytest.mark.parametrize("bits,kind", BARE)
@pytest.mark.parametrize("first", ["conv", "transposed", "depthwise", "grouped"])
def test_chains_where_activations_share_lines(B, bits, kind, first):
    test_chains_between_forms(B, bits, kind, first)


@pytest.mark.parametrize("bits,kind", BARE[:5])
@pytest.mark.parametrize("rows,Hs", [(65, 128), (65, 320)])
def test_time_steps_where_activations_share_lines(B, bits, kind, rows, Hs):
    test_time_steps_on_one_byte_entries(B, bits, kind, rows, Hs)


@pytest.mark.parametrize("bits,kind", BARE)
@pytest.mark.parametrize("M,K,N", [(512, 77, 37), (4097, 130, 33)])
def test_linear_where_activations_share_lines(B, bits, kind, M, K, N):
    """Packed and plain, the codes' whole int8 range (which wraps)."""
    rng = np.random.default_rng(bits + M)
    t, h = table(kind, bits, rng), 1 << (bits - 1)
    L = B.Lut(t, bits)
    a, w = rng.integers(-128, 128, size=(M, K)).astype(np.int8), wl.random_i8(rng, (N, K), bits)
    want = orc.approx_linear(t, bits, (((a.astype(np.int32) + h) & (2 * h - 1)) - h).astype(np.int8), w, threads=4)
    assert (host(B.adapt_approx_linear_packed(B.adapt_weights_pack_linear(L, dev(w)), dev(a))) == want).all()
    assert (host(B.adapt_approx_linear(L, dev(a), dev(w))) == want).all()


@pytest.mark.parametrize("M,K,N", [(3, 40, 512), (70, 33, 1024), (17, 1008, 1024), (5, 1024, 1024), (2, 9, 1536), (9, 12, 500)])
def test_row_offsets_a_multiple_of_two_kilobytes_apart(B, M, K, N):
    """512 columns and their multiples lie 16 further apart, where there is room (1008 x 1040 words are 4 MiB less 1 KiB of the call that
    allocates nothing; 1024 x 1024 fill it): packed, plain, without allocation, and as a transposed layer of one pixel; two-pass tables too."""
    rng = np.random.default_rng(K)
    for t in (table("beyond", 8, rng), rng.integers(-100000, 100000, size=(256, 256)).astype(np.int32)):
        L = B.Lut(t, 8)
        a, w = rng.integers(-128, 128, size=(M, K)).astype(np.int8), wl.random_i8(rng, (N, K), 8)
        want = orc.approx_linear(t, 8, a, w, threads=4)
        assert (host(B.adapt_approx_linear(L, dev(a), dev(w))) == want).all()
        assert (host(B.adapt_approx_linear_packed(B.adapt_weights_pack_linear(L, dev(w)), dev(a))) == want).all()
        out = torch.empty((M, N), dtype=torch.int32, device="cuda")
        B.adapt_approx_linear_noalloc(L, dev(a), dev(w), out)
        assert (host(out) == want).all()
        if N % 4 == 0 and K < 100:
            wt = wl.random_i8(rng, (K, N // 4, 2, 2), 8)
            x = a.reshape(M, K, 1, 1)
            pw = B.adapt_weights_pack_conv_transpose2d(L, dev(wt), 2)
            assert (host(B.adapt_approx_conv_transpose2d_packed(pw, dev(x), 0)) == orc.approx_conv_transpose2d(t, 8, x, wt, 2, 0, threads=4)).all()


@pytest.mark.parametrize("bits,kind", [(6, "product"), (6, "one_side"), (4, "product"), (8, "share2"), (2, "product")])
def test_one_row_tile_on_small_tables(B, bits, kind):
    """Up to 512 rows on tables of at most 16 KB: every remainder of a group of four steps, waves without rows, slices, and outputs that
    are no whole tile; sums, and the fused layer."""
    rng = np.random.default_rng(bits)
    t = table(kind, bits, rng)
    L = B.Lut(t, bits)
    for hw, K, N in [(1, 16, 16)] + [(22, k, 17) for k in range(4, 150, 16)] + [(3, 300, 40), (16, 517, 33), (22, 1030, 250)]:
        x, w = rng.standard_normal((1, K, hw, hw)).astype(np.float32), wl.random_i8(rng, (N, K, 1, 1), bits)
        s_x, s_out = np.float32(0.02), np.float32(2e-4)
        q, bias = orc.quantize(x, s_x, bits), rng.standard_normal(N).astype(np.float32)
        acc = orc.approx_conv2d(t, bits, q, w, (1, 1), (0, 0), threads=4)
        pw = B.adapt_weights_pack_conv2d(L, dev(w))
        assert (host(B.adapt_approx_conv2d_packed(pw, dev(q))) == acc).all(), (hw, K, N)
        assert bits_equal(host(B.adapt_conv2d_layer_f32(pw, dev(x), s_x, s_out, (1, 1), (0, 0), bias=dev(bias), act=1)), finish(acc, s_out, bias, None, 1))
