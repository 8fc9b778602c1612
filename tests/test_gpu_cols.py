"""GPU parity of the columns kernel (operands of 9 to 12 bits, tables that are an exact product plus an error of 16 bits)
against the CPU oracle: every sum bit-exact, at the edges of its runs, tiles, stages and slices, and of what counts as such a
table."""
import numpy as np
import pytest
import torch

import oracle as orc

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


def table(bits, span, rng, low=-1000):
    """exact product + an error from low to low + span, both ends in use"""
    h = 1 << (bits - 1)
    v = np.arange(-h, h, dtype=np.int64)
    t = v[:, None] * v[None, :] + rng.integers(low, low + span + 1, size=(2 * h, 2 * h))
    t[0, 0], t[-1, -1] = h * h + low, (h - 1) ** 2 + low + span
    return np.ascontiguousarray(t.astype(np.int32))


def codes(rng, shape, bits):
    h = 1 << (bits - 1)
    return rng.integers(-h, h, size=shape).astype(np.int16)


CONVS = [
    # bits, N, Cin, H, W, Cout, kh, kw, sh, sw, ph, pw, dh, dw
    (12, 1, 1, 1, 1, 1, 1, 1, 1, 1, 0, 0, 1, 1),            # one lookup: half a pair, one pixel, one channel
    (12, 2, 3, 9, 9, 5, 3, 3, 1, 1, 1, 1, 1, 1),            # odd channels, a tile and one channel, runs that end inside a row
    (11, 3, 6, 8, 13, 4, 3, 3, 2, 2, 1, 1, 1, 1),           # stride 2: columns in residue classes
    (10, 2, 7, 10, 17, 9, 5, 3, 1, 3, 2, 1, 1, 1),          # horizontal stride 3, a last stage that is not full
    (9, 1, 20, 12, 14, 8, 3, 3, 1, 2, 2, 2, 2, 2),          # dilation with stride 2, many slices
    (9, 1, 33, 16, 16, 6, 1, 1, 1, 1, 0, 0, 1, 1),          # 17 pairs: two stages and a bit
    (12, 5, 16, 32, 33, 7, 1, 1, 1, 1, 0, 0, 1, 1),         # two row tiles of one run per thread
    (10, 9, 8, 63, 64, 64, 1, 1, 1, 1, 0, 0, 1, 1),         # two runs per thread, units on eight dies
]


@pytest.mark.parametrize("case", CONVS)
def test_conv2d_bit_exact(B, case):
    bits, N, Cin, H, W, Cout, kh, kw, sh, sw, ph, pw, dh, dw = case
    rng = np.random.default_rng(sum(case))
    lut = table(bits, 65535, rng)
    x, w = codes(rng, (N, Cin, H, W), bits), codes(rng, (Cout, Cin, kh, kw), bits)
    got = host(B.adapt_approx_conv2d_i16(B.Lut16(bits, table=lut), dev(x), dev(w), (sh, sw), (ph, pw), (dh, dw)))
    want = orc.approx_conv2d_i16(bits, x, w, lut=lut, stride=(sh, sw), pad=(ph, pw), dil=(dh, dw), threads=4)
    assert (got == want).all()


@pytest.mark.parametrize("bits,M,K,N", [(9, 1, 1, 1), (12, 65, 33, 5), (10, 4097, 64, 3), (11, 300, 1001, 18)])
def test_linear_bit_exact(B, bits, M, K, N):
    rng = np.random.default_rng(bits + M)
    lut = table(bits, 65535, rng, low=-65000)
    a, w = codes(rng, (M, K), bits), codes(rng, (N, K), bits)
    got = host(B.adapt_approx_linear_i16(B.Lut16(bits, table=lut), dev(a), dev(w)))
    assert (got == orc.approx_linear_i16(lut, bits, a, w, threads=4)).all()


@pytest.mark.parametrize("span", [0, 65535, 65536])
def test_edge_of_the_form(B, span):
    """An error of 65536 does not fit: the product gathers from the whole table, with the same sums; so do 8-bit tables."""
    rng = np.random.default_rng(span)
    for bits in (8, 9):
        lut = table(bits, span, rng, low=-40000)
        a, w = codes(rng, (130, 48), bits), codes(rng, (21, 48), bits)
        got = host(B.adapt_approx_linear_i16(B.Lut16(bits, table=lut), dev(a), dev(w)))
        assert (got == orc.approx_linear_i16(lut, bits, a, w, threads=4)).all()


def test_codes_wrap_like_the_gathering_kernel(B):
    """Codes beyond the operand width select by their low bits."""
    rng = np.random.default_rng(5)
    a, w = rng.integers(-32768, 32768, size=(70, 31)).astype(np.int16), codes(rng, (6, 31), 10)
    wrapped = (((a.astype(np.int64) + 512) & 1023) - 512).astype(np.int16)
    for span in (65535, 65536):
        lut = table(10, span, rng)
        got = host(B.adapt_approx_linear_i16(B.Lut16(10, table=lut), dev(a), dev(w)))
        assert (got == orc.approx_linear_i16(lut, 10, wrapped, w, threads=4)).all()


def test_one_output_column_under_a_large_stride(B):
    """The horizontal stride does not matter where the window never moves."""
    rng = np.random.default_rng(3)
    h = 1 << 9
    v = np.arange(-h, h, dtype=np.int64)
    t = (v[:, None] * v[None, :] + rng.integers(-1000, 1000, size=(2 * h, 2 * h))).astype(np.int32)
    L = B.Lut16(10, table=t)
    x, w = rng.integers(-h, h, size=(3, 5, 20, 6)).astype(np.int16), rng.integers(-h, h, size=(6, 5, 3, 5)).astype(np.int16)
    xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    want = B.adapt_approx_conv2d_i16(L, xd[..., :5].contiguous(), wd)
    for sw in (4, 1 << 20, (1 << 31) - 1):
        assert torch.equal(B.adapt_approx_conv2d_i16(L, xd, wd, (1, sw)), want)
