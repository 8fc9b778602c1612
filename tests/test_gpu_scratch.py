"""Scratch memory of packed handles: once a handle has run at its largest input size its calls allocate nothing, so a recorded
graph stays valid across smaller calls - also those whose products are split more and leave more partial sums."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2203_04071_amd import binding
    binding.load()
    assert torch.cuda.is_available()
    return binding


def table(bits, form):
    h = 1 << (bits - 1)
    v = np.arange(-h, h, dtype=np.int64)
    t = v[:, None] * v[None, :]
    return np.ascontiguousarray((t if form == "byte" else t + ((v[:, None] * 7919 + v[None, :] * 104729) % 8192 - 4096)).astype(np.int32))


def pack(make, w):
    return make(w), make(w)


def free_bytes():
    """Memory that is free or held by torch's own allocator."""
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0] + torch.cuda.memory_reserved()


LAYERS = ["conv", "conv_strided", "linear_codes", "linear_f32", "transposed"]


def layer_calls(B, layer, form):
    """(largest size, smaller ones, outputs by size, call(size, handle), handle, another handle on the same weights)"""
    gen = torch.Generator(device="cuda").manual_seed(5)
    rnd = lambda *shape: torch.randint(-128, 128, shape, generator=gen, device="cuda", dtype=torch.int8)
    L = B.Lut(table(8, form), 8)
    if layer.startswith("conv"):
        st = 2 if layer.endswith("strided") else 1
        big, small = 64, [33, 8, 16, 1]
        pw, other = pack(lambda w: B.adapt_weights_pack_conv2d(L, w), rnd(64, 64, 3, 3))
        x, ho = rnd(big, 64, 32, 32), 32 // st
        outs = {n: torch.zeros((n, 64, ho, ho), dtype=torch.int32, device="cuda") for n in [big] + small}
        call = lambda n, pw: B.adapt_approx_conv2d_packed(pw, x[:n], (st, st), (1, 1), out=outs[n])
    elif layer == "transposed":
        big, small = 64, [5, 16, 1]
        pw, other = pack(lambda w: B.adapt_weights_pack_conv_transpose2d(L, w, 2), rnd(64, 32, 4, 4))
        x = rnd(big, 64, 8, 8)
        outs = {n: torch.zeros((n, 32, 16, 16), dtype=torch.int32, device="cuda") for n in [big] + small}
        call = lambda n, pw: B.adapt_approx_conv_transpose2d_packed(pw, x[:n], 1, out=outs[n])
    else:
        big, small = 6000, [1111, 4000, 777, 5, 4100]
        pw, other = pack(lambda w: B.adapt_weights_pack_linear(L, w), rnd(999, 777))
        x = rnd(big, 777)
        if layer == "linear_codes":
            outs = {n: torch.zeros((n, 999), dtype=torch.int32, device="cuda") for n in [big] + small}
            call = lambda n, pw: B.adapt_approx_linear_packed(pw, x[:n], out=outs[n])
        else:
            xf = x.float()
            outs = {n: torch.zeros((n, 999), dtype=torch.float32, device="cuda") for n in [big] + small}
            call = lambda n, pw: B.adapt_linear_layer_f32(pw, xf[:n], 1.0, 0.5, out=outs[n])
    return big, small, outs, call, pw, other


@pytest.mark.parametrize("form", ["byte", "general"])
@pytest.mark.parametrize("layer", LAYERS)
def test_smaller_calls_allocate_nothing(B, layer, form):
    big, small, outs, call, pw, other = layer_calls(B, layer, form)
    for n in [big] + small:         # (on a handle of its own: what loading kernels and comparing takes is taken by then)
        call(n, other)
        assert torch.equal(outs[n].clone(), outs[big][:n]), n
    call(big, pw)
    want = outs[big].clone()
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        call(big, pw)
    g.replay()                      # (the first replay may take memory of its own)
    free = free_bytes()
    for n in small + small:
        call(n, pw)
        assert free_bytes() == free, n      # nothing allocated, nothing given back
        assert torch.equal(outs[n], want[:n]), n
        outs[big].zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(outs[big], want), n


@pytest.mark.parametrize("form", ["byte", "general"])
@pytest.mark.parametrize("layer", LAYERS)
def test_smaller_sizes_may_be_recorded_before_they_have_run(B, layer, form):
    big, small, outs, call, pw, other = layer_calls(B, layer, form)
    for n in [big] + small:         # (kernels are loaded)
        call(n, other)
    call(big, pw)
    want = outs[big].clone()
    graphs = []
    for n in small:
        g = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(g):
            call(n, pw)
        graphs.append((n, g))
    for _ in range(3):
        for n, g in graphs:
            outs[n].zero_()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(outs[n], want[:n]), n
            call(big, pw)
