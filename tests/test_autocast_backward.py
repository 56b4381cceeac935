"""Backward of the gated layer inside an autocast region: the sum of its two input products
in the region's type, as the out-of-place sum gives it."""

import pytest

torch = pytest.importorskip("torch")
from paper_2406_16282_amd import nn as lnn  # noqa: E402


def operands(device):
    g = torch.Generator(device=device)
    g.manual_seed(3)
    return [torch.randint(-4, 5, s, generator=g, device=device).bfloat16() for s in ((6, 16), (16, 8), (6, 16), (16, 8))]


@pytest.mark.parametrize("dtype", [None, torch.float16, torch.bfloat16])
def test_two_products(dtype):
    a, b, c, d = operands("cpu")
    with torch.autocast("cpu", dtype=dtype or torch.bfloat16, enabled=dtype is not None):
        got = lnn._two_products(a, b, c, d)
    assert got.dtype == (dtype or torch.bfloat16)
    # whole numbers below 2^8 (bf16) and 2^11 (fp16) in size, except sums that bf16 rounds
    exact = a.double() @ b.double() + c.double() @ d.double()
    assert ((got.double() - exact).abs() <= exact.abs() * 2.0 ** -7 + 2.0).all()


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_gated_layer(dtype):
    layer = lnn.LinearReSwiGLU2(64, 48, device="cuda:0")
    x = torch.randn(33, 64, device="cuda:0", dtype=torch.bfloat16, requires_grad=True)
    dh = torch.randn(33, 48, device="cuda:0", dtype=torch.bfloat16)
    wrt = [x, layer.gate.weight, layer.up.weight]
    ref = torch.autograd.grad(layer(x), wrt, dh)
    y = layer(x)
    with torch.autocast("cuda", dtype=dtype):
        got = torch.autograd.grad(y, wrt, dh)
    for a, r in zip(got, ref):   # one more rounding to bf16 at most: 2^-8 of a value, two for dx
        assert a.dtype == torch.bfloat16
        assert (a.double() - r.double()).abs().max() <= r.double().abs().max() * 2.0 ** -6
