"""Norms of rows that start at any element: widths around a vector, a wave and the register
tile, and aligned widths at a shifted base, against float64 torch on the same values."""

import pytest

torch = pytest.importorskip("torch")
import paper_2406_16282_amd as lmbp  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def shifted(t, offset):
    room = torch.empty(t.numel() + offset + 8, dtype=t.dtype, device=DEV)
    out = room[offset:offset + t.numel()].view(t.shape)
    out.copy_(t)
    return out


@pytest.mark.parametrize("op", ["msln", "msrms"])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("rows,cols,offset", [
    (5, 1, 0), (7, 2, 1), (9, 7, 0), (3, 9, 1), (130, 63, 0), (66, 511, 1), (31, 513, 0), (33, 768, 1), (20, 1023, 0),
    (18, 1025, 3), (9, 2049, 0), (6, 4096, 1), (5, 4100, 2), (3, 16385, 0), (3, 16383, 1), (2, 32767, 0), (2, 32775, 0)])
def test_against_float64(op, dtype, rows, cols, offset):
    """Error bounds: bf16 outputs one rounding (2^-8 of the value), fp32 sums of `cols`
    terms kept to 1e-5 of the row's RMS (the stated figure for fp32 and rstd)."""
    print(f"[ragged] {op} {dtype} {rows}x{cols}+{offset}", flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(rows * 100003 + cols)
    x, dz = (shifted((torch.randn(rows, cols, generator=g, device=DEV) + 0.5).to(dtype), offset) for _ in range(2))
    eps = 1e-5
    fwd, bwd = (lmbp.msln_fwd, lmbp.msln_bwd) if op == "msln" else (lmbp.msrms_fwd, lmbp.msrms_bwd)
    z, rstd = fwd(x, eps, z=shifted(torch.zeros_like(x), offset))
    x64 = x.double()
    h = x64 - x64.mean(-1, keepdim=True) if op == "msln" else x64
    r64 = (h.square().mean(-1, keepdim=True) + eps).rsqrt()
    step = 2.0 ** -8 if dtype == torch.bfloat16 else 1e-5
    assert ((rstd.double() - r64[:, 0]).abs() <= 1e-5 * r64[:, 0]).all()
    z64 = h * r64
    scale = z64.square().mean(-1, keepdim=True).sqrt()
    assert ((z.double() - z64).abs() <= step * z64.abs() + 1e-5 * (scale + (x64 * r64).abs())).all()
    dx = bwd(dz, z, rstd, dx=shifted(torch.zeros_like(x), offset))
    d64, zs, rs = dz.double(), z.double(), rstd.double()[:, None]
    ref = d64 - zs * (zs * d64).mean(-1, keepdim=True)
    ref = rs * (ref - d64.mean(-1, keepdim=True) if op == "msln" else ref)
    terms = rs * d64.square().mean(-1, keepdim=True).sqrt()
    assert ((dx.double() - ref).abs() <= step * ref.abs() + 1e-5 * terms * (1 + zs.abs())).all()
    in_place = shifted(x, offset)
    fwd(in_place, eps, z=in_place)
    assert torch.equal(in_place, z)
