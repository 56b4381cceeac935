"""Fused linear layers in every form (split K, tiles), at the sizes where one can go wrong:
ragged last tiles, one K step (the load stream runs two tiles ahead), one row or column
more or less than a whole tile, more tiles than resident blocks, and a bias between words.
PLAIN_FORMS and GATED_FORMS say which form their sizes take, and the library is asked
whether they still do.

Inputs are small integers times powers of two, so every product and every fp32 sum is
exact in any order (|sum| < 2^24 units): the stored pre-activation must equal the rounding
of torch's fp32 product bit for bit, and y and the codes must be what the activation
kernels make of it."""

import ctypes

import pytest

torch = pytest.importorskip("torch")
import paper_2406_16282_amd as lmbp  # noqa: E402

DEV = "cuda:0"


def dyadic(shape, exp, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return torch.randint(-8, 9, shape, generator=g, device=DEV).float() * 2.0 ** exp


def product(x, w, b=None):
    z = x @ w.t()   # fp32, exact
    return (z if b is None else z + b).bfloat16()


# rows x output features x input features
SHAPES = [
    (1, 16, 8), (16, 3072, 768), (17, 48, 264), (31, 16, 1032), (33, 1040, 776),
    (90, 528, 520), (200, 2064, 136), (5, 16400, 2056),
    (777, 3088, 136), (3000, 4112, 72), (8000, 8208, 8),
    (1999, 3088, 72), (3001, 2064, 72), (9001, 2064, 640),
    (3001, 8176, 520), (4097, 5648, 776),
    (1999, 6160, 520), (3001, 4112, 520), (4097, 3056, 520), (4100, 11008, 1032), (8266, 10976, 8),
]
GATED = [
    (1, 16, 8), (16, 11008, 520), (17, 48, 264), (29, 5632, 2056), (100, 80, 776),
    (2, 16400, 1032), (129, 16400, 136), (700, 1552, 8), (4097, 4112, 8), (3001, 1040, 72),
    (1025, 3056, 72), (4097, 5648, 520), (1999, 5648, 776), (1999, 3088, 520),
    (2049, 3056, 520), (2048, 11008, 1032),
]
# Sizes by the form that they take (256 CUs): split K with 16 and 32 rows to a block, tiles of
# 256 x 256, 128 x 256, 128 x 128 and 64 x 128 (gated: half the columns); one or several row
# blocks (split K) or tiles to a block, several K steps or one (for which only the smallest
# tile is taken).
ROWS16, ROWS32, BIG, MID, SMALL, LOW = range(6)
PLAIN_FORMS = [
    (ROWS16, (5, 64, 8)), (ROWS16, (23, 16, 8)), (ROWS16, (12, 16, 72)), (ROWS16, (31, 16, 88)),
    (ROWS32, (19, 4320, 8)), (ROWS32, (4597, 16, 8)), (ROWS32, (17, 4272, 72)), (ROWS32, (315, 416, 72)),
    (BIG, (3851, 2208, 840)), (BIG, (5789, 4384, 600)),
    (MID, (2784, 2528, 1032)), (MID, (3465, 6096, 264)),
    (SMALL, (1735, 1424, 520)), (SMALL, (3879, 2112, 464)),
    (LOW, (166, 4256, 8)), (LOW, (8316, 656, 16)), (LOW, (1158, 688, 72)), (LOW, (8235, 656, 72)),
]
GATED_FORMS = [
    (ROWS16, (6, 16, 24)), (ROWS16, (32, 16, 8)), (ROWS16, (1, 16, 72)), (ROWS16, (36, 16, 72)),
    (ROWS32, (17, 2160, 8)), (ROWS32, (36, 1488, 16)), (ROWS32, (17, 2144, 72)), (ROWS32, (52, 1120, 72)),
    (BIG, (1223, 4416, 264)), (BIG, (1471, 8864, 264)),
    (MID, (1560, 2272, 264)), (MID, (3488, 2768, 232)),
    (SMALL, (1265, 832, 520)), (SMALL, (4483, 944, 520)),
    (LOW, (33, 4368, 8)), (LOW, (257, 9824, 8)), (LOW, (414, 624, 72)), (LOW, (257, 9808, 72)),
]


@pytest.mark.parametrize("gated,sizes", [(0, PLAIN_FORMS), (1, GATED_FORMS)])
def test_every_form_is_covered(gated, sizes):
    """The sizes take the forms that they are listed for, and no form is left out."""
    L, seen = lmbp.lib(), set()
    for form, (m, n, k) in sizes:
        rounds = ctypes.c_int64()
        assert L.lmbp_linear_form(m, n, k, gated, rounds) == form, (m, n, k)
        several = m > 16 * (form + 1) if form <= ROWS32 else rounds.value > 1
        seen.add((form, several, k > 64))
    assert seen >= {(f, s, True) for f in range(6) for s in (False, True)}
    assert seen >= {(f, s, False) for f in (ROWS16, ROWS32, LOW) for s in (False, True)}


@pytest.mark.gpu
@pytest.mark.parametrize("act", ["gelu", "silu"])
@pytest.mark.parametrize("m,n,k", SHAPES + [s for _, s in PLAIN_FORMS])
def test_plain(m, n, k, act):
    print(f"[tiles] plain {m} {n} {k} {act}", flush=True)
    x, w, b = dyadic((m, k), -3, 1), dyadic((n, k), -4, 2), dyadic((n,), -7, 3)
    y, codes, z = lmbp.linear_act_fwd(x.bfloat16(), w.bfloat16(), b.bfloat16(), act=act, store_z=True)
    ref = product(x, w, b)
    assert torch.equal(z, ref)
    y_r, c_r = (lmbp.regelu2_fwd if act == "gelu" else lmbp.resilu2_fwd)(ref)
    assert torch.equal(y.view(torch.int16), y_r.view(torch.int16))
    assert torch.equal(codes, c_r)


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,k", GATED + [s for _, s in GATED_FORMS])
def test_gated(m, n, k):
    print(f"[tiles] gated {m} {n} {k}", flush=True)
    x, wg, wu = dyadic((m, k), -3, 1), dyadic((n, k), -4, 2), dyadic((n, k), -4, 3)
    h, s, u, codes, g = lmbp.linear_swiglu_fwd(x.bfloat16(), wg.bfloat16(), wu.bfloat16(), store_g=True)
    g_r, u_r = product(x, wg), product(x, wu)
    assert torch.equal(g, g_r) and torch.equal(u, u_r)
    h_r, s_r, c_r = lmbp.reswiglu2_fwd(g_r, u_r)
    for a, r in ((h, h_r), (s, s_r)):
        assert torch.equal(a.view(torch.int16), r.view(torch.int16))
    assert torch.equal(codes, c_r)


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,k", [s for _, s in PLAIN_FORMS] + [(13, 144, 72), (1000, 3088, 72), (1999, 3088, 72), (3001, 8176, 520), (3001, 4112, 520)])
def test_bias_between_words(m, n, k):
    """A bias that starts 2 bytes past a 4-byte word gives the same bytes as an aligned one."""
    x, w, b = dyadic((m, k), -3, 1).bfloat16(), dyadic((n, k), -4, 2).bfloat16(), dyadic((n,), -7, 3).bfloat16()
    room = torch.zeros(n + 3, dtype=torch.bfloat16, device=DEV)
    odd = room[1:n + 1]
    assert odd.data_ptr() % 4 == 2
    odd.copy_(b)
    for a, r in zip(lmbp.linear_act_fwd(x, w, odd, store_z=True), lmbp.linear_act_fwd(x, w, b, store_z=True)):
        assert torch.equal(a, r)


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,k", [s for _, s in PLAIN_FORMS] + [(1, 16, 8), (65, 112, 72), (27, 2064, 2056), (900, 3088, 72), (1999, 3088, 72), (3001, 8176, 520), (3001, 4112, 520)])
def test_norm_in_front(m, n, k):
    """z and rstd are the norm kernel's; x w^T is exact in fp32, so the pre-activation is
    within one fp32 and one bf16 rounding (2^-24 and 2^-8 of the value) of rstd (x w^T)."""
    x, w = dyadic((m, k), -3, 1), dyadic((n, k), -4, 2)
    y, codes, z, rstd, pre = lmbp.msrms_linear_act_fwd(x.bfloat16(), w.bfloat16(), 1e-5, store_pre=True)
    z_r, rstd_r = lmbp.msrms_fwd(x.bfloat16(), 1e-5)
    assert torch.equal(z, z_r) and torch.equal(rstd, rstd_r.reshape(-1))
    exact = (x @ w.t()).double() * rstd.double()[:, None]
    assert ((pre.double() - exact).abs() <= exact.abs() * 2.0 ** -8 * (1 + 1e-4)).all()
    y_r, c_r = lmbp.resilu2_fwd(pre)
    assert torch.equal(y.view(torch.int16), y_r.view(torch.int16)) and torch.equal(codes, c_r)
