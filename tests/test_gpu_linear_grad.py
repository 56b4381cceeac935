"""Parameter gradients of the fused linear layers: dW = dz^T x in every tile configuration
and with the rows split or whole, ragged in every dimension, and the activation backward
with the bias gradient. Inputs of the products are small integers times powers of two, so
that every fp32 sum is exact in any order and dW must equal the rounding of torch's."""

import ctypes

import pytest

torch = pytest.importorskip("torch")
import paper_2406_16282_amd as lmbp  # noqa: E402
from paper_2406_16282_amd import nn as lnn  # noqa: E402

DEV = "cuda:0"


def dyadic(shape, exp, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return torch.randint(-8, 9, shape, generator=g, device=DEV).float() * 2.0 ** exp


# rows x output features x input features
SHAPES = [
    (0, 32, 16), (1, 16, 8), (63, 144, 264), (65, 400, 136), (197, 3072, 768),
    (700, 272, 136), (3001, 272, 520), (9001, 272, 264),
    (4100, 528, 1032), (5000, 3072, 768), (6001, 1040, 520),
    (333, 11008, 4104), (130, 11024, 4104), (1030, 8208, 2056), (1999, 5632, 2048),
    (2048, 11008, 4096), (12609, 3072, 776),
]
# Sizes by the tile that they take (256 CUs: 0 .. 2 for 256 x 256, 128 x 256, 128 x 128), the
# rows whole or split, one or several units of work to a block.
FORMS = [
    (0, (1412, 5520, 1808)), (0, (1099, 11584, 2312)), (0, (5837, 2000, 1312)), (0, (7838, 3472, 2360)),
    (1, (548, 12528, 392)), (1, (29, 11360, 1336)), (1, (3780, 1344, 904)), (1, (13601, 1600, 3344)),
    (2, (65, 16, 8)), (2, (7, 8544, 904)), (2, (356, 16, 8)), (2, (2978, 11584, 8)), (2, (50001, 64, 72)),
]


def test_every_form_is_covered():
    L, seen = lmbp.lib(), set()
    for tile, (m, n, k) in FORMS:
        splits, rounds = ctypes.c_int64(), ctypes.c_int64()
        assert L.lmbp_linear_grad_form(m, n, k, splits, rounds) == tile, (m, n, k)
        seen.add((tile, splits.value > 1, rounds.value > 1))
    assert len(seen) == 12 and splits.value > 12   # the last one: many shares


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,k", SHAPES + [s for _, s in FORMS])
def test_weight_grad_exact(m, n, k):
    print(f"[grad] {m} {n} {k}", flush=True)
    dz, x = dyadic((m, n), -3, 1), dyadic((m, k), -4, 2)
    dw = lmbp.linear_weight_grad(dz.bfloat16(), x.bfloat16())
    assert torch.equal(dw, (dz.t() @ x).bfloat16())


@pytest.mark.gpu
@pytest.mark.parametrize("act", ["gelu", "silu"])
@pytest.mark.parametrize("m,n,k", [(0, 32, 16), (1, 16, 8), (64, 528, 16), (129, 1040, 24), (3001, 272, 520),
                                   (700, 3072, 768)])
def test_act_bwd_with_bias(m, n, k, act):
    """dz is the activation backward's, dw the product's of that dz; db is the rounding of
    an fp32 sum of m values: within m 2^-24 of their absolute sum, plus one rounding (2^-8)."""
    print(f"[grad] act {m} {n} {k} {act}", flush=True)
    pre, dy, x = dyadic((m, n), -1, 1).bfloat16(), dyadic((m, n), -6, 2).bfloat16(), dyadic((m, k), -4, 3).bfloat16()
    fwd, bwd = (lmbp.regelu2_fwd, lmbp.regelu2_bwd) if act == "gelu" else (lmbp.resilu2_fwd, lmbp.resilu2_bwd)
    codes = fwd(pre)[1]
    dz, dw, db = lmbp.linear_act_bwd(dy, codes, x, act)
    ref = bwd(dy, codes)
    assert torch.equal(dz.view(torch.int16), ref.view(torch.int16))
    assert torch.equal(dw, lmbp.linear_weight_grad(ref, x))
    exact, size = ref.double().sum(0), ref.double().abs().sum(0)
    assert ((db.double() - exact).abs() <= exact.abs() * 2.0 ** -8 + size * m * 2.0 ** -24 * 1.01).all()
    dz2, none, db2 = lmbp.linear_act_bwd(dy, codes, x, act, weight_grad=False)
    assert none is None and torch.equal(dz2, dz) and torch.equal(db2, db)


@pytest.mark.gpu
@pytest.mark.parametrize("m,n", [
    (1, 16), (511, 16), (513, 16), (5, 32), (257, 48), (1025, 64), (129, 128), (70001, 144), (33, 256), (20011, 272),
    (100001, 512), (4099, 1040), (3001, 4112),       # lanes to a row 2 .. 64, one and several groups to a block
    (600011, 240), (33001, 4112), (9001, 16400),     # eight pieces at once
    (1, 1 << 20)])                                   # more blocks along the columns than are wanted in all
def test_bias_gradient_pieces(m, n):
    """dz and db without dw; bounds as above."""
    print(f"[grad] db {m} {n}", flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(m + n)
    dy = torch.randn((m, n), generator=g, device=DEV, dtype=torch.bfloat16)
    codes = torch.randint(-2 ** 31, 2 ** 31, (m * n // 16,), generator=g, device=DEV, dtype=torch.int32)
    dz, _, db = lmbp.linear_act_bwd(dy, codes, torch.empty((m, 8), device=DEV, dtype=torch.bfloat16), "silu",
                                    weight_grad=False)
    assert torch.equal(dz.view(torch.int16), lmbp.resilu2_bwd(dy, codes).view(torch.int16))
    exact, size = dz.sum(0, dtype=torch.float64), dz.abs().sum(0, dtype=torch.float64)
    assert ((db.double() - exact).abs() <= exact.abs() * 2.0 ** -8 + size * m * 2.0 ** -24 * 1.01).all()
    db2 = lmbp.linear_act_bwd(dy, codes, torch.empty((m, 8), device=DEV, dtype=torch.bfloat16), "silu")[2]
    assert torch.equal(db, db2)   # the same sums in the same order


@pytest.mark.gpu
@pytest.mark.parametrize("needs", [(True, True, True), (False, True, True), (True, False, True), (True, True, False)])
def test_module_gradients_against_recorded_backward(needs):
    """The kernels' gradients against those of a recorded backward (create_graph), which
    are torch's products of the same dz: one rounding apart at most."""
    layer = lnn.LinearReGELU2(264, 272, device=DEV)
    x = torch.randn(3, 67, 264, device=DEV, dtype=torch.bfloat16)
    dy = torch.randn(3, 67, 272, device=DEV, dtype=torch.bfloat16)
    x.requires_grad_(needs[0])
    layer.weight.requires_grad_(needs[1])
    layer.bias.requires_grad_(needs[2])
    wrt = [t for t in (x, layer.weight, layer.bias) if t.requires_grad]
    got = torch.autograd.grad(layer(x), wrt, dy)
    ref = torch.autograd.grad(layer(x), wrt, dy, create_graph=True)
    for a, r in zip(got, ref):
        d = (a.double() - r.double()).abs()
        assert (d <= r.double().abs() * 2.0 ** -7 + 1e-3 * r.double().square().mean().sqrt()).all()


@pytest.mark.gpu
def test_saved_tensor_hooks_may_change_the_layout():
    layer = lnn.LinearReSiLU2(64, 48, device=DEV)
    x = torch.randn(33, 64, device=DEV, dtype=torch.bfloat16, requires_grad=True)
    dy = torch.randn(33, 48, device=DEV, dtype=torch.bfloat16)
    ref = torch.autograd.grad(layer(x), [x, layer.weight, layer.bias], dy)

    def unpack(t):   # the same values in another layout
        return t.t().contiguous().t() if t.dim() == 2 else t

    with torch.autograd.graph.saved_tensors_hooks(lambda t: t, unpack):
        y = layer(x)
        got = torch.autograd.grad(y, [x, layer.weight, layer.bias], dy)
    for a, r in zip(got, ref):
        assert torch.allclose(a.float(), r.float(), rtol=2.0 ** -6, atol=1e-2)


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,k", [(65, 144, 136), (700, 272, 136)])   # rows whole and split
def test_infinities_and_nan_stay_in_their_rows_and_columns(m, n, k):
    """dw, dz and db carry an infinity or NaN where a sum over its column meets it, and the
    same bits as without it everywhere else (tile edges, other shares of the rows)."""
    dy, x = dyadic((m, n), -3, 1).bfloat16(), dyadic((m, k), -4, 2).bfloat16() + 1.0
    codes = lmbp.resilu2_fwd(torch.full((m, n), 30.0, device=DEV, dtype=torch.bfloat16))[1]   # slope 1 throughout
    clean = lmbp.linear_act_bwd(dy, codes, x, "silu")
    bad_dy, bad_x = dy.clone(), x.clone()
    bad_dy[m - 1, 0], bad_dy[0, n - 1], bad_dy[m // 2, 17] = float("inf"), float("-inf"), float("nan")
    bad_x[m - 1, k - 1] = float("nan")
    dz, dw, db = lmbp.linear_act_bwd(bad_dy, codes, bad_x, "silu")
    assert torch.equal(dw.view(torch.int16), lmbp.linear_weight_grad(bad_dy, bad_x).view(torch.int16))
    rows = torch.zeros(n, dtype=torch.bool, device=DEV)
    rows[[0, 17, n - 1]] = True
    assert torch.equal(dz.view(torch.int16), bad_dy.view(torch.int16))
    assert torch.equal(~db.isfinite(), rows) and torch.equal(db[~rows], clean[2][~rows])
    assert db[0] == float("inf") and db[n - 1] == float("-inf") and db[17].isnan()
    good = ~rows[:, None] & (torch.arange(k, device=DEV) < k - 1)[None]
    assert torch.equal(dw[good], clean[1][good])
    assert not dw[rows].isfinite().any() and dw[:, k - 1].isnan().all()
