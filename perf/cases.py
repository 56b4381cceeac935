"""The work that a user of this package has it do, as cases that can be timed and compared.

``listed()`` names twelve cases, ``draw(rng)`` makes one more of the same ranges. A case
has a ``kind`` (what is called), its sizes, storage type and options:

* ``norm``: MS-LN / MS-RMSNorm forward, then backward from the saved z and rstd;
* ``act``: ReGELU2 / ReSiLU2 forward, then backward from the saved codes;
* ``glu``: ReSiLU2 inside SwiGLU, forward and backward;
* ``kbit``: a k-bit member of the family with runtime tables, forward and backward;
* ``linear_train``: the fused linear + activation module, forward and all gradients;
* ``linear_eval``: the same module without gradients (evaluation);
* ``glu_eval``: the fused SwiGLU input side without gradients (evaluation, generation);
* ``norm_glu``: MS-RMSNorm + the SwiGLU input side in one call, all saved tensors kept;
* ``mlp_train``: a LLaMA MLP block (norm, gate and up, SwiGLU, down), forward and all
  gradients.
"""

import functools
import math

import torch
import torch.nn.functional as F

import paper_2406_16282_amd as lmbp
from paper_2406_16282_amd import nn as lnn

DEVICE = "cuda:0"
DTYPES = {"bf16": torch.bfloat16, "fp32": torch.float32}
BYTES = {"bf16": 2, "fp32": 4}
NORM_EPS = {"msln": 1e-6, "msrms": 1e-5}


def listed():
    return [
        # The norm of one ViT-B image in fp32: the smallest call, all launch and host cost.
        {"name": "norm_vit_b_image_fp32", "kind": "norm", "op": "msln", "dtype": "fp32", "rows": 197, "cols": 768,
         "x_std": 1.0, "g_std": 1.0, "outliers": False},
        # A norm of ViT-B fine-tuning at batch 64 (24 of these in a step).
        {"name": "norm_vit_b_bs64_bf16", "kind": "norm", "op": "msln", "dtype": "bf16", "rows": 64 * 197, "cols": 768,
         "x_std": 1.5, "g_std": 1e-2, "outliers": False},
        # A norm of LLaMA-7B fine-tuning, 4 sequences of 2048.
        {"name": "norm_llama7b_bf16", "kind": "norm", "op": "msrms", "dtype": "bf16", "rows": 4 * 2048, "cols": 4096,
         "x_std": 1.0, "g_std": 1e-3, "outliers": False},
        # A width that no vector divides: rows start at any element.
        {"name": "norm_odd_width_bf16", "kind": "norm", "op": "msln", "dtype": "bf16", "rows": 2439, "cols": 1025,
         "x_std": 1.0, "g_std": 1.0, "outliers": False},
        # The MLP activation of ViT-B in fp32, batch 8.
        {"name": "act_vit_b_fp32", "kind": "act", "op": "regelu2", "dtype": "fp32", "rows": 8 * 197, "cols": 3072,
         "x_std": 1.0, "g_std": 1.0, "outliers": False},
        # The gated activation of LLaMA-13B fine-tuning with outlier channels, 2 sequences of 4096.
        {"name": "glu_llama13b_outliers_bf16", "kind": "glu", "dtype": "bf16", "rows": 2 * 4096, "cols": 13824,
         "x_std": 1.0, "g_std": 1e-3, "outliers": True},
        # A fitted 4-bit member of the family on the ViT-B MLP at batch 64.
        {"name": "kbit4_gelu_vit_b_bs64_bf16", "kind": "kbit", "act": "gelu", "bits": 4, "dtype": "bf16",
         "rows": 64 * 197, "cols": 3072, "x_std": 1.5, "g_std": 1e-2},
        # The first MLP projection of ViT-B with ReGELU2, one training step at batch 64.
        {"name": "linear_vit_b_bs64_train", "kind": "linear_train", "act": "gelu", "m": 64 * 197, "n": 3072, "k": 768,
         "bias": True},
        # The same layer evaluated on one image.
        {"name": "linear_vit_b_image_eval", "kind": "linear_eval", "act": "gelu", "m": 197, "n": 3072, "k": 768,
         "bias": True},
        # LLaMA-7B's MLP input side while 16 sequences are generated token by token.
        {"name": "glu_llama7b_decode_16", "kind": "glu_eval", "m": 16, "n": 11008, "k": 4096},
        # LLaMA-7B's norm + MLP input side on one sequence of 2048, tensors kept for the backward.
        {"name": "norm_glu_llama7b_2048", "kind": "norm_glu", "m": 2048, "n": 11008, "k": 4096},
        # A whole LLaMA-7B MLP block, one training step on 4 sequences of 2048: the largest call.
        {"name": "mlp_llama7b_train", "kind": "mlp_train", "m": 4 * 2048, "n": 11008, "k": 4096},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


# (features, hidden features) of the MLPs in this repository's configurations, and others
# of the same kind: (input, output) of the first projection.
_GELU_LAYERS = ((768, 3072), (768, 3072), (512, 2048), (1024, 4096), (1000, 4000))
_GLU_LAYERS = ((4096, 11008), (4096, 11008), (5120, 13824), (2048, 5632), (520, 4112))


def draw(rng):
    kind = rng.choice(("norm", "norm", "norm", "act", "act", "glu", "kbit", "kbit", "linear_train", "linear_eval",
                       "linear_eval", "glu_eval", "glu_eval", "norm_glu", "mlp_train"))
    if kind == "norm":
        op, dtype = rng.choice(("msln", "msrms")), rng.choice(("bf16", "bf16", "fp32"))
        cols = rng.choice((768, 1024, 4096, 5120, 1000, 1023, 1025, 8191, _log_int(rng, 100, 16000),
                           _log_int(rng, 100, 16000)))
        rows = _log_int(rng, 1, max(2, min(16384, 60_000_000 // cols)))
        return {"kind": kind, "op": op, "dtype": dtype, "rows": rows, "cols": cols, "x_std": rng.choice((1.0, 1.5)),
                "g_std": rng.choice((1.0, 1e-2, 1e-3)), "outliers": rng.random() < 0.25}
    if kind in ("act", "glu", "kbit"):
        dtype = rng.choice(("bf16", "bf16", "fp32"))
        cols = rng.choice((3072, 4096, 11008, 13824, 1000, 1023, 8191, _log_int(rng, 500, 14000)))
        rows = _log_int(rng, 8, 110_000_000 // cols)
        case = {"kind": kind, "dtype": dtype, "rows": rows, "cols": cols, "x_std": rng.choice((1.0, 1.5, 2.0)),
                "g_std": rng.choice((1.0, 1e-2, 1e-3))}
        if kind == "kbit":
            return dict(case, act=rng.choice(("gelu", "silu")), bits=rng.choice((1, 2, 3, 4)))
        case["outliers"] = rng.random() < 0.25
        return dict(case, op=rng.choice(("regelu2", "resilu2"))) if kind == "act" else case
    if kind.startswith("linear"):
        k, n = rng.choice(_GELU_LAYERS)
        return {"kind": kind, "act": rng.choice(("gelu", "gelu", "silu")), "m": _log_int(rng, 1, 16384), "n": n, "k": k,
                "bias": rng.random() < 0.75}
    k, n = rng.choice(_GLU_LAYERS)
    if kind == "mlp_train":
        return {"kind": kind, "m": _log_int(rng, 64, 4096), "n": n, "k": k}
    return {"kind": kind, "m": _log_int(rng, 1, 4096), "n": n, "k": k}


# ------------------------------------------------------------------------- inputs

def _normal(gen, shape, std, dtype, outliers=False):
    x = torch.randn(shape, generator=gen, device=DEVICE, dtype=torch.float32) * std
    if outliers:   # 1% of the values from N(0, 30^2)
        big = torch.rand(shape, generator=gen, device=DEVICE) < 0.01
        x = torch.where(big, torch.randn(shape, generator=gen, device=DEVICE) * 30.0, x)
    return x.to(dtype)


def _tables(case):
    """Evenly spaced biases and the slopes of act's combination: the secants of act."""
    count = 1 << case["bits"]
    edge = 3.2 if case["act"] == "gelu" else 6.4
    thresholds = [0.0] if count == 2 else [-edge + 2 * edge * i / (count - 2) for i in range(count - 1)]
    f = (lambda v: v * 0.5 * math.erfc(-v / math.sqrt(2.0))) if case["act"] == "gelu" else \
        (lambda v: v / (1.0 + math.exp(-v)))
    inner = [(f(b) - f(a)) / (b - a) for a, b in zip(thresholds, thresholds[1:])]
    return thresholds, [0.0] + inner + [1.0]


@functools.lru_cache(maxsize=1)
def _gen():
    return torch.Generator(device=DEVICE)


def _inputs(case, seed):
    gen = _gen()
    gen.manual_seed(seed)
    kind = case["kind"]
    if kind in ("norm", "act", "glu", "kbit"):
        shape, dt = (case["rows"], case["cols"]), DTYPES[case["dtype"]]
        out = {"x": _normal(gen, shape, case["x_std"], dt, case.get("outliers", False)),
               "dy": _normal(gen, shape, case["g_std"], dt)}
        if kind == "glu":
            out["u"] = _normal(gen, shape, 1.0, dt)
        return out
    m, n, k = case["m"], case["n"], case["k"]
    dt = torch.bfloat16
    out = {"x": _normal(gen, (m, k), 1.0, dt), "w": _normal(gen, (n, k), 2.0 / math.sqrt(k), dt)}
    if case.get("bias"):
        out["b"] = _normal(gen, (n,), 0.1, dt)
    if kind in ("glu_eval", "norm_glu", "mlp_train"):
        out["w_up"] = _normal(gen, (n, k), 1.0 / math.sqrt(k), dt)
    if kind == "linear_train":
        out["dy"] = _normal(gen, (m, n), 1e-2, dt)
    if kind == "mlp_train":
        out["w_down"] = _normal(gen, (k, n), 1.0 / math.sqrt(n), dt)
        out["dy"] = _normal(gen, (m, k), 1e-3, dt)
    return out


def _linear(cls, k, n, weight, bias=None):
    layer = cls(k, n, bias=bias is not None, device=DEVICE, dtype=torch.bfloat16)
    layer.weight = torch.nn.Parameter(weight)
    if bias is not None:
        layer.bias = torch.nn.Parameter(bias)
    return layer


def prepare(case, seed):
    kind, t = case["kind"], _inputs(case, seed)
    state = {"case": case, "t": t}
    if kind == "kbit":
        state["tables"] = _tables(case)
    elif kind in ("linear_train", "linear_eval"):
        cls = lnn.LinearReGELU2 if case["act"] == "gelu" else lnn.LinearReSiLU2
        state["layer"] = _linear(cls, case["k"], case["n"], t["w"], t.get("b"))
    elif kind in ("glu_eval", "mlp_train"):
        layer = lnn.LinearReSwiGLU2(case["k"], case["n"], device="meta")
        layer.gate.weight, layer.up.weight = torch.nn.Parameter(t["w"]), torch.nn.Parameter(t["w_up"])
        state["layer"] = layer
        if kind == "mlp_train":
            state["norm"] = lnn.MSRMSNorm(NORM_EPS["msrms"])
            state["down"] = _linear(torch.nn.Linear, case["n"], case["k"], t["w_down"])
    if kind in ("linear_train", "mlp_train"):
        t["x"].requires_grad_(True)
    return state


# --------------------------------------------------------------------------- runs

def run(state):
    case, t = state["case"], state["t"]
    kind = case["kind"]
    if kind == "norm":
        if case["op"] == "msln":
            z, rstd = lmbp.msln_fwd(t["x"], NORM_EPS["msln"])
            dx = lmbp.msln_bwd(t["dy"], z, rstd)
        else:
            z, rstd = lmbp.msrms_fwd(t["x"], NORM_EPS["msrms"])
            dx = lmbp.msrms_bwd(t["dy"], z, rstd)
        return {"z": z, "rstd": rstd, "dx": dx}
    if kind == "act":
        if case["op"] == "regelu2":
            y, codes = lmbp.regelu2_fwd(t["x"])
            dx = lmbp.regelu2_bwd(t["dy"], codes)
        else:
            y, codes = lmbp.resilu2_fwd(t["x"])
            dx = lmbp.resilu2_bwd(t["dy"], codes)
        return {"y": y, "codes": codes, "dx": dx}
    if kind == "glu":
        h, s, codes = lmbp.reswiglu2_fwd(t["x"], t["u"])
        dg, du = lmbp.reswiglu2_bwd(t["dy"], t["u"], s, codes)
        return {"h": h, "s": s, "codes": codes, "dg": dg, "du": du}
    if kind == "kbit":
        thresholds, levels = state["tables"]
        y, codes = lmbp.stepact_fwd(t["x"], case["act"], thresholds, case["bits"])
        dx = lmbp.stepact_bwd(t["dy"], codes, levels, case["bits"])
        return {"y": y, "codes": codes, "dx": dx}
    if kind == "linear_train":
        layer = state["layer"]
        y = layer(t["x"])
        wrt = {"dx": t["x"], "dw": layer.weight}
        if layer.bias is not None:
            wrt["db"] = layer.bias
        return dict(zip(wrt, torch.autograd.grad(y, list(wrt.values()), t["dy"])), y=y)
    if kind in ("linear_eval", "glu_eval"):
        with torch.no_grad():
            return {"y": state["layer"](t["x"])}
    if kind == "norm_glu":
        h, s, u, codes, z, rstd = lmbp.msrms_linear_swiglu_fwd(t["x"], t["w"], t["w_up"], NORM_EPS["msrms"])
        return {"h": h, "s": s, "u": u, "codes": codes, "z": z, "rstd": rstd}
    layer, down = state["layer"], state["down"]
    y = down(layer(state["norm"](t["x"])))
    wrt = {"dx": t["x"], "dw_gate": layer.gate.weight, "dw_up": layer.up.weight, "dw_down": down.weight}
    return dict(zip(wrt, torch.autograd.grad(y, list(wrt.values()), t["dy"])), y=y)


# -------------------------------------------------------------- work and tolerance

def work(case):
    """Each input read once, each output (and tensor kept for the backward) written once;
    a backward reads its gradient and what the forward kept."""
    kind = case["kind"]
    if kind in ("norm", "act", "glu", "kbit"):
        count, b = case["rows"] * case["cols"], BYTES[case["dtype"]]
        if kind == "norm":
            return {"bytes": 5 * b * count + 8 * case["rows"], "flops": 12 * count}
        per = 32 // case.get("bits", 2)
        codes = 2 * 4 * -(-count // per)
        return {"bytes": (9 if kind == "glu" else 4) * b * count + codes, "flops": 25 * count}
    m, n, k = case["m"], case["n"], case["k"]
    gemm = 2 * m * n * k
    codes = m * n // 4
    if kind == "linear_eval":
        return {"bytes": 2 * (m * k + n * k + m * n) + codes, "flops": gemm}
    if kind == "linear_train":
        return {"bytes": 2 * (m * k + n * k + m * n) + codes + 2 * (m * n + 2 * m * k + 2 * n * k) + codes,
                "flops": 3 * gemm}
    if kind == "glu_eval":
        return {"bytes": 2 * (m * k + 2 * n * k + 3 * m * n) + codes, "flops": 2 * gemm}
    if kind == "norm_glu":
        return {"bytes": 2 * (2 * m * k + 2 * n * k + 3 * m * n) + codes + 4 * m, "flops": 2 * gemm}
    return {"bytes": 2 * (3 * n * k + 3 * m * k + 4 * m * n) + codes + 2 * (6 * n * k + 4 * m * k + 3 * m * n) + codes,
            "flops": 9 * gemm}


def tolerance(case):
    """bf16 results are one rounding of an fp32 value: two correct orders of the sums
    before it differ in single roundings (one step is 2^-8 to 2^-7 of a value, and fewer
    than one value in a thousand turns). fp32 results differ by the order of their sums
    and the last bits of exp and rsqrt. Codes of a stored input are decided exactly; codes
    of a matrix product may turn where its sum's last bits cross a bias or a rounding tie.
    Limits are about four times what the products showed against sums over two halves of k
    (norm_glu: rel 7e-5, max 0.015, 3e-6 of the code words; mlp_train: 1.5e-4, 0.043)."""
    kind = case["kind"]
    if kind in ("norm", "act", "glu", "kbit"):
        if case["dtype"] == "fp32":
            return {"rel": 1e-6, "max": 1e-5, "differ": 0.0}
        return {"rel": 3e-4, "max": 3.2e-2, "differ": 0.0}
    size = case["m"] * case["n"]
    # a code that turns at the middle bias changes one gradient value by its own size
    turned = 3.0 / math.sqrt(size)
    if kind == "mlp_train":
        # single roundings of z, s, u and h travel through the down projection and back
        return {"rel": 6e-4 + turned, "max": 0.2, "differ": 0.0}
    return {"rel": 3e-4 + (turned if kind == "linear_train" else 0.0), "max": 6e-2, "differ": min(1e-2, 2e-5 + 32.0 / size)}


# -------------------------------------------------------------------- 64-bit values

# The three-ReLU combinations: weights a1, a2 (the third makes the sum 1) and biases.
_STEPS = {
    "gelu": ((-0.04922261145617846, 1.0979632065417297),
             (-3.1858810036855245, -0.001178821281161997, 3.190832613414926)),
    "silu": ((-0.04060357190528599, 1.080925428529668),
             (-6.3050461001646445, -0.0008684942046214787, 6.325815242089708)),
}


def _act64(x, act):
    if act == "gelu":
        return x * 0.5 * torch.special.erfc(x * -math.sqrt(0.5))
    return x * torch.sigmoid(x)


def _slope64(x, thresholds, levels):
    code = torch.zeros(x.shape, dtype=torch.int64, device=x.device)
    for c in thresholds:
        code += x > c
    return torch.tensor(levels, dtype=torch.float64, device=x.device)[code]


def _step64(x, act):
    (a1, a2), c = _STEPS[act]
    return _slope64(x, c, (0.0, a1, a1 + a2, 1.0))


def _norm64(x, op):
    h = x - x.mean(-1, keepdim=True) if op == "msln" else x
    rstd = (h.square().mean(-1, keepdim=True) + NORM_EPS[op]).rsqrt()
    return h * rstd, rstd


def _norm_back64(dz, z, rstd, op):
    d = dz - z * (z * dz).mean(-1, keepdim=True)
    return rstd * (d - dz.mean(-1, keepdim=True) if op == "msln" else d)


@torch.no_grad()
def exact(case, seed):
    kind = case["kind"]
    t = {name: v.double() for name, v in _inputs(case, seed).items()}
    x = t["x"]
    if kind == "norm":
        z, rstd = _norm64(x, case["op"])
        return {"z": z, "rstd": rstd.reshape(-1), "dx": _norm_back64(t["dy"], z, rstd, case["op"])}
    if kind == "act":
        act = "gelu" if case["op"] == "regelu2" else "silu"
        return {"y": _act64(x, act), "codes": None, "dx": t["dy"] * _step64(x, act)}
    if kind == "kbit":
        return {"y": _act64(x, case["act"]), "codes": None, "dx": t["dy"] * _slope64(x, *_tables(case))}
    if kind == "glu":
        s = _act64(x, "silu")
        return {"h": s * t["u"], "s": s, "codes": None, "dg": t["dy"] * t["u"] * _step64(x, "silu"),
                "du": t["dy"] * s}
    if kind in ("linear_train", "linear_eval"):
        pre = F.linear(x, t["w"], t.get("b"))
        y = _act64(pre, case["act"])
        if kind == "linear_eval":
            return {"y": y}
        dp = t["dy"] * _step64(pre, case["act"])
        out = {"dx": dp @ t["w"], "dw": dp.t() @ x, "y": y}
        return dict(out, db=dp.sum(0)) if "b" in t else out
    z, rstd = _norm64(x, "msrms") if kind != "glu_eval" else (x, None)
    g, u = z @ t["w"].t(), z @ t["w_up"].t()
    s = _act64(g, "silu")
    if kind == "glu_eval":
        return {"y": s * u}
    if kind == "norm_glu":
        return {"h": s * u, "s": s, "u": u, "codes": None, "z": z, "rstd": rstd.reshape(-1)}
    h = s * u
    dy = t["dy"]
    dh = dy @ t["w_down"]
    dg, du = dh * u * _step64(g, "silu"), dh * s
    dz = dg @ t["w"] + du @ t["w_up"]
    return {"dx": _norm_back64(dz, z, rstd, "msrms"), "dw_gate": dg.t() @ z, "dw_up": du.t() @ z,
            "dw_down": dy.t() @ h, "y": h @ t["w_down"].t()}
