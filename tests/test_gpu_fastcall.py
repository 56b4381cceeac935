"""The native form of the binding's calls against the Python path: the same bytes for the
forms that it takes, and the Python path's results or errors for those that it declines."""

import pytest

torch = pytest.importorskip("torch")
import paper_2406_16282_amd as lmbp  # noqa: E402
from paper_2406_16282_amd import binding  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


class Sub(torch.Tensor):
    pass


def calls(shape, dtype):
    torch.manual_seed(0)
    x, y, u = (torch.randn(shape, device=DEV).to(dtype) for _ in range(3))
    z, rstd = lmbp.msln_fwd(x, 1e-6, stream=torch.cuda.current_stream())
    codes = lmbp.resilu2_fwd(x, stream=torch.cuda.current_stream())[1]
    s = lmbp.reswiglu2_fwd(x, u, stream=torch.cuda.current_stream())[1]
    yield "regelu2_fwd", (x,)
    yield "resilu2_bwd", (y, codes)
    yield "msln_fwd", (x, 1e-6)
    yield "msrms_bwd", (y, z, rstd)
    yield "reswiglu2_fwd", (x, u)
    yield "reswiglu2_bwd", (y, u, s, codes)
    if dtype == torch.bfloat16 and shape[-1] % 8 == 0:
        w, w2 = (torch.randn(48, shape[-1], device=DEV, dtype=dtype) for _ in range(2))
        yield "linear_act_fwd", (x, w)
        yield "linear_act_fwd", (x, w, torch.randn(48, device=DEV, dtype=dtype), "silu")
        yield "linear_swiglu_fwd", (x, w, w2)
        yield "msrms_linear_act_fwd", (x, w, 1e-5)
        yield "msrms_linear_act_fwd", (x, w, 1e-5, torch.randn(48, device=DEV, dtype=dtype), "gelu")
        yield "msrms_linear_swiglu_fwd", (x, w, w2, 1e-5)


def tensors(out):
    return out if isinstance(out, tuple) else (out,)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("shape", [(1,), (3, 40), (2, 5, 64), (0, 16), (7, 1023)])
def test_same_results(shape, dtype):
    lmbp.lib()
    assert binding._fast is not None
    for op, args in calls(shape, dtype):
        got = tensors(getattr(lmbp, op)(*args))
        ref = tensors(getattr(lmbp, op)(*args, stream=torch.cuda.current_stream()))   # the Python path
        sub = tensors(getattr(lmbp, op)(args[0].as_subclass(Sub), *args[1:]))          # declined
        for a, b, c in zip(got, ref, sub):
            assert type(a) is torch.Tensor and a.shape == b.shape and a.dtype == b.dtype and a.stride() == b.stride()
            assert torch.equal(a.reshape(-1).view(torch.uint8), b.reshape(-1).view(torch.uint8))
            assert torch.equal(b.reshape(-1).view(torch.uint8), c.reshape(-1).view(torch.uint8))


def test_side_stream():
    s = torch.cuda.Stream()
    x = torch.randn(513, 768, device=DEV)
    ref = lmbp.msln_fwd(x, 1e-6)
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        got = lmbp.msln_fwd(x, 1e-6)
    s.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(got, ref))


def test_declined_forms_keep_their_errors():
    x = torch.randn(4, 32, device=DEV, dtype=torch.bfloat16)
    codes = lmbp.resilu2_fwd(x)[1]
    z, rstd = lmbp.msrms_fwd(x, 1e-5)
    for kind, call in (
            (TypeError, lambda: lmbp.regelu2_fwd(x.half())), (ValueError, lambda: lmbp.regelu2_fwd(x.t())),
            (ValueError, lambda: lmbp.regelu2_fwd(x.cpu())), (TypeError, lambda: lmbp.regelu2_fwd([1.0])),
            (ValueError, lambda: lmbp.resilu2_bwd(x, codes[:1])), (ValueError, lambda: lmbp.resilu2_bwd(x, codes.long())),
            (ValueError, lambda: lmbp.msln_fwd(x[0, 0], 1e-6)), (ValueError, lambda: lmbp.msrms_bwd(x, z.float(), rstd)),
            (ValueError, lambda: lmbp.msrms_bwd(x, z, rstd.double())), (ValueError, lambda: lmbp.reswiglu2_fwd(x, z.float())),
            (TypeError, lambda: lmbp.linear_act_fwd(x.float(), x)), (ValueError, lambda: lmbp.linear_act_fwd(x, z[:, :8].contiguous())),
            (TypeError, lambda: lmbp.msrms_linear_swiglu_fwd(x, x.float(), x, 1e-5)),
            (ValueError, lambda: lmbp.msrms_linear_act_fwd(x, z[:, :8].contiguous(), 1e-5)),
            (lmbp.LmbpError, lambda: lmbp.linear_act_fwd(x, x)), (lmbp.LmbpError, lambda: lmbp.msln_fwd(x, -1.0))):
        with pytest.raises(kind):
            call()
    assert lmbp.msln_fwd(x, 1)[0].shape == x.shape   # an eps that is no float
