"""The gradients' workspace belongs to the stream of the launch: the caller never sees it,
so only the allocator can keep another use of its memory behind the kernels that fill it."""

import contextlib

import pytest

torch = pytest.importorskip("torch")
import paper_2406_16282_amd as lmbp  # noqa: E402
from paper_2406_16282_amd import binding as B  # noqa: E402

DEV = "cuda:0"


def calls(dy, x, codes, stream):
    yield lmbp.linear_weight_grad(dy, x, stream=stream), "linear_weight_grad"
    yield lmbp.linear_act_bwd(dy, codes, x, stream=stream), "linear_act_bwd"


class Recorder:
    """Stands for the GPU: notes under which stream the workspace is allocated and launched."""

    def __init__(self, monkeypatch):
        self.current, self.work, self.launched = None, [], []
        empty = torch.empty

        def recorded(*size, dtype=None, device=None):
            if dtype is torch.uint8:
                self.work.append(self.current)
            return empty(*size, dtype=dtype)

        @contextlib.contextmanager
        def under(stream):
            before, self.current = self.current, stream
            yield
            self.current = before

        class Lib:
            lmbp_linear_grad_bytes = staticmethod(lambda *a: 64)
            lmbp_codes_bytes = staticmethod(lambda n: 4 * -(-n // 16))
            linear_weight_grad = linear_act_bwd = staticmethod(lambda *a: self.launched.append(a[-1].value) or B.OK)

        monkeypatch.setattr(B, "lib", lambda: Lib)
        monkeypatch.setattr(B, "_dev", lambda t, what: t)
        monkeypatch.setattr(B, "_device_of", lambda t: contextlib.nullcontext())
        monkeypatch.setattr(B, "_raw_stream", lambda index: 0)
        monkeypatch.setattr(torch, "empty", recorded)
        monkeypatch.setattr(torch.cuda, "stream", under)
        monkeypatch.setattr(torch.cuda, "ExternalStream", lambda handle, device=None: handle)


@pytest.mark.parametrize("stream", [None, 0x1230])
def test_allocated_on_the_launch_stream(monkeypatch, stream):
    r = Recorder(monkeypatch)
    dy, x, codes = torch.zeros(4, 16).bfloat16(), torch.zeros(4, 8).bfloat16(), torch.zeros(4, dtype=torch.int32)
    for _ in calls(dy, x, codes, stream):
        pass
    assert r.launched == [stream, stream]   # c_void_p(0).value is None: the default stream
    assert r.work == [stream, stream]


@pytest.mark.gpu
@pytest.mark.parametrize("raw", [False, True])
def test_side_stream_keeps_its_workspace(raw):
    """Work queued on a side stream delays the gradients there; memory taken and filled on
    the current stream meanwhile must neither change them nor be changed by them."""
    m, n, k = 9001, 272, 264   # rows split: partial sums in the workspace
    g = torch.Generator(device=DEV)
    g.manual_seed(1)
    dy, x = (torch.randint(-8, 9, s, generator=g, device=DEV).bfloat16() for s in ((m, n), (m, k)))
    codes = lmbp.regelu2_fwd(dy)[1]
    refs = [out if isinstance(out, tuple) else (out,) for out, _ in calls(dy, x, codes, None)]
    side = torch.cuda.Stream()
    busy = torch.randn(4096, 4096, device=DEV)
    torch.cuda.synchronize()
    for i in range(2):
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            chain = busy
            for _ in range(8):
                chain = chain @ busy * 1e-3
        op = list((lmbp.linear_weight_grad, lambda a, b, **kw: lmbp.linear_act_bwd(a, codes, b, **kw)))[i]
        out = op(dy, x, stream=side.cuda_stream if raw else side)
        nbytes = lmbp.lib().lmbp_linear_grad_bytes(m, n, k, i)
        assert nbytes > 0
        others = [torch.full((nbytes,), 0x7F, dtype=torch.uint8, device=DEV) for _ in range(4)]
        torch.cuda.synchronize()
        assert all(bool((o == 0x7F).all()) for o in others)
        for a, b in zip(out if isinstance(out, tuple) else (out,), refs[i]):
            assert torch.equal(a, b)
        del others
