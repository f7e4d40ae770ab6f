"""The natively marshalled calls: the same results and the same refusals as the calls that Python marshals."""
import pytest

from paper_2502_20493_amd import binding as ukst

pytestmark = pytest.mark.gpu


class _Spy:
    """The extension module, keeping what its functions returned."""

    def __init__(self, module):
        self.module, self.results = module, []

    def __getattr__(self, name):
        def call(*args):
            self.results.append(getattr(self.module, name)(*args))
            return self.results[-1]
        return call


@pytest.fixture
def native(monkeypatch):
    module = ukst._load_native()
    assert module is not ukst._Ctypes
    spy = _Spy(module)
    monkeypatch.setattr(ukst, "_native", spy)
    return spy


def _calls(x, w, dy, bias, stream):
    """Pairs of (native call, the same call marshalled in Python): an explicit stream is never marshalled natively."""
    n, P, (H, W) = w.shape[2], 1, x.shape[2:]
    F = ukst.ukst_conv_transpose2d
    yield lambda: F(x, w, P), lambda: F(x, w, P, stream=stream)
    yield lambda: F(x, w, P, workspace=None), lambda: F(x, w, P, workspace=None, stream=stream)
    for f in (ukst.ukst_conv_transpose2d_ws, ukst.ukst_conv_transpose2d_bias_act):
        for kw in (dict(), dict(bias=bias), dict(bias=bias, act=ukst.UKST_ACT_TANH)):
            yield lambda: f(x, w, P, **kw), lambda: f(x, w, P, stream=stream, **kw)
    # act=None is no activation, with the bias or without
    for f in (ukst.ukst_conv_transpose2d_ws, ukst.ukst_conv_transpose2d_bias_act):
        for b in (None, bias):
            for ws in (None, False):
                yield (lambda: f(x, w, P, bias=b, act=None, workspace=ws),
                       lambda: f(x, w, P, bias=b, act=ukst.UKST_ACT_NONE, workspace=ws, stream=stream))
                yield (lambda: f(x, w, P, bias=b, act=ukst.UKST_ACT_NONE, workspace=ws),
                       lambda: f(x, w, P, bias=b, act=None, workspace=ws, stream=stream))
    yield (lambda: ukst.ukst_conv_transpose2d_grad_input(dy, w, H, W, P),
           lambda: ukst.ukst_conv_transpose2d_grad_input(dy, w, H, W, P, stream=stream))
    yield (lambda: ukst.ukst_conv_transpose2d_grad_weight(x, dy, n, P),
           lambda: ukst.ukst_conv_transpose2d_grad_weight(x, dy, n, P, stream=stream))
    yield lambda: ukst.ukst_conv_transpose2d_strided(x, w, P, 3), lambda: ukst.ukst_conv_transpose2d_strided(x, w, P, 3, stream=stream)
    yield lambda: ukst.ukst_dilated_conv2d(x, w, P, 2), lambda: ukst.ukst_dilated_conv2d(x, w, P, 2, stream=stream)


@pytest.mark.parametrize("side", [False, True])
@pytest.mark.parametrize("dtype", ["float32", "bfloat16"])
def test_same_results(dtype, side, native):
    import torch
    t = getattr(torch, dtype)
    x, w = torch.randn(2, 70, 9, 8, device="cuda").to(t), torch.randn(24, 70, 4, 4, device="cuda").to(t)
    dy, bias = torch.randn(2, 24, 16, 14, device="cuda").to(t), torch.randn(24, device="cuda")
    torch.cuda.synchronize()
    s = torch.cuda.Stream() if side else torch.cuda.current_stream()
    with torch.cuda.stream(s):
        for first, plain in _calls(x, w, torch.nn.Parameter(dy), bias, s):
            native.results.clear()
            a = first()
            assert len(native.results) == 1 and native.results[0] is a  # (marshalled natively, and at once)
            b = plain()
            assert len(native.results) == 1
            assert a.dtype == b.dtype and a.shape == b.shape and not a.requires_grad
            s.synchronize()
            assert torch.equal(a, b)
    if dtype == "bfloat16":
        native.results.clear()
        assert ukst.ukst_conv_transpose2d(x, w, 1, out_bf16=True).dtype == torch.bfloat16
        assert native.results[0] is not None


def _error(call):
    with pytest.raises((ValueError, TypeError, RuntimeError)) as e:
        call()
    return type(e.value), str(e.value)


def test_same_refusals(native):
    import torch
    s = torch.cuda.current_stream()
    x, w = torch.zeros(1, 4, 6, 6, device="cuda"), torch.zeros(8, 4, 3, 3, device="cuda")
    F, G = ukst.ukst_conv_transpose2d_ws, ukst.ukst_conv_transpose2d_grad_weight
    big = torch.zeros(8, 4, 8, 8, device="cuda")   # a kernel side that the library does not take
    for call in (lambda **k: F(x.cpu(), w, 1, **k), lambda **k: F(x, w.double(), 1, **k), lambda **k: F(x, w.to(torch.bfloat16), 1, **k),
                 lambda **k: F(x.transpose(2, 3)[:, :, 1:], w, 1, **k), lambda **k: F(x, w[:, :3].contiguous(), 1, **k),
                 lambda **k: F(x, w, -1, **k), lambda **k: F(x, big, 1, **k), lambda **k: F(x, w, 1 << 29, **k),
                 lambda **k: F(x[0], w, 1, **k), lambda **k: F(x, w, 1, bias=torch.zeros(7, device="cuda"), **k),
                 lambda **k: F(x, w, 1, out_bf16=True, **k), lambda **k: F(x, w, 1, act=7, **k),
                 lambda **k: F(x[:, :, :1, :1].contiguous(), w, 0, **k), lambda **k: F(torch.zeros(1, 4, 0, 5, device="cuda"), w, 2, **k),
                 lambda **k: G(x, x, 3, 1, **k), lambda **k: ukst.ukst_conv_transpose2d_grad_input(x, w, 5, 5, 1, **k),
                 lambda **k: ukst.ukst_dilated_conv2d(x, w, 0, 9, **k), lambda **k: ukst.ukst_dilated_conv2d(x, w, 0, 4, **k),
                 lambda **k: ukst.ukst_conv_transpose2d_strided(x, big, 1, 3, **k)):
        native.results.clear()
        assert _error(call) == _error(lambda: call(stream=s))
        assert native.results and all(r is None for r in native.results)
