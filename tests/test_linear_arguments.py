"""The linear calls of the binding refuse tensors that are not what the kernels take them for, without a GPU: stand-ins for the
tensors, and nothing reaches the library.
"""
import types

import pytest
import torch

from paper_2410_20650_amd import binding as nz

TOKENS, IN, OUT = 3, 256, 40


class Stub:
    """What the binding asks of a tensor."""

    def __init__(self, numel, dtype, cuda=True, contiguous=True):
        self.is_cuda, self.dtype, self.device = cuda, dtype, "cuda:0"
        self._numel, self._contiguous = numel, contiguous

    def numel(self):
        return self._numel

    def is_contiguous(self):
        return self._contiguous

    def element_size(self):
        return self.dtype.itemsize

    def data_ptr(self):
        return 0x1000


def x_of(numel=TOKENS * IN, dtype=torch.bfloat16, **kw):
    return Stub(numel, dtype, **kw)


def f32(numel, dtype=torch.float32, **kw):
    return Stub(numel, dtype, **kw)


BAD = {
    "x float32": (TypeError, dict(x=x_of(dtype=torch.float32))),
    "x on the host": (TypeError, dict(x=x_of(cuda=False))),
    "x strided": (TypeError, dict(x=x_of(contiguous=False))),
    "x with a remainder": (ValueError, dict(x=x_of(TOKENS * IN + 1))),
    "y short": (TypeError, dict(ys=[f32(TOKENS * OUT - 1)])),
    "y bf16": (TypeError, dict(ys=[f32(TOKENS * OUT, torch.bfloat16)])),
    "y on the host": (TypeError, dict(ys=[f32(TOKENS * OUT, cuda=False)])),
    "y strided": (TypeError, dict(ys=[f32(TOKENS * OUT, contiguous=False)])),
    "two results": (ValueError, dict(ys=[f32(TOKENS * OUT)] * 2)),
    "two widths": (ValueError, dict(outs=[OUT, OUT])),
    "two biases": (ValueError, dict(biases=[None, None])),
    "bias short": (TypeError, dict(biases=[f32(OUT - 1)])),
    "bias bf16": (TypeError, dict(biases=[f32(OUT, torch.bfloat16)])),
    "bias on the host": (TypeError, dict(biases=[f32(OUT, cuda=False)])),
    "bias strided": (TypeError, dict(biases=[f32(OUT, contiguous=False)])),
    "scratch on the host": (TypeError, dict(scratch=Stub(1 << 20, torch.uint8, cuda=False))),
    "scratch strided": (TypeError, dict(scratch=Stub(1 << 20, torch.uint8, contiguous=False))),
}


@pytest.fixture
def called(monkeypatch):
    """The names of the library's functions that are called."""
    names = []

    class Library:
        def __getattr__(self, name):
            return lambda *args: names.append(name) or 0

    monkeypatch.setattr(nz, "_lib", Library())
    monkeypatch.setattr(nz, "_stream_handle", lambda stream: None)
    return names


def arguments(x=None, outs=(OUT,), biases=None, ys=None):
    weight = types.SimpleNamespace(handle=types.SimpleNamespace(value=0x2000))
    return [weight], list(outs), IN, x or x_of(), biases, ys or [f32(TOKENS * OUT)]


@pytest.mark.parametrize("what", BAD)
def test_refused(called, what):
    error, bad = BAD[what]
    scratch = {"scratch": bad["scratch"]} if "scratch" in bad else {}
    args = arguments(**{name: value for name, value in bad.items() if name != "scratch"})
    with pytest.raises(error):
        nz.neuzip_linear_batch_scratch(*args, **scratch)
    if not scratch:
        with pytest.raises(error):
            nz.neuzip_linear_batch(*args)
    assert called == []


def test_accepted(called):
    nz.neuzip_linear_batch_scratch(*arguments(biases=[f32(OUT)]), scratch=Stub(1 << 20, torch.uint8))
    nz.neuzip_linear_batch_scratch(*arguments(biases=[None]))
    nz.neuzip_linear_batch(*arguments())
    assert called == ["neuzip_linear_batch_scratch", "neuzip_linear_batch", "neuzip_linear_batch"]
