"""The bias arithmetic of the layer wrapper (torch only; the codec's calls are stood in for on the CPU)."""
import numpy as np
import pytest
import torch

from paper_2410_20650_amd import layer


def a_layer(out_features, in_features, bias):
    made = layer.CompressedLinear.__new__(layer.CompressedLinear)
    made.out_features, made.in_features = out_features, in_features
    made.blob, made.bias = None, bias
    made.held = torch.randn(out_features, in_features, generator=torch.Generator().manual_seed(3)).to(torch.bfloat16)
    made.weight_into = lambda space: made.held
    return made


@pytest.mark.parametrize("shape", [(), (1,), (5,), (1, 5)])
def test_forward_of_a_training_batch_is_float32_for_every_shape_of_bias(shape):
    out_features = 1 if shape in ((), (1,)) else 5
    bias = torch.full(shape, 1.0 + 2.0 ** -20)          # more bits than bf16 has
    made = a_layer(out_features, 128, bias)
    x = torch.randn(65, 128, generator=torch.Generator().manual_seed(4)).to(torch.bfloat16)
    y = made.forward(x, None)
    want = torch.matmul(x, made.held.t()).float() + bias
    assert y.dtype == torch.float32 and y.shape == (65, out_features) and torch.equal(y, want)


@pytest.mark.parametrize("lr", [0.25, 1, True, np.float32(0.25), np.float64(0.25), torch.tensor(0.25), torch.tensor([0.25])])
def test_bias_step_takes_every_rate_that_the_weight_step_takes(monkeypatch, lr):
    monkeypatch.setattr(layer.nz, "neuzip_update", lambda *args, **kw: [0])
    made = a_layer(5, 128, torch.ones(5))
    x = torch.ones(3, 128, dtype=torch.bfloat16)
    grad_y = torch.full((3, 5), 0.5, dtype=torch.bfloat16)
    space = torch.empty(5 * 128, dtype=torch.bfloat16)
    made.backward_and_update(x, grad_y, lr, space, torch.empty_like(space))
    assert torch.equal(made.bias, torch.full((5,), 1.0 - float(lr) * 1.5))
