"""The linear layer's scratch memory and another thread's capture (-m gpu): a call with its result at hand allocates nothing but scratch
memory, and where that has to come from the device it neither fails nor ends the capture.
"""
import threading

import pytest
import torch

from paper_2410_20650_amd import inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("batch", [False, True])
def test_scratch_memory_while_another_thread_captures(batch):
    from paper_2410_20650_amd import binding as nz
    out_f, in_f, tokens = 520, 4096, 64
    w = inputs.gaussian_bf16((out_f, in_f), 4700, device=DEV)
    x = inputs.gaussian_bf16((tokens, in_f), 4701, std=1.0, device=DEV)
    blob = nz.neuzip_compress(w, 7)
    y = torch.zeros((tokens, out_f), dtype=torch.float32, device=DEV)
    assert nz.neuzip_linear_scratch_bytes([out_f], in_f, tokens) > 0
    side = torch.cuda.Stream()
    a = torch.ones(1000, device=DEV)
    torch.cuda.synchronize()
    failed = []

    def call():
        try:
            if batch:
                nz.neuzip_linear_batch([blob], [out_f], in_f, x, None, [y], stream=side)
            else:
                nz.neuzip_linear(blob, out_f, in_f, x, None, y, stream=side)
        except Exception as e:  # (told below: a thread's exception is nobody's)
            failed.append(e)

    graph = torch.cuda.CUDAGraph()
    torch.cuda.empty_cache()
    with torch.cuda.graph(graph):   # (the global mode)
        a += 1
        thread = threading.Thread(target=call)
        thread.start()
        thread.join()
        a += 1
    assert not failed, failed
    for k in range(1, 4):
        graph.replay()
        torch.cuda.synchronize()
        assert bool((a == 1 + 2 * k).all())
    want = x.double().cpu() @ w.double().cpu().t()
    mag = x.double().cpu().abs() @ w.double().cpu().abs().t()
    worst = ((y.double().cpu() - want).abs() / (2.0 * (in_f + 64) * 2.0 ** -24 * mag)).max().item()
    assert worst <= 1.0, worst  # (the classical bound of a float32 sum in any order)
