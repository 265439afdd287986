"""Tensors whose words exceed a decoder workgroup's LDS window in a few chunks only, and the size of the workgroups that the
library takes for them: it chooses as many chunks as fit by the tensor's average, so a tensor that is wide throughout gets
workgroups that hold all of their words, and only a tensor that is wide in places still has some that are read from the blob.
"""
import numpy as np
import torch

from paper_2410_20650_amd import inputs

DEV = "cuda:0"
CHUNK = 4096


def window(k):
    """Bytes of words that a workgroup has room for (k = 1 and 0 hold a table of their own inside it)."""
    return 62 * 1024 - {1: 2048, 0: 128}.get(k, 0)


def runs(container):
    """(bytes of words of every chunk, total bytes)."""
    nc = int(container[36:40].view(np.uint32)[0])
    offsets = container[64 + 512:64 + 512 + 4 * (nc + 1)].view(np.uint32).astype(np.int64)
    per_chunk = 2 * np.diff(offsets)
    return per_chunk, int(per_chunk.sum())


def fitting_chunks(container, k):
    per_chunk, total = runs(container)
    room = window(k) - window(k) // 100
    return max(4, min(32, room // (total // per_chunk.size + 1) // 4 * 4))


def chunks_of_a_workgroup(container, k, kind):
    """Chunks of a workgroup of a tensor's own launch."""
    nc, fit = runs(container)[0].size, fitting_chunks(container, k)
    if nc <= 4096:
        spread = (-(-nc // 256) + 3) // 4 * 4
        return min(max(8, min(16, spread)), fit)
    return min(16 if kind == "f16" else 32, fit)


def widest(container, chunks):
    """The most bytes of words that a workgroup of `chunks` chunks holds."""
    per_chunk = runs(container)[0]
    return int(max(per_chunk[i:i + chunks].sum() for i in range(0, per_chunk.size, chunks)))


def exceeds(container, chunks, k):
    """Whether the words of some workgroup of so many chunks are read from the blob."""
    return widest(container, chunks) > window(k)


def narrow_but_for(kind, n, seed, first=1000, chunks=64):
    """Gaussian, with `chunks` chunks of bits without structure from chunk `first` on (about 12 bits per symbol: the table has
    next to nothing for them)."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    at, upto = first * CHUNK, (first + chunks) * CHUNK
    assert upto <= n
    if kind == "f32":
        w = inputs.gaussian_f32(n, seed, device=DEV)
        w.view(torch.int32)[at:upto] = torch.randint(-2 ** 31, 2 ** 31, (upto - at,), generator=g, device=DEV).to(torch.int32)
        return w
    w = (inputs.gaussian_f16 if kind == "f16" else inputs.gaussian_bf16)(n, seed, device=DEV)
    w.view(torch.int16)[at:upto] = torch.randint(-2 ** 15, 2 ** 15, (upto - at,), generator=g, device=DEV).to(torch.int16)
    return w


def raw(t):
    return t.view(torch.int32 if t.dtype == torch.float32 else torch.int16)
