"""GPU parity where lanes of a ragged last chunk stand at the top of the states' interval and have no symbol behind that (-m gpu):
a last chunk of less than a turn beside whole chunks of its wave, and one that ends in the turn above the entry points.
Every form of the encoder against the oracle, byte by byte, and the words that come back.
"""
import numpy as np
import pytest
import torch

import high_states as H
from oracle import oracle as O
from oracle import update as U
from paper_2410_20650_amd import inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
KINDS = {
    "bf16": (H.Bf16, inputs.gaussian_bf16, inputs.bits, 7, 0),
    "bf16 k=3": (H.Bf16, inputs.gaussian_bf16, inputs.bits, 3, 0),
    "blocks of 64": (H.Bf16, inputs.gaussian_bf16, inputs.bits, 3, 64),
    "f16": (H.F16, inputs.gaussian_f16, inputs.bits16, 7, 0),
    "f32": (H.F32, inputs.gaussian_f32, inputs.bits32, 7, 0),
}


@pytest.fixture(scope="module")
def nz():
    from paper_2410_20650_amd import binding
    return binding


def compress(name, words, **kw):
    _, _, _, k, block = KINDS[name]
    if name == "f16":
        return O.compress_f16(words, threads=8, **kw)
    if name == "f32":
        return O.compress_f32(words, threads=8, **kw)
    return O.compress(words, k, threads=8, block=block, **kw)


def on_gpu(words, like):
    signed = words.view(np.int32 if words.dtype == np.uint32 else np.int16)
    return torch.from_numpy(signed.copy()).to(DEV).view(like.dtype)


def tensor(name, n, seed):
    _, gaussian, bits, _, block = KINDS[name]
    w = gaussian(n, seed, device=DEV)
    words = bits(w).copy()
    if block:
        words &= 0xFF80   # (every block's coefficient is one, so the words that are coded are these)
    return on_gpu(words, w), words


def check(nz, name, blob, want, words, end):
    _, _, bits, k, _ = KINDS[name]
    assert H.high_lanes(want, end), (name, len(words))
    assert np.array_equal(nz.neuzip_export(blob), want), (name, len(words))
    out = on_gpu(np.zeros_like(words), torch.empty(0, dtype={"f16": torch.float16, "f32": torch.float32}.get(name, torch.bfloat16)))
    nz.neuzip_decompress(blob, out)
    nz.neuzip_check(blob)
    assert np.array_equal(bits(out), words if k == 7 else O.truncate(words, k)), (name, len(words))


@pytest.mark.parametrize("end", [7, 127, 2048 + 8, 2048 + 127])
@pytest.mark.parametrize("name", KINDS)
def test_high_states_behind_which_nothing_is_coded(nz, name, end):
    kind, _, _, k, block = KINDS[name]
    for whole in (1, 18):
        n = whole * 4096 + end
        before, words = tensor(name, n, 9000 + n)
        # fresh statistics
        high = H.end_on_high_states(words, end, O.blob_info(compress(name, words))["freq"], kind, end)
        blob = nz.neuzip_compress_blockwise(on_gpu(high, before), k, block)
        check(nz, name, blob, compress(name, high), high, end)
        if block:
            continue
        # the kept table
        (kept,) = nz.neuzip_compress_guarded([before], k, 8)
        table = nz.neuzip_frequencies(kept).copy()
        high = H.end_on_high_states(words, end, table, kind, end)
        (rebuilt,) = nz.neuzip_recompress([on_gpu(high, before)], [kept])
        assert not rebuilt
        check(nz, name, kept, compress(name, high, guard=8, freq=table), high, end)
        # the weight step, from the blob and with the weights at hand
        for mode in (0, 1) if name == "bf16" else ():
            w, g = on_gpu(high, before), torch.zeros_like(before)
            (blob,) = nz.neuzip_compress_guarded([w], 7, 8)
            want, want_rebuilt, want_words = U.training_step(nz.neuzip_export(blob), inputs.bits(g), 1e-2, threads=8)
            (rebuilt,) = nz.neuzip_update([blob], [g], [w], 1e-2, weights_ready=mode)
            assert rebuilt == want_rebuilt and np.array_equal(inputs.bits(w), want_words), (n, mode)
            check(nz, name, blob, want, high, end)
