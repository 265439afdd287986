"""What a compress call reads back while its compaction is still running (-m gpu): stream lengths, stale flags and statistics
of every tensor of a batch, call after call, with tensors of one and of many encoder workgroups.
"""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2410_20650_amd import inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def nz():
    from paper_2410_20650_amd import binding
    return binding


@pytest.mark.parametrize("sizes", [(1,), (16 * 4096,), (16 * 4096 + 1, 5, 700_001), (4096,) * 8, (300_000, 1, 65_537, 2, 90_000, 3, 1_000_003)])
def test_lengths_and_statistics_of_every_call(nz, sizes):
    blobs = None
    for call in range(12):
        ws = [inputs.gaussian_bf16(n, 5000 + 10 * call + i, device=DEV) * (2.0 ** (call % 3)) for i, n in enumerate(sizes)]
        blobs = nz.neuzip_compress_batch(ws, 7, blobs=blobs)
        for w, blob in zip(ws, blobs):
            words = inputs.bits(w)
            assert np.array_equal(nz.neuzip_histogram(blob).astype(np.uint64), O.histogram(words))
            if call in (0, 1, 11):
                assert np.array_equal(nz.neuzip_export(blob), O.compress(words, 7, threads=4))


def test_stale_flags_of_every_call(nz):
    # in turn one, another and none of three tensors leave their tables
    sizes = (40_000, 16 * 4096 * 3 + 7, 5_000)
    ws = [inputs.gaussian_bf16(n, 5200 + i, device=DEV) for i, n in enumerate(sizes)]
    blobs = None
    for call in range(9):
        blobs = nz.neuzip_compress_guarded(ws, 7, 8, blobs=blobs)
        out = call % 3
        vs = [inputs.synthetic_update(w, 5300 + call) for w in ws]
        if out < 2:
            vs[out][123 + call] = 2.0 ** 60
        assert nz.neuzip_recompress(vs, blobs) == [1 if i == out and out < 2 else 0 for i in range(3)]
        for blob, v in zip(blobs, vs):
            back = torch.empty_like(v)
            nz.neuzip_decompress(blob, back)
            nz.neuzip_check(blob)
            assert torch.equal(back.view(torch.int16), v.view(torch.int16))
