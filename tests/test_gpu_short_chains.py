"""GPU parity of the decoder from the entry points at the edges of its launches, and of the launch that copies its words
straight into LDS (-m gpu): whole and ragged last chunks, workgroups with one chunk, waves with and without chunks, every
number of chunks per workgroup, word runs beyond the LDS window, tables of few and of all symbols.
"""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2410_20650_amd import inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
WG = 32 * 4096      # elements of a workgroup that walks whole states


@pytest.fixture(scope="module")
def nz():
    from paper_2410_20650_amd import binding
    return binding


def decoded(nz, blob, like):
    out = torch.full_like(like, float("nan"))
    nz.neuzip_decompress(blob, out)
    nz.neuzip_check(blob)
    return out


# 8 chunks per workgroup up to 2048 chunks, 12 up to 3072, 16 beyond; a wave holds 2 chunks
@pytest.mark.parametrize("chunks", [1, 2, 7, 8, 9, 2048, 2049, 3072, 3073, 4096])
@pytest.mark.parametrize("less", [0, 1, 2047, 2049, 4095])    # elements that the last chunk is short of
@pytest.mark.parametrize("kind", ["bf16", "f32"])
def test_edges_of_the_launch_from_the_entry_points(nz, chunks, less, kind):
    n = chunks * 4096 - less
    w = (inputs.gaussian_f32 if kind == "f32" else inputs.gaussian_bf16)(n, 4100 + chunks + less, device=DEV)
    raw = torch.int32 if kind == "f32" else torch.int16
    blob = nz.neuzip_compress(w, 7)
    assert torch.equal(decoded(nz, blob, w).view(raw), w.view(raw))
    back = torch.full_like(w, float("nan"))
    nz.neuzip_decompress_batch([blob], [back])
    assert torch.equal(back.view(raw), w.view(raw))


@pytest.mark.parametrize("k, block", [(3, 0), (1, 0), (0, 0), (3, 512), (0, 32)])
@pytest.mark.parametrize("n", [8 * 4096, 9 * 4096 + 2049])
def test_lossy_and_normalised_from_the_entry_points(nz, n, k, block):
    w = inputs.student_t4_bf16(n, 4200 + k, device=DEV)
    blob = nz.neuzip_compress_blockwise(w, k, block)
    words = inputs.bits(w)
    want = O.lossy_blockwise(words, k, block) if block else O.truncate(words, k)
    assert np.array_equal(inputs.bits(decoded(nz, blob, w)), want)


@pytest.mark.parametrize("kind", ["bf16", "f16", "f32"])
def test_wide_words_from_the_entry_points(nz, kind):
    # 16 chunks of 8 bits per symbol are 64 KiB of words, more than the window: the workgroups have 12 (binary16, whose upper
    # bytes hold 8 bits too, likewise), and all of their words in LDS
    n = 3500 * 4096 + 777
    if kind == "f32":
        g = torch.Generator(device=DEV).manual_seed(4300)
        w = torch.randint(-2 ** 31, 2 ** 31, (n,), generator=g, device=DEV, dtype=torch.int64).to(torch.int32).view(torch.float32)
    else:
        w = inputs.random_bits_bf16(n, 4301, device=DEV)
        w = w.view(torch.float16) if kind == "f16" else w
    raw = torch.int32 if kind == "f32" else torch.int16
    blob = nz.neuzip_compress(w, 7)
    assert torch.equal(decoded(nz, blob, w).view(raw), w.view(raw))


def test_tables_with_steps_inside_pieces_and_on_their_edges(nz):
    # frequencies of 1 to 4095 slots, at multiples of 8 and between them; one exponent (no words at all); all 256
    rng = np.random.default_rng(4400)
    for weights in ([1, 1, 1, 1, 4092], [8, 8, 16, 4064], [7, 9, 4080], [4095, 1], [1] * 200 + [3896], [16] * 256, [1]):
        p = np.array(weights, float) / sum(weights)
        symbols = rng.choice(len(weights), size=70_001, p=p) + (0 if len(weights) == 256 else 20)
        words = (symbols.astype(np.uint16) << 7) | rng.integers(0, 128, symbols.size).astype(np.uint16)
        w = inputs.from_bits(words, device=DEV)
        blob = nz.neuzip_compress(w, 7)
        assert np.array_equal(nz.neuzip_export(blob), O.compress(words, 7, threads=4))
        assert np.array_equal(inputs.bits(decoded(nz, blob, w)), words)


# launches whose words are copied straight into LDS, from the largest tensor with entry points up to the streaming sizes
@pytest.mark.parametrize("n", [128 * WG, 128 * WG + 1, 200 * WG + 77, 256 * WG, 257 * WG - 4000, 415 * WG + 4096, 416 * WG, 416 * WG - 4095, 448 * WG + 4097, 512 * WG - 8, 512 * WG])
@pytest.mark.parametrize("k", [7, 1])
def test_both_sides_of_the_direct_copies(nz, n, k):
    w = inputs.gaussian_bf16(n, 4500 + n % 97, device=DEV)
    blob = nz.neuzip_compress(w, k)
    mask = ~((1 << (7 - k)) - 1)
    assert torch.equal(decoded(nz, blob, w).view(torch.int16), w.view(torch.int16) & mask)


def test_wide_words_at_the_size_of_the_direct_copies(nz):
    w = inputs.random_bits_bf16(420 * WG + 99, 4600, device=DEV)     # 128 KiB of words per 32 chunks: 12 to a workgroup, no direct copies
    blob = nz.neuzip_compress(w, 7)
    assert torch.equal(decoded(nz, blob, w).view(torch.int16), w.view(torch.int16))


# workgroups of fewer chunks where the words of more would not fit the window: single tensors of 4 to 8 bits per symbol, and
# batches in which such tensors are most, or few, of the elements
def wide_exponents(n, bits, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    e = torch.randint(0, 1 << bits, (n,), generator=g, device=DEV, dtype=torch.int32)
    return ((e << 7) | torch.randint(0, 128, (n,), generator=g, device=DEV, dtype=torch.int32)).to(torch.int16).view(torch.bfloat16)


@pytest.mark.parametrize("bits", [4, 5, 6, 8])
@pytest.mark.parametrize("n", [40_000, 3 * 4096, 9_000_001, 20_000_003])
def test_workgroups_as_large_as_their_words_allow(nz, n, bits):
    w = wide_exponents(n, bits, 4700 + bits)
    blob = nz.neuzip_compress(w, 7)
    assert torch.equal(decoded(nz, blob, w).view(torch.int16), w.view(torch.int16))


@pytest.mark.parametrize("sizes", [(5_000_000, 100_000), (100_000, 5_000_000), (30_000_000, 45_000_000), (70_000_000, 1_000_000)])
def test_batches_of_wide_and_narrow_exponents(nz, sizes):
    ws = [wide_exponents(sizes[0], 7, 4800), inputs.gaussian_bf16(sizes[1], 4801, device=DEV)]
    blobs = nz.neuzip_compress_batch(ws, 7)
    outs = [torch.full_like(w, float("nan")) for w in ws]
    nz.neuzip_decompress_batch(blobs, outs)
    for blob, out, w in zip(blobs, outs, ws):
        nz.neuzip_check(blob)
        assert torch.equal(out.view(torch.int16), w.view(torch.int16))
    space = torch.zeros(sum(sizes) + 256, dtype=torch.bfloat16, device=DEV)
    for at, w in zip(nz.neuzip_decompress_sequence(blobs, space), ws):
        assert torch.equal(space[at:at + w.numel()].view(torch.int16), w.view(torch.int16))


def test_a_kept_table_that_the_weights_have_left(nz):
    # exponents that the table gives one slot cost 12 bits each
    w = inputs.gaussian_bf16(4096 * 4096, 4900, device=DEV)
    (blob,) = nz.neuzip_compress_guarded([w], 7, 8)
    moved = (w.float() * 64.0).to(torch.bfloat16)
    assert nz.neuzip_recompress([moved], [blob]) == [0]
    assert 8 * blob.compressed_bytes > 14 * w.numel()
    assert torch.equal(decoded(nz, blob, moved).view(torch.int16), moved.view(torch.int16))


# the linear layer's walks with and without a branch (launches of at most 256 workgroups, and of more), lanes without a chunk
# and without a turn of their own in the half behind the entry point, columns that are copied in more than one piece
@pytest.mark.parametrize("shapes, k", [([(1, 128)], 7), ([(17, 128)], 3), ([(15, 384)], 7), ([(33, 2176)], 7), ([(130, 1152)], 0),
                                       ([(2048, 4096)], 1), ([(2100, 4096), (2100, 4096)], 7), ([(700, 8192), (3, 8192)], 3)])
@pytest.mark.parametrize("tokens", [1, 16, 40])
def test_linear_walks_at_the_edges_of_their_launches(nz, shapes, k, tokens):
    in_f = shapes[0][1]
    mask = ~((1 << (7 - k)) - 1)
    ws = [inputs.gaussian_bf16(s, 5400 + i, device=DEV) for i, s in enumerate(shapes)]
    held = [(w.view(torch.int16) & mask).view(torch.bfloat16) for w in ws]
    blobs = [nz.neuzip_compress(w, k) for w in ws]
    g = torch.Generator(device=DEV).manual_seed(5500)
    x = torch.randn((tokens, in_f), generator=g, device=DEV).to(torch.bfloat16)
    for y, w, blob in zip(nz.neuzip_linear_batch(blobs, [s[0] for s in shapes], in_f, x), held, blobs):
        nz.neuzip_check(blob)
        want, size = x.double() @ w.double().t(), x.double().abs() @ w.double().abs().t()
        assert bool(((y.double() - want).abs() <= 2 * (in_f + 64) * 2.0 ** -24 * size + 1e-30).all())   # float32 sums, any order
