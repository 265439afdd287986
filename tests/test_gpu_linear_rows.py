"""GPU parity of how the linear layer's sums leave and how it reads its activations (-m gpu): rows that end in every
turn, inside chunks, and beyond them; sums stored whole, added to the result, or stored by pieces for a second launch;
activations as they lie and laid out in scratch memory; groups with as many columns as their words fit.

The bar is the classical bound for a float32 sum in any order, |error| <= 2 (in_features + 64) 2^-24 sum |w x|, against
float64 on the CPU.
"""
import pytest
import torch

from paper_2410_20650_amd import inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def nz():
    from paper_2410_20650_amd import binding
    return binding


def within_the_bound(y, x, w, in_f, bias=None):
    x64, w64 = x.double().cpu(), w.double().cpu()
    want, mag = x64 @ w64.t(), x64.abs() @ w64.abs().t()
    if bias is not None:
        want, mag = want + bias.double().cpu(), mag + bias.double().cpu().abs()
    worst = ((y.double().cpu() - want).abs() / (2.0 * (in_f + 64) * 2.0 ** -24 * mag + 1e-30)).max().item()
    assert worst <= 1.0, worst


# rows of one turn; whole rows in halves of chunks; odd multiples of 128 (32 rows between columns); 8 and 4 rows between them
@pytest.mark.parametrize("out_f,in_f", [(700, 128), (300, 384), (260, 512), (130, 640), (90, 1920), (60, 2048), (70, 4224), (50, 5632),
                                        (40, 5120)])
@pytest.mark.parametrize("tokens", [1, 7, 8, 16, 17, 31, 33, 64, 66])
def test_rows_with_and_without_scratch(nz, out_f, in_f, tokens):
    w = inputs.gaussian_bf16((out_f, in_f), 4100 + in_f, device=DEV)
    x = inputs.gaussian_bf16((tokens, in_f), 4200 + tokens, std=1.0, device=DEV)
    bias = torch.linspace(-1, 1, out_f, dtype=torch.float32, device=DEV)
    blob = nz.neuzip_compress(w, 7)
    size = nz.neuzip_linear_scratch_bytes([out_f], in_f, tokens)
    room = torch.full((size + 64,), 0xFF, dtype=torch.uint8, device=DEV)      # (NaN in either type)
    for scratch in (None, room[:size]):
        y = torch.full((tokens, out_f), float("nan"), dtype=torch.float32, device=DEV)
        nz.neuzip_linear_batch_scratch([blob], [out_f], in_f, x, [bias], [y], scratch)
        within_the_bound(y, x, w, in_f, bias)
    assert bool((room[size:] == 0xFF).all())
    nz.neuzip_check(blob)


# enough sums for the launch that adds pieces up, at each of its three limits
@pytest.mark.parametrize("out_f,in_f", [(3600, 896), (6000, 384), (4000, 640), (11000, 1536), (2600, 1920), (1600, 4224)])
@pytest.mark.parametrize("tokens", [8, 16, 31, 64, 66])
def test_rows_by_pieces(nz, out_f, in_f, tokens):
    w = inputs.gaussian_bf16((out_f, in_f), 4150 + in_f, device=DEV)
    x = inputs.gaussian_bf16((tokens, in_f), 4250 + tokens, std=1.0, device=DEV)
    blob = nz.neuzip_compress(w, 7)
    size = nz.neuzip_linear_scratch_bytes([out_f], in_f, tokens)
    assert size > 4 * out_f * min(tokens, 64)
    room = torch.full((size + 64,), 0xFF, dtype=torch.uint8, device=DEV)
    y = torch.full((tokens, out_f), float("nan"), dtype=torch.float32, device=DEV)
    nz.neuzip_linear_batch_scratch([blob], [out_f], in_f, x, None, [y], room[:size])
    within_the_bound(y, x, w, in_f)
    assert bool((room[size:] == 0xFF).all())


# beyond the entry points: 32 columns, several groups, the last columns without a chunk
@pytest.mark.parametrize("out_f,in_f", [(26500, 640), (3600, 4736), (8200, 2048)])
@pytest.mark.parametrize("tokens", [5, 20, 50])
def test_rows_of_large_weights(nz, out_f, in_f, tokens):
    w = inputs.gaussian_bf16((out_f, in_f), 4300 + in_f, device=DEV)
    x = inputs.gaussian_bf16((tokens, in_f), 4400 + tokens, std=1.0, device=DEV)
    blob = nz.neuzip_compress(w, 7)
    within_the_bound(nz.neuzip_linear(blob, out_f, in_f, x), x, w, in_f)
    without = torch.empty((tokens, out_f), dtype=torch.float32, device=DEV)
    nz.neuzip_linear_batch_scratch([blob], [out_f], in_f, x, None, [without])
    within_the_bound(without, x, w, in_f)


# weights with entry points that share CUs, as x lies: in halves up to 20 tokens, whole beyond (weights that hold no slot table beside
# ones that do)
@pytest.mark.parametrize("in_f,outs", [(4096, (4096, 500)), (1920, (5000, 4000, 60)), (1024, (14336, 3000))])
@pytest.mark.parametrize("tokens", [20, 21, 33, 64])
def test_batches_without_scratch(nz, in_f, outs, tokens):
    ws = [inputs.gaussian_bf16((o, in_f), 4350 + i, device=DEV) for i, o in enumerate(outs)]
    x = inputs.gaussian_bf16((tokens, in_f), 4450 + tokens, std=1.0, device=DEV)
    biases = [torch.linspace(-1, 1, o, dtype=torch.float32, device=DEV) for o in outs]
    blobs = [nz.neuzip_compress(w, 7) for w in ws]
    ys = [torch.full((tokens, o), float("nan"), dtype=torch.float32, device=DEV) for o in outs]
    nz.neuzip_linear_batch_scratch(blobs, outs, in_f, x, biases, ys)
    for y, w, b, blob in zip(ys, ws, biases, blobs):
        within_the_bound(y, x, w, in_f, b)
        nz.neuzip_check(blob)


# the last calls whose waves add their sums to the result by themselves, and the first whose do not; two sets whose rows end in
# other turns
@pytest.mark.parametrize("in_f", [384, 640])
@pytest.mark.parametrize("tokens,most", [(3, 15000), (5, 2000), (6, 833), (7, 357), (16, 156)])
def test_sums_by_themselves_and_added_up(nz, in_f, tokens, most):
    x = inputs.gaussian_bf16((tokens, in_f), 4460 + tokens, std=1.0, device=DEV)
    for out_f in (most, most + 1):
        w = inputs.gaussian_bf16((out_f, in_f), 4470 + out_f, device=DEV)
        bias = torch.linspace(-1, 1, out_f, dtype=torch.float32, device=DEV)
        blob = nz.neuzip_compress(w, 7)
        within_the_bound(nz.neuzip_linear(blob, out_f, in_f, x, bias), x, w, in_f, bias)
        nz.neuzip_check(blob)


# words of 5 bits and more: groups of fewer columns than the form has, in halves and whole
@pytest.mark.parametrize("out_f,in_f", [(96, 1024), (4100, 4736)])
@pytest.mark.parametrize("tokens", [3, 40])
def test_columns_as_many_as_their_words_fit(nz, out_f, in_f, tokens):
    g = torch.Generator(device=DEV).manual_seed(4500)
    n = out_f * in_f
    expo = torch.randint(100, 140, (n,), generator=g, device=DEV, dtype=torch.int32)
    rest = torch.randint(0, 256, (n,), generator=g, device=DEV, dtype=torch.int32)
    words = ((rest & 0x80) << 8) | (expo << 7) | (rest & 0x7F)
    w = (words - 65536 * (words >= 32768)).to(torch.int16).view(torch.bfloat16).view(out_f, in_f)
    x = inputs.gaussian_bf16((tokens, in_f), 4600 + tokens, std=1.0, device=DEV)
    blob = nz.neuzip_compress(w, 7)
    within_the_bound(nz.neuzip_linear(blob, out_f, in_f, x), x, w, in_f)
    nz.neuzip_check(blob)


def test_batch_by_pieces_and_under_capture(nz):
    in_f, outs, tokens = 640, (3000, 900, 410), 24
    ws = [inputs.gaussian_bf16((o, in_f), 4700 + o, device=DEV) for o in outs]
    x = inputs.gaussian_bf16((tokens, in_f), 4701, std=1.0, device=DEV)
    biases = [torch.linspace(-1, 1, outs[0], dtype=torch.float32, device=DEV), None, None]
    blobs = [nz.neuzip_compress(w, 7) for w in ws]
    for y, w, b in zip(nz.neuzip_linear_batch(blobs, outs, in_f, x, biases), ws, biases):
        within_the_bound(y, x, w, in_f, b)
    ys = [torch.empty((tokens, o), dtype=torch.float32, device=DEV) for o in outs]
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            nz.neuzip_linear_batch(blobs, outs, in_f, x, biases, ys, stream=side)
    for _ in range(3):
        for y in ys:
            y.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for y, w, b in zip(ys, ws, biases):
            within_the_bound(y, x, w, in_f, b)


def test_scratch_arguments(nz):
    in_f, out_f, tokens = 640, 50, 40
    assert nz.neuzip_linear_scratch_bytes([out_f], in_f, nz.LINEAR_SCRATCH_TOKENS - 1) == 0
    size = nz.neuzip_linear_scratch_bytes([out_f], in_f, tokens)
    assert size >= tokens * in_f * 2
    w = inputs.gaussian_bf16((out_f, in_f), 4800, device=DEV)
    x = inputs.gaussian_bf16((tokens, in_f), 4801, std=1.0, device=DEV)
    blob = nz.neuzip_compress(w, 7)
    y = torch.empty((tokens, out_f), dtype=torch.float32, device=DEV)
    room = torch.zeros(size + 16, dtype=torch.uint8, device=DEV)
    with pytest.raises(nz.NeuzipError):
        nz.neuzip_linear_batch_scratch([blob], [out_f], in_f, x, None, [y], room[1:])     # not on 16 bytes
    nz.neuzip_linear_batch_scratch([blob], [out_f], in_f, x, None, [y], room[:size - 1])  # too small: not used
    within_the_bound(y, x, w, in_f)
    assert not bool(room.any())
