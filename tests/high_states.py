"""Tensors whose ragged last chunk brings rANS states into the top of their interval, [0xFFFF0000, 2^32).

Random weights do that about once per million of lanes; here the exponents of a lane's last 1..8 elements are searched for
with the coding function written out, under the table that the tensor will have.
"""
import numpy as np

from oracle import oracle as O

HIGH = 0xFFFF0000
TURN, RUN, STATES = 128, 8, 16


def states_after(freq, sequences):
    """States after coding the symbols of every row, last one first, from 2^16 on: x <- (x / f) * 4096 + x mod f + cum, a word
    given away before where x >= f * 2^20."""
    freq = np.asarray(freq, dtype=np.uint64)
    cum = np.concatenate([[0], np.cumsum(freq)[:-1]]).astype(np.uint64)
    x = np.full(len(sequences), 1 << 16, np.uint64)
    for t in range(sequences.shape[1] - 1, -1, -1):
        f, c = freq[sequences[:, t]], cum[sequences[:, t]]
        x = np.where(x >= f << np.uint64(20), x >> np.uint64(16), x)
        x = x // f * np.uint64(4096) + x % f + c
    return x


def high_sequences(freq, symbols, length, seed, prefixes=1 << 17, most=64):
    """Some sequences of `length` (3 or more) of `symbols` after which the state is high: ways of going on for two symbols from
    random ones.  A step ends high where x / f was 2^20 - 16 or more in front of it."""
    rng = np.random.default_rng(seed)
    freq = np.asarray(freq)
    found = np.zeros((0, length), np.int64)
    for _ in range(16):
        later = symbols[rng.integers(0, symbols.size, (prefixes, length - 2))]
        for second in rng.permutation(symbols)[:16]:
            seqs = np.column_stack([np.full(prefixes, second), later])
            x = states_after(freq, seqs)
            for first in rng.permutation(symbols)[:16]:
                f = np.uint64(freq[first])
                hits = seqs[(x >= f * np.uint64((1 << 20) - 16)) & (x < f << np.uint64(20))]
                found = np.concatenate([found, np.column_stack([np.full(len(hits), first), hits])])
        if len(found) >= most:
            break
    assert len(found) == 0 or (states_after(freq, found) >= HIGH).all()
    return found[rng.permutation(len(found))[:most]]


def tail_lanes(end):
    """(lane, first element in the chunk, elements) of every lane with elements in the incomplete turn."""
    first = end // TURN * TURN
    rest = end - first
    return [(j, first + j * RUN, min(rest - j * RUN, RUN)) for j in range(STATES) if rest > j * RUN]


class Bf16:
    """Exponents of bf16 words.  The mantissas of those that are set are zero."""
    mask, shift, keep = 0x7F80, 7, 0x8000


class F16:
    """Upper bytes of binary16 words."""
    mask, shift, keep = 0xFF00, 8, 0x00FF


class F32:
    """Exponents of binary32 words."""
    mask, shift, keep = 0x7F800000, 23, 0x807FFFFF


def symbols_of(words, kind):
    return ((words & words.dtype.type(kind.mask)) >> words.dtype.type(kind.shift)).astype(np.int64)


def with_symbol(words, symbols, kind):
    return (words & words.dtype.type(kind.keep)) | (np.asarray(symbols).astype(words.dtype) << words.dtype.type(kind.shift))


def end_on_high_states(words, end, freq, kind, seed):
    """words with the lanes of the last chunk's incomplete turn, where they have seven elements or more, replaced by ones that
    end high under `freq`, as far as the tensor has the symbols for them.  The symbols that go in the tail come from the chunks before, which get those that were there: the
    tensor's counts are what they were, and so is its own table."""
    words, base = words.copy(), len(words) - end
    body = symbols_of(words[:base], kind)
    free = {int(s): list(np.flatnonzero(body == s)) for s in np.unique(body)}
    often = np.array([s for s, at in free.items() if len(at) >= 3])
    sequences = {}
    for j, first, n in tail_lanes(end):
        if n < 7:
            continue
        if n not in sequences:
            sequences[n] = high_sequences(freq, often, n, seed + n)
        for sequence in np.roll(sequences[n], j, axis=0):
            at = slice(base + first, base + first + n)
            if all(len(free.get(int(s), [])) >= (sequence == s).sum() for s in sequence):
                there = [free[int(s)].pop() for s in sequence]
                words[there] = with_symbol(words[there], symbols_of(words[at], kind), kind)
                words[at] = with_symbol(words[at], sequence, kind)
                break
    return words


def high_lanes(container, end):
    """Lanes of the last chunk's incomplete turn whose state after that turn is high, by the oracle's container: its states
    if the chunk has no other turns, else decoded down to there by the coding function's inverse."""
    info = O.blob_info(container)
    freq = info["freq"].astype(np.int64)
    cum = np.concatenate([[0], np.cumsum(freq)])
    at = O.sections(container)
    states = container[slice(*at["states"])].view(np.uint32)[-STATES:]
    lens = container[slice(*at["lens"])].reshape(-1, STATES).astype(np.int64)
    words = container[slice(*at["words"])].view(np.uint16)[:info["total_words"]]
    runs = words[info["total_words"] - int(lens[-1].sum()):]
    high = []
    begin = 0
    for j, _, n in tail_lanes(end):
        begin = int(lens[-1][:j].sum())
        x, wp = int(states[j]), begin
        for _ in range(end // TURN * RUN):
            s = int(np.searchsorted(cum, x & 4095, side="right")) - 1
            x = int(freq[s]) * (x >> 12) + (x & 4095) - int(cum[s])
            if x < 1 << 16:
                x, wp = x << 16 | int(runs[wp]), wp + 1
        if x >= HIGH:
            high.append(j)
    return high
