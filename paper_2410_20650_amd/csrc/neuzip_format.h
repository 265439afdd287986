// Format constants and the device-side structures shared by the compression and decompression
// kernels of the NeuZip codec (see neuzip.hip for the stream format).
#pragma once

#include <hip/hip_runtime.h>
#include <cstddef>
#include <cstdint>
#include "neuzip.h"

namespace nz {

constexpr uint32_t kProbBits = NEUZIP_PROB_BITS;
constexpr uint32_t kM = 1u << kProbBits;
constexpr uint32_t kChunk = NEUZIP_CHUNK;
constexpr uint32_t kStates = NEUZIP_STATES_PER_CHUNK;
constexpr uint32_t kRun = NEUZIP_RUN;
constexpr uint32_t kTurn = kStates * kRun;          // symbols per turn of all states (128)
constexpr uint32_t kTurns = kChunk / kTurn;         // turns per full chunk (32)
constexpr uint32_t kRansL = 1u << 16;
// Words one state can emit for its 256 symbols.  Every step grows log2(x + 1) by at most 12 bits and
// every emitted word shrinks it by at least 16 - log2(17/16) bits, which bounds a run by 193 words.
constexpr uint32_t kRunCap = 200;
constexpr uint32_t kMagic = 0x315A554Eu;            // "NUZ1"
constexpr uint32_t kHeaderBytes = 64;

// Decoder launch shape: at most 512 threads = 8 waves, each wave walks 4 chunks (4 x 16 states).
constexpr uint32_t kDecThreads = 512;
constexpr uint32_t kDecChunksPerWg = kDecThreads / kStates;   // 32
// LDS: 16 KB slot table + staged word runs.  Two workgroups share a CU's 160 KB.
constexpr uint32_t kStageBytes = 62 * 1024;
// Turns (of 8 symbols per state) whose loads and stores are issued together: 2 for tensors that
// live in the last-level cache and for the lossy widths, 4 for lossless tensors that stream
// through HBM (more bytes in flight; measured +2-3 % there, -6 % on cache-resident sizes and
// -7 % on the lossy widths).
constexpr uint32_t kTurnGroup = 2;
constexpr uint32_t kTurnGroupStream = 4;
static_assert(kTurns % kTurnGroup == 0 && kTurns % kTurnGroupStream == 0, "a chunk is a whole number of turn groups");


// Entry points.  A state is a chain of 256 dependent decoding steps, and a tensor of few chunks does not have
// the waves to hide it: whatever its size, its decoding takes as long as the chain.  A blob of at most
// kSplitChunks chunks therefore also holds, per state, where the chain stands before turn kMidTurn -- the
// state (4 bytes) and the words consumed so far (1 byte) -- and two lanes walk the two halves.  It is derived
// data, like the tables: the encoder passes that point anyway, an import walks to it, and the container does not
// have it.  Measured, lossless, one launch per tensor, whole states / halves: 1 M elements 19.7 / 9.8 us, 4 M
// 20.4 / 10.7, 16.8 M 23.0 / 14.0; linear layer 4096 x 4096, 1 token, 28.2 / 15.3.  The line lies where the lanes
// of whole states come to one wave per SIMD (1024 waves of 64 states): beyond it the launch has waves to hide the
// chain behind (58.7 M elements with twice the lanes: no faster), and the 0.16 bits per element the entry points
// cost would be held by the matrices that make up most of a model (on an 8B-shaped layer they are 0.3 % of the
// container as it is).
constexpr uint32_t kMidTurn = kTurns / 2;
constexpr uint32_t kSplitChunks = 4096;
__host__ __device__ constexpr bool has_entry_points(uint32_t n_chunks) { return n_chunks > 0 && n_chunks <= kSplitChunks; }

// The decoder's slot table (16 KB) is held by blobs without entry points, whose decoders copy it, and by those of
// them that have at least kTableChunks chunks: in a batch beyond the cache these are walked whole beside larger
// ones, and with the table in the blob that launch is the plain one, which makes no tables (5 tensors of 16.8 M:
// 55.8 us, 56.9 with every workgroup making its own; 0.3 % of such a blob, of smaller ones it would be more).
constexpr uint32_t kTableChunks = 1024;
__host__ __device__ constexpr bool holds_table(uint32_t n_chunks) { return n_chunks >= kTableChunks; }
static_assert(kTableChunks <= kSplitChunks, "a blob without entry points holds the table");

constexpr uint32_t kSteps = 264;  // occupied symbols of a table (at most 256) and what a search reads behind them

// Division of 32-bit numbers by one that the host knows: exact for every n (round-up method, Granlund and Montgomery 1994).
struct Divisor {
    uint32_t by, mul, shift1, shift2;
    __host__ void set(uint32_t d)
    {
        uint32_t l = 0;  // ceil(log2 d)
        while (l < 32 && (1ull << l) < d)
            ++l;
        by = d;
        mul = static_cast<uint32_t>(((1ull << 32) * ((1ull << l) - d)) / d + 1);
        shift1 = l < 1 ? l : 1;
        shift2 = l < 1 ? 0 : l - 1;
    }
    __host__ __device__ __forceinline__ uint32_t quotient(uint32_t n) const
    {
        const uint32_t t = static_cast<uint32_t>((static_cast<uint64_t>(mul) * n) >> 32);
        return (t + ((n - t) >> shift1)) >> shift2;
    }
    __host__ __device__ __forceinline__ uint32_t rest(uint32_t n) const { return n - quotient(n) * by; }
};

// A launch's arguments come to a CU cache line by cache line, and a line that is first asked for when it is needed is 550
// cycles (the first of all 1000, one that is there 80): a kernel asks for all lines of `a` with its first instructions.
template <class Args>
__device__ __forceinline__ void fetch_arguments(const Args &a)
{
    const uint32_t *at = reinterpret_cast<const uint32_t *>(&a);
#pragma unroll
    for (uint32_t i = 0; i < sizeof(Args); i += 64)
        asm volatile("" ::"s"(at[i / 4]));
}

// ------------------------------------------------------------------------------------------
// Device-side table block that sits at the start of every blob's fixed allocation.
// ------------------------------------------------------------------------------------------
struct TableBlock {
    uint16_t freq[256];    // quantised frequencies (stored in the container)
    uint16_t cum[264];     // exclusive cumulative frequencies, cum[256] = 4096 (derived)
    uint32_t status[4];    // [0] != 0: a decode found a malformed stream
    uint32_t lone;         // the only exponent value of the tensor (its f is 4096), else 256
    uint32_t pad[47];
    // the occupied symbols in order (derived): cum << 8 | symbol; the rest of the array is 4096 << 8
    uint32_t steps[kSteps];
    // which of them slot 8i belongs to (derived; blobs with entry points)
    uint8_t step_of[kM / 8];
    // decoder slot table (derived): lut[slot] = symbol | f << 8 | (slot - cum[symbol]) << 20.  Small blobs do not
    // have it (their allocation ends before it, see holds_table); from the entry points every workgroup of a decoder
    // makes it from the steps, which a tensor beyond the size of those blobs, with several rounds of workgroups, would
    // pay several times (28672 x 8192: 145 us with the table read from the blob, 161 us without).
    uint32_t lut[kM];
};
constexpr uint64_t table_bytes(bool with_lut) { return with_lut ? sizeof(TableBlock) : offsetof(TableBlock, lut); }
static_assert(offsetof(TableBlock, lut) % 256 == 0, "either way the sections behind it stay aligned");
static_assert(sizeof(TableBlock) % 256 == 0, "table block keeps later sections aligned");

// Per-symbol encoder constants (16 bytes, one ds_read_b128), derived by every encoder workgroup from
// the frequencies and cumulative frequencies of the tensor's table.
//   The step is x <- (x / f) * M + (x mod f) + cum = q * (M - f) + x + cum with q = floor(x / f).
//   limit_cum: the state is renormalised before the step when x >= f << 20, so q < 2^20.  f << 20
//   has no bits in its lower half, so the test compares the upper halves only (x >> 16 against the
//   largest that stays, f << 4 less 1) and the lower half of the same dword carries cum (both halves are read
//   through the sub-dword operand selects of the compare and the add, without an instruction to extract them).
//   Nothing is above 0xFFFF: f = 4096 (a tensor of one symbol) and f = 0 never renormalise.
//   mul, shift_inc: with s = floor(log2 f), q is the upper dword of (x + inc) * mul, shifted right by s
//   (division by an invariant: Granlund and Montgomery 1994, Robison 2005).  For x < f << 20 and f < 2^12
//   it is exact with mul = ceil(2^(32+s) / f), inc = 0 as long as (mul * f - 2^(32+s)) * f <= 2^(12+s), and
//   with mul = floor(2^(32+s) / f), inc = 1 as long as (2^(32+s) - mul * f) * f <= 2^(12+s); the two errors
//   add up to f < 2^(s+1), so the smaller one is at most f / 2 and satisfies its condition.  A power of two
//   takes mul = 2^32 - 1, inc = 1.  The multiply-high runs at a quarter of the vector rate, but it takes the
//   place of six instructions that depend on one another (two conversions, a float product, a remainder, its
//   compare and the correction).
struct EncSym {
    uint32_t mul;
    uint32_t limit_cum;  // ((f << 4) - 1) << 16 | cum
    uint32_t shift_inc;  // s | inc << 16
    uint32_t cmpl;       // M - f
};
__host__ __device__ constexpr uint32_t limit_of(uint32_t f) { return ((f << 4) - 1u) << 16; }
__host__ __device__ constexpr bool renormalises(uint32_t x, uint32_t limit_cum) { return (x >> 16) > (limit_cum >> 16); }

// Of no symbol, for turns that a ragged chunk does not have: q = 0, nothing is added, nothing is renormalised, so every state
// stays as it is, up to 2^32 - 1 (compared with >=, the limit sent the states from 0xFFFF0000 on away).  The multiplier is not
// zero: this is no symbol without room.
constexpr EncSym kNoSymbol = {1u, limit_of(0), 0u, 0u};

// ------------------------------------------------------------------------------------------
// Compression works on a batch of up to 8 tensors that share mantissa_bits and block size (the
// weights of a layer): every kernel of the pipeline is launched once for the whole batch, so
// tensors too small to fill the chip overlap with the others.  A single tensor is a batch of one.
// ------------------------------------------------------------------------------------------
constexpr uint32_t kBatchMax = 8;

struct CompressItem {
    const void *src;       // bf16 words, or binary32 words when the batch is of that type
    uint64_t n;
    // A tensor whose encoder slots would exceed the workspace limit goes through the encoder and the
    // compaction in tiles of whole chunks.  A tile is an item of its own whose pointers (source, states,
    // lens, offsets, fields, ...) start at the tile's first chunk and whose n is the tile's elements;
    // table_n is the element count of the whole tensor (the table is the tensor's), words_before the
    // words of the tiles before it (its chunk offsets and its place in the word section start there).
    uint64_t table_n;
    uint64_t words_before;
    TableBlock *tb;
    uint32_t *offsets;
    uint32_t *states;
    uint8_t *lens;
    uint32_t *mid_states;  // entry points (nullptr: the blob holds none)
    uint8_t *mid_lens;
    uint8_t *sm;
    uint8_t *coef;
    uint16_t *low;         // binary32 tensors: the plane of lower halves
    const uint16_t *grad;  // weight step fused into the encoder: the gradient (src is then written too)
    uint16_t *words;       // the blob's word section (the compaction's destination) ...
    uint64_t words_cap;    // ... and the words it has room for
    uint32_t n_chunks;
    uint32_t block;        // 0: no block-wise normalisation
    uint32_t guard;        // exponents this far outside the occupied range keep f = 1 in the table
    uint32_t group_base;   // first encoder group (16 chunks) of this tensor in the workspace arrays
    uint32_t super_base;   // first entry of this tensor in the array of words per 64 encoder groups
    uint32_t hist_end;     // first workgroup after this tensor's in the histogram launch
    uint32_t enc_end;      // ... in the encode launch
    uint32_t compact_end;  // ... in the compaction launch
};

struct CompressBatch {
    CompressItem it[kBatchMax];
    uint32_t count;
    uint32_t seq;  // stamp of this call
    float lr;      // learning rate of the fused weight step
    uint32_t keep_new;  // fused weight step: write the new weight back over the source
    uint32_t tidy;      // compaction launch: also close the offsets and tidy the workspace
    uint32_t keep_counts;  // ... but leave the histogram bins: further tiles of the tensor need them
};

// What the encoder workgroups of a call add up for the compaction and for the host, in the workspace.  (A tensor's words
// are fewer than 2^32 and its encoder workgroups at most 2^16: both fit one atomic, whose result tells who is last.)
// There are two copies, used by alternate calls: while one call's compaction reads its copy, it
// returns the other one (and the histogram bins) to zero for the call that follows.
constexpr unsigned long long kOneDone = 1ull << 40;
struct CallState {
    unsigned long long total[kBatchMax];  // words of tensor i, + kOneDone per workgroup that has added its own
    uint32_t stale[kBatchMax];            // recompression met an exponent without room in tensor i's table
    uint32_t pad[8];
};
constexpr uint32_t kSuperGroups = 64;  // encoder groups whose words are also added up in one entry

// Host-visible results of one compress call (pinned host memory the kernels write directly).
struct HostRecord {
    struct Item {
        // the words of this item alone (the host adds up the tiles of a tensor), flags, and the stamp of the compress call
        // whose results are complete: written last, in one piece
        unsigned long long told;
        uint32_t pad[2];  // (the arrays are 16-byte aligned)
        uint32_t counts[256];
        uint16_t freq[256];
    } item[kBatchMax];
};
constexpr uint32_t kStampMask = (1u << 30) - 1;
__host__ __device__ inline unsigned long long told_of(unsigned long long words, uint32_t stale, uint32_t seq)
{
    const unsigned long long beyond = words >> 32 ? 1u : 0u;  // too long for 32-bit offsets
    return (words & 0xFFFFFFFFull) | (beyond << 32) | (static_cast<unsigned long long>(stale ? 1u : 0u) << 33) |
           (static_cast<unsigned long long>(seq & kStampMask) << 34);
}
__host__ __device__ inline uint32_t told_words(unsigned long long told) { return static_cast<uint32_t>(told); }
__host__ __device__ inline bool told_beyond(unsigned long long told) { return told >> 32 & 1u; }
__host__ __device__ inline bool told_stale(unsigned long long told) { return told >> 33 & 1u; }  // recompression only: an exponent had no room in the blob's table
__host__ __device__ inline uint32_t told_stamp(unsigned long long told) { return static_cast<uint32_t>(told >> 34); }
static_assert(sizeof(HostRecord::Item) % 16 == 0 && offsetof(HostRecord, item) % 16 == 0, "whole-wave 128-bit stores");

}  // namespace nz
