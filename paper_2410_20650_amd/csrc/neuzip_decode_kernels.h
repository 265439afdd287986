// Fused rANS decode + merge kernels of the NeuZip codec for gfx950 (single tensor and batch).
#pragma once

#include <type_traits>

#include "neuzip_format.h"
#include "neuzip_compress_kernels.h"

namespace nz {

// ------------------------------------------------------------------------------------------
// Kernel 6: fused decoder (Alg. 1 "decompression" + "merge"; Sec. 2.2 Eq. (3)).
//
// A workgroup owns blockDim.x / 16 neighbouring chunks (at most 32; half as many of a blob with entry points).  It copies
// the 4096-entry slot table (symbol | f << 8 | (slot - cum) << 20), or makes it from the tensor's table, in LDS, copies the
// chunks' word runs -- one contiguous piece of the blob -- there with 128-bit loads, through registers or straight, and then
// every lane walks one state, or the half of a state before or behind its entry point: 32 (16) turns of 8 symbols; per symbol
// one table read, one multiply-add, one compare, and a lane-private refill.  The 8 decoded exponents are merged with the 8
// sign|mantissa fields and leave as one 128-bit store; the fields of the next turns are requested before a turn is decoded.
// ------------------------------------------------------------------------------------------
template <int KB>
__device__ __forceinline__ uint64_t load_fields(const uint8_t *__restrict__ sm, uint64_t first_elem)
{
    // the (KB+1)*8 field bits of 8 neighbouring elements
    if constexpr (KB == 7) {
        const uint2 v = *reinterpret_cast<const uint2 *>(sm + first_elem);
        return static_cast<uint64_t>(v.x) | (static_cast<uint64_t>(v.y) << 32);
    } else if constexpr (KB == 3) {
        return *reinterpret_cast<const uint32_t *>(sm + first_elem / 2);
    } else if constexpr (KB == 1) {
        return *reinterpret_cast<const uint16_t *>(sm + first_elem / 4);
    } else {
        return sm[first_elem / 8];
    }
}

// Two bf16 words (sign << 15 | exponent << 7 | kept mantissa bits << (7 - KB)) from the field
// bits of a pair of neighbouring elements and the two slot-table entries that decoded them
// (exponent in the low byte of an entry).
template <int KB>
__device__ __forceinline__ uint32_t merge_pair(uint64_t fields, int pair, uint32_t entry_lo, uint32_t entry_hi)
{
    // [0, exponent_hi, 0, exponent_lo]
    const uint32_t expo = __builtin_amdgcn_perm(entry_hi, entry_lo, 0x0c040c00u);
    if constexpr (KB == 7) {
        // lossless: a field is the byte sign << 7 | mantissa.  Spread the two bytes over the two
        // halfwords ([b1, b1, b0, b0]) and keep bit 15 and bits 6..0 of each.
        const uint32_t half = static_cast<uint32_t>(fields >> (32 * (pair >> 1)));
        const uint32_t twice = __builtin_amdgcn_perm(half, half, (pair & 1) ? 0x03030202u : 0x01010000u);
        return (expo << 7) | (twice & 0x807F807Fu);
    } else if constexpr (KB == 3) {
        // byte `pair` of the 32 field bits holds two nibbles s m2 m1 m0 (low nibble = first element).
        // Nibbles into halfwords, then one multiply by 2^4 + 2^12 puts m at bits 6..4 and s at bit 15.
        const uint32_t v = static_cast<uint32_t>(fields);
        const uint32_t even = v & 0x0F0F0F0Fu, odd = (v >> 4) & 0x0F0F0F0Fu;
        const uint32_t nib = __builtin_amdgcn_perm(odd, even, 0x0c000c00u | ((4u + pair) << 16) | pair);
        return (expo << 7) | (__umul24(nib, 0x1010u) & 0x80708070u);
    } else if constexpr (KB == 1) {
        // nibble `pair` of the 16 field bits is s1 m1 s0 m0: m0 -> bit 6, s0 -> 15, m1 -> 22, s1 -> 31
        const uint32_t f2 = (static_cast<uint32_t>(fields) >> (4 * pair)) & 0xFu;
        const uint32_t spread = __umul24(f2 << 16, 0x1010u) + __umul24(f2, 0x4040u);
        return (expo << 7) | (spread & 0x80408040u);
    } else {
        // bits 2*pair and 2*pair + 1 of the 8 field bits are the two signs
        const uint32_t v = static_cast<uint32_t>(fields);
        return (expo << 7) | ((v << (15 - 2 * pair)) & 0x8000u) | ((v << (30 - 2 * pair)) & 0x80000000u);
    }
}

// binary16 words: the decoded symbol is the word's upper byte, the field its lower byte.
__device__ __forceinline__ uint32_t merge_pair_half(uint64_t fields, int pair, uint32_t entry_lo, uint32_t entry_hi)
{
    const uint32_t sym = __builtin_amdgcn_perm(entry_hi, entry_lo, 0x0c040c00u);  // [0, symbol_hi, 0, symbol_lo]
    const uint32_t half = static_cast<uint32_t>(fields >> (32 * (pair >> 1)));
    // [symbol_hi, field_hi, symbol_lo, field_lo]
    return __builtin_amdgcn_perm(sym, half, (pair & 1) ? 0x06030402u : 0x06010400u);
}

// Lossy tensors with one or no mantissa bit: spreading a few field bits over two bf16 words costs more
// vector instructions than the decoding itself, so it is looked up instead.  A small LDS table, filled
// by the workgroup, maps
//   k = 1: a byte of field bits (four elements, s m per element) to the sign and mantissa bits of two
//          dwords of output (256 entries of 8 bytes);
//   k = 0: a nibble of sign bits (four elements) to the sign bits of two dwords (16 entries).
// A turn's 8 elements take two reads; few distinct addresses are in flight at a time for k = 0.
template <int KB>
constexpr uint32_t kSpreadEntries = KB == 1 ? 256u : (KB == 0 ? 16u : 1u);
template <int KB>
constexpr uint32_t kStageBytesOf = kStageBytes - (KB == 1 ? 2048u : (KB == 0 ? 128u : 0u));  // same LDS in all

template <int KB>
__device__ __forceinline__ uint2 spread_entry(uint32_t i)
{
    if constexpr (KB == 1) {
        // nibble s1 m1 s0 m0: m0 -> bit 6, s0 -> 15, m1 -> 22, s1 -> 31
        auto one = [](uint32_t f) { return ((f & 1u) << 6) | ((f & 2u) << 14) | ((f & 4u) << 20) | ((f & 8u) << 28); };
        return make_uint2(one(i & 0xFu), one(i >> 4));
    } else {
        // signs s3 s2 s1 s0: even elements -> bit 15, odd ones -> bit 31
        return make_uint2(((i & 1u) << 15) | ((i & 2u) << 30), ((i & 4u) << 13) | ((i & 8u) << 28));
    }
}

// The four output dwords of a turn (k = 1 or 0) from its field bits, the eight slot-table entries
// that decoded its exponents, and the table above.
template <int KB>
__device__ __forceinline__ uint4 merge_turn_small(uint64_t fields, const uint32_t (&e)[8], const uint2 *__restrict__ spread)
{
    static_assert(KB == 1 || KB == 0, "wider fields are merged arithmetically");
    const uint32_t v = static_cast<uint32_t>(fields);
    const uint2 a = spread[KB == 1 ? (v & 0xFFu) : (v & 0xFu)];
    const uint2 b = spread[KB == 1 ? ((v >> 8) & 0xFFu) : ((v >> 4) & 0xFu)];
    uint4 o;
    o.x = (__builtin_amdgcn_perm(e[1], e[0], 0x0c040c00u) << 7) | a.x;
    o.y = (__builtin_amdgcn_perm(e[3], e[2], 0x0c040c00u) << 7) | a.y;
    o.z = (__builtin_amdgcn_perm(e[5], e[4], 0x0c040c00u) << 7) | b.x;
    o.w = (__builtin_amdgcn_perm(e[7], e[6], 0x0c040c00u) << 7) | b.y;
    return o;
}

struct LdsWords {
    const uint8_t *base;  // LDS copy of the workgroup's runs
    __device__ __forceinline__ uint32_t peek(uint32_t at) const { return *reinterpret_cast<const uint16_t *>(base + at); }
};
struct GlobalWords {
    const uint8_t *base;  // the lane's run inside the blob
    __device__ __forceinline__ uint32_t peek(uint32_t at) const { return *reinterpret_cast<const uint16_t *>(base + at); }
};
struct NoWords {
    __device__ __forceinline__ uint32_t peek(uint32_t) const { return 0; }
};

// One rANS decoding step of a lane's state; returns the slot-table entry (symbol in its low
// byte).  `next` always holds the word at byte position wp of the lane's word source, so a
// refill is a shift-or.
//   EAGER = false: the following word is fetched only where one has been consumed, behind a branch over the wave's mask.
//   EAGER = true: no branch; the refilled state is selected and the word at wp is fetched again whether it moved or not.
// A wave that has its SIMD to itself issues an instruction about every 8 cycles whatever it depends on, and the mask's
// save, branch and restore cost more there than the two selects: 116 cycles a symbol without them, 139 with (the loop alone,
// 1 to 4 waves per CU; at 8 waves 132 and 147).  With four waves per SIMD the vector unit's time counts, and the branch skips
// some of it: 30 M elements walked whole, k = 3, 26.3 us, without the branch 28.7.
template <bool EAGER, class WordSrc>
__device__ __forceinline__ uint32_t rans_get(const uint32_t *__restrict__ lut, uint32_t &x, uint32_t &wp,
                                             uint32_t &next, const WordSrc &src)
{
    const uint32_t e = lut[x & (kM - 1)];
    const uint32_t y = __umul24((e >> 8) & 0xFFFu, x >> kProbBits) + (e >> 20);
    if constexpr (EAGER) {
        const bool refill = y < kRansL;
        x = refill ? (y << 16) | next : y;
        wp = refill ? wp + 2 : wp;
        next = src.peek(wp);
    } else {
        x = y;
        if (x < kRansL) {
            x = (x << 16) | next;
            wp += 2;
            next = src.peek(wp);
        }
    }
    return e;
}

// Walks one state over its part of chunk [base, base + m) and writes the merged bf16 words.
// LONE: the tensor has a single exponent value (f = 4096): the state never moves and there are
// no words.  Returns through x / wp what the well-formedness check needs.
// Field bits of 8 neighbouring elements; with block-wise normalisation (KB < 7, so the fields
// take at most 32 bits) the block's coefficient byte rides in bits 32..39.
template <int KB, bool NORM>
__device__ __forceinline__ uint64_t load_turn(const uint8_t *__restrict__ sm, const uint8_t *__restrict__ coef,
                                              uint32_t block, uint64_t first_elem)  // block: log2 of the block size
{
    uint64_t f = load_fields<KB>(sm, first_elem);
    if constexpr (NORM)
        f |= static_cast<uint64_t>(coef[first_elem >> block]) << 32;  // `block` is log2 of the block size here
    return f;
}

// bf16(stored * c) on the two halves of a merged dword: two multiplies, one packed conversion;
// a NaN keeps its bits and gets the quiet bit, as in normalise_word
__device__ __forceinline__ uint32_t denormalise_pair(uint32_t d, float c)
{
    typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2_t;
    typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2_t;
    const f32x2_t prod = {__fmul_rn(__uint_as_float(d << 16), c), __fmul_rn(__uint_as_float(d & 0xFFFF0000u), c)};
    uint32_t r = __builtin_bit_cast(uint32_t, __builtin_convertvector(prod, bf16x2_t));
    // c lies in [1, 2): a product is a NaN only if the stored word is one; one compare finds either
    if (__builtin_expect(__builtin_isunordered(prod[0], prod[1]), 0)) {
        if (bf16_is_nan(d & 0xFFFFu))
            r = (r & 0xFFFF0000u) | (d & 0xFFFFu) | 0x40u;
        if (bf16_is_nan(d >> 16))
            r = (r & 0x0000FFFFu) | (d & 0xFFFF0000u) | 0x400000u;
    }
    return r;
}

// The four output dwords of a turn from its field bits (load_turn) and the eight slot-table entries that
// decoded its symbols.
template <int KB, bool NORM, bool HALF>
__device__ __forceinline__ uint4 merge_turn(uint64_t fields, const uint32_t (&e)[8], const uint2 *__restrict__ spread)
{
    uint4 o;
    if constexpr (HALF) {
        o.x = merge_pair_half(fields, 0, e[0], e[1]);
        o.y = merge_pair_half(fields, 1, e[2], e[3]);
        o.z = merge_pair_half(fields, 2, e[4], e[5]);
        o.w = merge_pair_half(fields, 3, e[6], e[7]);
    } else if constexpr (KB <= 1) {
        o = merge_turn_small<KB>(fields, e, spread);
    } else {
        o.x = merge_pair<KB>(fields, 0, e[0], e[1]);
        o.y = merge_pair<KB>(fields, 1, e[2], e[3]);
        o.z = merge_pair<KB>(fields, 2, e[4], e[5]);
        o.w = merge_pair<KB>(fields, 3, e[6], e[7]);
    }
    if constexpr (NORM) {
        const float c = coefficient(static_cast<uint32_t>(fields >> 32) & 0x7Fu);
        o.x = denormalise_pair(o.x, c);
        o.y = denormalise_pair(o.y, c);
        o.z = denormalise_pair(o.z, c);
        o.w = denormalise_pair(o.w, c);
    }
    return o;
}

// What a workgroup's beginning has requested of a state's first turns: the fields, and the lower halves of a binary32 tensor that is
// walked from the entry points.  There they are requested for every lane (addresses stay inside the tensor), and waves with a
// ragged chunk use them too; in whole walks for whole chunks only.
constexpr uint32_t kTurnsAhead = 4;
static_assert(kTurnsAhead >= kTurnGroup && kTurnsAhead >= kTurnGroupStream, "at least a group of turns");
struct TurnsAhead {
    uint64_t fields[kTurnsAhead];
    uint4 lows[kTurnsAhead];
};

// Marks a loaded value as used here, at the end of a path beside a hot loop: the compiler lays the two out one
// behind the other, takes the path's loads for outstanding in the loop, and would wait there in every turn for
// the stores of the turn before (28672 x 8192, k = 3, block 512: 158 us instead of 147).
__device__ __forceinline__ void settle(uint64_t v)
{
    asm volatile("" ::"v"(static_cast<uint32_t>(v)), "v"(static_cast<uint32_t>(v >> 32)));
}

// The end of a tensor's ragged last chunk (and of the whole chunks that share its wave): the turns from turn0 on that the walk in
// groups has left, fewer than a group of whole ones and one possibly with fewer than 8 elements of the lane's own; m elements, or
// as many as lie before the lane's entry point.  Fields are read a whole turn at a time and one turn ahead: the sections of the
// blob they come from are padded by 256 bytes, so the last read may pass the tensor's end.  The gradient is
// the caller's, so the elements of an incomplete turn are read one by one there, as they are written.
// (Walked from its beginning a turn at a time, with the stores of a turn waited for in the next, a ragged chunk was the last to
// end: 58.7 M elements less 1000 52.2 us, 46.8 now and without a ragged end, 45 M 45.2 / 41.3, 4 M
// 12.3 / 11.0, binary32 2.9 M 14.0 / 13.5.)
template <int KB, bool LONE, bool NORM, bool UPD, bool HALF, bool EAGER, class WordSrc>
__device__ __forceinline__ void walk_ragged(const uint32_t *__restrict__ lut, const uint2 *__restrict__ spread,
                                            const WordSrc &src, uint32_t lone, uint32_t &x, uint32_t &wp,
                                            const uint8_t *__restrict__ sm, const uint8_t *__restrict__ coef,
                                            uint32_t block, uint16_t *__restrict__ out, uint64_t base, uint32_t m,
                                            uint32_t j, uint32_t turn0, uint64_t fields, const uint16_t *__restrict__ grad,
                                            float lr)
{
    uint32_t next = LONE ? 0u : src.peek(wp);
    uint32_t at = turn0 * kTurn + j * kRun;  // this lane's run of the turn, inside the chunk; `fields` are its
    for (; at < m; at += kTurn) {
        const uint64_t here = base + at;
        uint64_t fields_next = 0;
        if (at + kTurn < m)
            fields_next = load_turn<KB, NORM>(sm, coef, block, here + kTurn);
        const uint32_t valid = m - at < kRun ? m - at : kRun;
        uint4 g = make_uint4(0, 0, 0, 0);
        uint32_t e[8];
        if (valid == kRun) {
            if constexpr (UPD)
                g = *reinterpret_cast<const uint4 *>(grad + here);
#pragma unroll
            for (int t = 0; t < 8; ++t)
                e[t] = LONE ? lone : rans_get<EAGER>(lut, x, wp, next, src);
        } else {
            if constexpr (UPD) {
                uint32_t one[8];
#pragma unroll
                for (uint32_t t = 0; t < 8; ++t)
                    one[t] = t < valid ? grad[here + t] : 0u;
                g = make_uint4(one[0] | (one[1] << 16), one[2] | (one[3] << 16), one[4] | (one[5] << 16),
                               one[6] | (one[7] << 16));
            }
#pragma unroll
            for (uint32_t t = 0; t < 8; ++t) {
                e[t] = 0;
                if (t < valid)
                    e[t] = LONE ? lone : rans_get<EAGER>(lut, x, wp, next, src);
            }
        }
        uint4 o = merge_turn<KB, NORM, HALF>(fields, e, spread);
        if constexpr (UPD) {
            o.x = update_pair(o.x, g.x, lr);
            o.y = update_pair(o.y, g.y, lr);
            o.z = update_pair(o.z, g.z, lr);
            o.w = update_pair(o.w, g.w, lr);
        }
        if (valid == kRun) {
            *reinterpret_cast<uint4 *>(out + here) = o;
        } else {
            const uint32_t d[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
            for (uint32_t t = 0; t < 8; ++t)
                if (t < valid)
                    out[here + t] = static_cast<uint16_t>(d[t >> 1] >> (16 * (t & 1)));
        }
        fields = fields_next;
    }
    settle(fields);
}

// SPLIT: the lane walks one half of its state, from or up to the entry point (see rans_get for the step).
// UPD: the words written are the decoded weights after the update with the gradient `grad` (bf16
// words, same indexing as the output) and the rate lr.  HALF: the tensor is binary16.
template <int KB, bool LONE, bool NORM, bool STREAM, bool UPD, bool HALF, bool SPLIT, bool EAGER, class WordSrc>
__device__ __forceinline__ void walk_state(const uint32_t *__restrict__ lut, const uint2 *__restrict__ spread,
                                           const WordSrc &src, uint32_t lone,
                                           uint32_t &x, uint32_t &wp, const uint8_t *__restrict__ sm,
                                           const uint8_t *__restrict__ coef, uint32_t block,
                                           uint64_t (&fields)[kTurnsAhead],
                                           uint16_t *__restrict__ out,
                                           uint64_t base, uint32_t m, uint32_t j, uint32_t turn0, uint64_t last_run,
                                           const uint16_t *__restrict__ grad = nullptr, float lr = 0.0f)
{
    static_assert(!(UPD || HALF) || (KB == 7 && !NORM), "trained weights and binary16 tensors are lossless only");
    static_assert(!(UPD && HALF), "only bf16 weights are trained");
    // `fields` arrives holding the field bits of the state's first turns (from the entry points; else of whole chunks only)
    constexpr uint32_t kGroup = (STREAM && KB == 7 && !UPD) ? kTurnGroupStream : kTurnGroup;
    constexpr uint32_t turns = SPLIT ? kMidTurn : kTurns;
    // The whole turns, in groups: all of them where all chunks of the wave are whole (WHOLE), else as many groups as this lane has.
    auto groups = [&](auto whole_wave, uint32_t upto) {
        constexpr bool WHOLE = decltype(whole_wave)::value;
        if (!WHOLE && upto == 0)
            return;
        uint32_t next = LONE ? 0u : src.peek(wp);
        const uint64_t from = base + turn0 * kTurn;
        uint4 *out4 = reinterpret_cast<uint4 *>(out + from) + j;
        const uint64_t first = from + j * kRun;
        // the gradients of a turn: the 128 bits the lane's output words come from
        const uint4 *grad4 = UPD ? reinterpret_cast<const uint4 *>(grad + from) + j : nullptr;
        if constexpr (!WHOLE && !SPLIT) {  // (from the entry points they have been requested for all lanes)
#pragma unroll
            for (uint32_t r = 0; r < kGroup; ++r)
                fields[r] = load_turn<KB, NORM>(sm, coef, block, first + r * kTurn);
        }
        uint4 grads[kGroup];
        if constexpr (UPD) {
#pragma unroll
            for (uint32_t r = 0; r < kGroup; ++r)
                grads[r] = grad4[r * kStates];
        }
        // Turns are taken in groups: the field loads of the next group are issued together before
        // the current group is decoded, and the group's 128-bit stores leave back to back, so
        // each state keeps several memory requests in flight and a chunk is written in bursts of
        // kGroup * 256 contiguous bytes.
        for (uint32_t q0 = 0; q0 < upto; q0 += kGroup) {
            uint64_t fields_next[kGroup];
            // the last group re-reads its own fields (stays in bounds)
            const uint32_t qn = q0 + kGroup < upto ? q0 + kGroup : q0;
#pragma unroll
            for (uint32_t r = 0; r < kGroup; ++r)
                fields_next[r] = load_turn<KB, NORM>(sm, coef, block, first + (qn + r) * kTurn);
            uint4 grads_next[kGroup];
            if constexpr (UPD) {
#pragma unroll
                for (uint32_t r = 0; r < kGroup; ++r)
                    grads_next[r] = grad4[(qn + r) * kStates];
            }
            uint4 o[kGroup];
#pragma unroll
            for (uint32_t r = 0; r < kGroup; ++r) {
                uint32_t e[8];
#pragma unroll
                for (int t = 0; t < 8; ++t)
                    e[t] = LONE ? lone : rans_get<EAGER>(lut, x, wp, next, src);
                o[r] = merge_turn<KB, NORM, HALF>(fields[r], e, spread);
                if constexpr (UPD) {
                    o[r].x = update_pair(o[r].x, grads[r].x, lr);
                    o[r].y = update_pair(o[r].y, grads[r].y, lr);
                    o[r].z = update_pair(o[r].z, grads[r].z, lr);
                    o[r].w = update_pair(o[r].w, grads[r].w, lr);
                }
            }
#pragma unroll
            for (uint32_t r = 0; r < kGroup; ++r) {
                uint4 *dst = &out4[(q0 + r) * kStates];
                if constexpr (STREAM) {
                    // a tensor larger than the last-level cache: non-temporal stores
                    __builtin_nontemporal_store(o[r].x, &dst->x);
                    __builtin_nontemporal_store(o[r].y, &dst->y);
                    __builtin_nontemporal_store(o[r].z, &dst->z);
                    __builtin_nontemporal_store(o[r].w, &dst->w);
                } else {
                    *dst = o[r];
                }
                fields[r] = fields_next[r];
                if constexpr (UPD)
                    grads[r] = grads_next[r];
            }
        }
        if constexpr (!WHOLE) {
#pragma unroll
            for (uint32_t r = 0; r < kGroup; ++r)
                settle(fields[r]);
        }
    };
    if (__builtin_expect(__all(m == kChunk), 1)) {
        groups(std::true_type{}, turns);
    } else {
        // (what the groups leave is requested in front of them, where a walk is short; the address stays inside the tensor)
        const uint32_t have = min(m / kTurn, turn0 + turns), done = have > turn0 ? (have - turn0) / kGroup * kGroup : 0u;
        const uint64_t at = min(base + (turn0 + done) * kTurn + j * kRun, last_run);
        uint64_t rest = SPLIT ? load_turn<KB, NORM>(sm, coef, block, at) : 0;
        groups(std::false_type{}, done);
        if constexpr (!SPLIT)
            rest = load_turn<KB, NORM>(sm, coef, block, at);
        walk_ragged<KB, LONE, NORM, UPD, HALF, EAGER>(lut, spread, src, lone, x, wp, sm, coef, block, out, base,
                                                      min(m, (turn0 + turns) * kTurn), j, turn0 + done, rest, grad, lr);
    }
}

// The same walk for a binary32 tensor (lossless only): the decoded bf16 word is the upper half
// of the element and the lower half comes from the raw plane, so a turn reads 16 B of lower
// halves next to its 8 B of fields and writes two 128-bit pieces.
template <bool LONE, bool STREAM, bool SPLIT, bool ALONE, bool EAGER, class WordSrc>
__device__ __forceinline__ void walk_state_wide(const uint32_t *__restrict__ lut, const WordSrc &src, uint32_t lone,
                                                uint32_t &x, uint32_t &wp, const uint8_t *__restrict__ sm,
                                                const uint16_t *__restrict__ low, uint32_t *__restrict__ out,
                                                uint64_t base, uint32_t m, uint32_t j, uint32_t turn0, uint64_t last_run,
                                                const TurnsAhead &ahead)
{
    constexpr uint32_t kGroup = kTurnGroup;
    constexpr uint32_t turns = SPLIT ? kMidTurn : kTurns;
    // Groups of turns whose inputs are held: one, and the next is requested before it is decoded and moves up behind it; or
    // two that are used in rotation, each requested again once it is merged (from the entry points, with a wave or two per
    // SIMD to wait for memory with: 10 M elements 18.5 us with one, 17.6 with two).  In batches of more workgroups than CUs
    // memory has enough to do with one (25 M elements in three tensors 50.7 us, with two 53.8; 28 M in two 51.0 / 54.6).
    constexpr uint32_t kDepth = SPLIT && ALONE ? 2 : 1;
    static_assert(turns % (kGroup * kDepth) == 0, "whole rotations");
    uint32_t next = LONE ? 0u : src.peek(wp);
    // (see walk_state)
    auto groups = [&](auto whole_wave, uint32_t upto) {
        constexpr bool WHOLE = decltype(whole_wave)::value;
        constexpr uint32_t kHeld = WHOLE ? kDepth : 1;
        if (!WHOLE && upto == 0)
            return;
        // where this lane stores: its own pieces 2j and 2j + 1 of a turn's 32, or, after the exchange
        // described below, pieces (j / 8) * 16 + j % 8 and 8 further
        const uint64_t from = base + turn0 * kTurn;
        uint4 *out4 = reinterpret_cast<uint4 *>(out + from) + (STREAM ? (j >> 3) * 16 + (j & 7) : 2 * j);
        const uint32_t lane = threadIdx.x & 63u;
        const uint32_t pull[2] = {((lane & ~7u) + ((lane & 7u) >> 1)) * 4u, ((lane & ~7u) + 4u + ((lane & 7u) >> 1)) * 4u};
        const bool odd = lane & 1u;
        const uint4 *low4 = reinterpret_cast<const uint4 *>(low + from) + j;
        const uint64_t first = from + j * kRun;
        uint64_t fields[kHeld][kGroup];
        uint4 lows[kHeld][kGroup];
        auto request = [&](uint64_t (&f)[kGroup], uint4 (&l)[kGroup], uint32_t q) {
#pragma unroll
            for (uint32_t r = 0; r < kGroup; ++r) {
                f[r] = load_fields<7>(sm, first + (q + r) * kTurn);
                l[r] = low4[(q + r) * kStates];
            }
        };
        static_assert(kHeld == 1 || kHeld * kGroup == kTurnsAhead, "requested by the workgroup's beginning");
#pragma unroll
        for (uint32_t d = 0; d < kHeld; ++d) {
            if constexpr (kHeld == 1)
                request(fields[d], lows[d], 0);
#pragma unroll
            for (uint32_t r = 0; kHeld > 1 && r < kGroup; ++r) {  // (requested for all lanes)
                fields[d][r] = ahead.fields[d * kGroup + r];
                lows[d][r] = ahead.lows[d * kGroup + r];
            }
        }
        for (uint32_t q0 = 0; q0 < upto; q0 += kGroup * kHeld) {
#pragma unroll
            for (uint32_t d = 0; d < kHeld; ++d) {
                const uint32_t q = q0 + d * kGroup;
                uint64_t (&f)[kGroup] = fields[d];
                uint4 (&l)[kGroup] = lows[d];
                uint64_t fields_next[kGroup];
                uint4 lows_next[kGroup];
                // (behind the last group: its own again, in bounds and not used)
                const uint32_t qn = q + kHeld * kGroup < upto ? q + kHeld * kGroup : q;
                if constexpr (kHeld == 1)
                    request(fields_next, lows_next, qn);
                uint4 o[2 * kGroup];
#pragma unroll
                for (uint32_t r = 0; r < kGroup; ++r) {
                    uint32_t e[8];
#pragma unroll
                    for (int t = 0; t < 8; ++t)
                        e[t] = LONE ? lone : rans_get<EAGER>(lut, x, wp, next, src);
                    const uint32_t h[4] = {merge_pair<7>(f[r], 0, e[0], e[1]), merge_pair<7>(f[r], 1, e[2], e[3]),
                                           merge_pair<7>(f[r], 2, e[4], e[5]), merge_pair<7>(f[r], 3, e[6], e[7])};
                    const uint32_t lo[4] = {l[r].x, l[r].y, l[r].z, l[r].w};
                    // element = upper half << 16 | lower half: this lane's 8 elements as 16-byte pieces 2j, 2j + 1
                    // of the turn's 32
                    uint32_t mine[2][4];
#pragma unroll
                    for (int d = 0; d < 4; ++d) {
                        mine[d >> 1][2 * (d & 1)] = __builtin_amdgcn_perm(h[d], lo[d], 0x05040100u);
                        mine[d >> 1][2 * (d & 1) + 1] = __builtin_amdgcn_perm(h[d], lo[d], 0x07060302u);
                    }
                    // A 128-bit store of piece 2j by every lane leaves every other 16 bytes of a cache line
                    // to a second instruction.  In the cache that is harmless, but once the tensor streams
                    // to HBM such half-written lines cost a third of the store rate.  There the 8 lanes of
                    // an octet trade pieces: store `half` of lane t writes piece 8 * half + t of the
                    // octet's 16, which lane 4 * half + t / 2 holds (its first piece for even t), and each
                    // store instruction covers whole 128-byte lines.  (The 16 lane exchanges per turn cost
                    // 20 % of the rate of a cache-resident tensor, which therefore keeps the plain stores.)
#pragma unroll
                    for (int half = 0; half < 2; ++half) {
                        uint32_t got[4];
#pragma unroll
                        for (int d = 0; d < 4; ++d) {
                            if constexpr (STREAM) {
                                const uint32_t first = __builtin_amdgcn_ds_bpermute(static_cast<int>(pull[half]),
                                                                                    static_cast<int>(mine[0][d]));
                                const uint32_t second = __builtin_amdgcn_ds_bpermute(static_cast<int>(pull[half]),
                                                                                     static_cast<int>(mine[1][d]));
                                got[d] = odd ? second : first;
                            } else {
                                got[d] = mine[half][d];
                            }
                        }
                        o[2 * r + half] = make_uint4(got[0], got[1], got[2], got[3]);
                    }
                }
                if constexpr (kHeld > 1)
                    request(f, l, qn);
#pragma unroll
                for (uint32_t r = 0; r < kGroup; ++r) {
#pragma unroll
                    for (uint32_t half = 0; half < 2; ++half) {
                        uint4 *dst = &out4[(q + r) * kStates * 2 + half * (STREAM ? 8 : 1)];
                        const uint4 v = o[2 * r + half];
                        if constexpr (STREAM) {
                            __builtin_nontemporal_store(v.x, &dst->x);
                            __builtin_nontemporal_store(v.y, &dst->y);
                            __builtin_nontemporal_store(v.z, &dst->z);
                            __builtin_nontemporal_store(v.w, &dst->w);
                        } else {
                            *dst = v;
                        }
                    }
                    if constexpr (kHeld == 1) {
                        f[r] = fields_next[r];
                        l[r] = lows_next[r];
                    }
                }
            }
        }
        if constexpr (!WHOLE) {
#pragma unroll
            for (uint32_t d = 0; d < kHeld; ++d)
#pragma unroll
                for (uint32_t r = 0; r < kGroup; ++r) {
                    settle(fields[d][r]);
                    settle(lows[d][r].x | (static_cast<uint64_t>(lows[d][r].w) << 32));
                }
        }
    };
    if (__builtin_expect(__all(m == kChunk), 1)) {
        groups(std::true_type{}, turns);
    } else {
        // what the groups leave (see walk_ragged), requested in front of them.  In groups only where the words are in LDS: with a second
        // copy of the group loop for the others, which hardly ever come here, the kernel is 25.7 KB of code instead of 22.5, and all waves of
        // a launch took longer (10 M elements 16.17 us, 16.07 now, 1 M 11.81 / 11.73, mean of 42 placements).
        constexpr bool kGroups = std::is_same<WordSrc, LdsWords>::value;
        const uint32_t have = min(m / kTurn, turn0 + turns);
        const uint32_t done = kGroups && have > turn0 ? (have - turn0) / kGroup * kGroup : 0u;
        uint32_t at = (turn0 + done) * kTurn + j * kRun;
        const uint64_t from = min(base + at, last_run);
        uint64_t fields = load_fields<7>(sm, from);
        uint4 lows = *reinterpret_cast<const uint4 *>(low + from);
        if constexpr (kGroups)
            groups(std::false_type{}, done);
        m = min(m, (turn0 + turns) * kTurn);
        for (; at < m; at += kTurn) {
            const uint64_t here = base + at;
            uint64_t fields_next = 0;
            uint4 lows_next = make_uint4(0, 0, 0, 0);
            if (at + kTurn < m) {
                fields_next = load_fields<7>(sm, here + kTurn);
                lows_next = *reinterpret_cast<const uint4 *>(low + here + kTurn);
            }
            const uint32_t valid = m - at < kRun ? m - at : kRun;
            uint32_t e[8];
            if (valid == kRun) {
#pragma unroll
                for (int t = 0; t < 8; ++t)
                    e[t] = LONE ? lone : rans_get<EAGER>(lut, x, wp, next, src);
            } else {
#pragma unroll
                for (uint32_t t = 0; t < 8; ++t) {
                    e[t] = 0;
                    if (t < valid)
                        e[t] = LONE ? lone : rans_get<EAGER>(lut, x, wp, next, src);
                }
            }
            const uint32_t h[4] = {merge_pair<7>(fields, 0, e[0], e[1]), merge_pair<7>(fields, 1, e[2], e[3]),
                                   merge_pair<7>(fields, 2, e[4], e[5]), merge_pair<7>(fields, 3, e[6], e[7])};
            const uint32_t l[4] = {lows.x, lows.y, lows.z, lows.w};
            uint32_t v[8];
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                v[2 * d] = __builtin_amdgcn_perm(h[d], l[d], 0x05040100u);
                v[2 * d + 1] = __builtin_amdgcn_perm(h[d], l[d], 0x07060302u);
            }
            if (valid == kRun) {
                reinterpret_cast<uint4 *>(out + here)[0] = make_uint4(v[0], v[1], v[2], v[3]);
                reinterpret_cast<uint4 *>(out + here)[1] = make_uint4(v[4], v[5], v[6], v[7]);
            } else {
#pragma unroll
                for (uint32_t t = 0; t < 8; ++t)
                    if (t < valid)
                        out[here + t] = v[t];
            }
            fields = fields_next;
            lows = lows_next;
        }
        settle(fields);
        settle(lows.x | (static_cast<uint64_t>(lows.w) << 32));
    }
}

// What the decoder needs to know about one tensor (all device pointers).
struct DecodeArgs {
    const TableBlock *tb;
    const uint32_t *offsets;
    const uint32_t *states;
    const uint8_t *lens;
    const uint32_t *mid_states;  // entry points (nullptr: the blob has none)
    const uint8_t *mid_lens;
    const uint16_t *words;
    const uint8_t *sm;
    const uint8_t *coef;  // block coefficients (block-wise normalised blobs only)
    const uint16_t *low;  // lower halves (binary32 blobs only)
    const uint16_t *grad; // gradient of the weight, bf16 words (update variant only)
    float lr;             // learning rate (update variant only)
    void *out;            // bf16 words, or binary32 words for a binary32 blob
    uint32_t *status;
    uint64_t n;
    uint32_t n_chunks;
    uint32_t block;       // 0: no block-wise normalisation
    uint32_t stream_out;  // non-zero: the output does not fit the last-level cache, store non-temporally
    uint32_t wg_end;      // batches: first workgroup index after this tensor's
    uint32_t fit;         // (for the host: chunks whose words fit a workgroup's LDS window)
    uint32_t in_step;     // (for the host: the states' runs are of one length, see runs_in_step)
};

// MODE: what a decoder writes -- the decoded bf16 words (kPlain), binary32 words joined with their
// lower halves (kWide), the decoded weights after the update of the backward loop (kUpdate), or
// binary16 words (kHalf).
enum DecodeMode { kPlain = 0, kWide = 1, kUpdate = 2, kHalf = 3 };

// The walk of the mode.
template <int KB, bool LONE, bool NORM, bool STREAM, int MODE, bool SPLIT, bool ALONE, class WordSrc>
__device__ __forceinline__ void walk_mode(const uint32_t *__restrict__ lut, const uint2 *__restrict__ spread,
                                          const WordSrc &src, uint32_t lone, uint32_t &x, uint32_t &wp, const DecodeArgs &a,
                                          uint32_t block, TurnsAhead &ahead, uint64_t base, uint32_t m, uint32_t j,
                                          uint32_t turn0)
{
    // (a word read from memory is fetched only when it is needed)
    constexpr bool EAGER = ALONE && !std::is_same<WordSrc, GlobalWords>::value;
    const uint64_t last_run = (a.n - 1) & ~static_cast<uint64_t>(kRun - 1);  // where the tensor's last 8 elements, or fewer, begin
    if constexpr (MODE == kWide)
        walk_state_wide<LONE, STREAM, SPLIT, ALONE, EAGER>(lut, src, lone, x, wp, a.sm, a.low, static_cast<uint32_t *>(a.out), base, m, j,
                                             turn0, last_run, ahead);
    else
        walk_state<KB, LONE, NORM, STREAM, MODE == kUpdate, MODE == kHalf, SPLIT, EAGER>(
            lut, spread, src, lone, x, wp, a.sm, a.coef, block, ahead.fields, static_cast<uint16_t *>(a.out), base, m, j, turn0, last_run,
            a.grad, a.lr);
}

// 16 bytes per lane from memory straight into LDS: lane l's piece goes to `to` (the same for the wave) + 16 l.
__device__ __forceinline__ void copy_to_lds(const uint4 *from, uint8_t *to)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(from),
                                     (__attribute__((address_space(3))) void *)(to), 16, 0, 0);
}

// A barrier for what the workgroup's waves have written to LDS themselves, which does not wait for direct copies.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// The slot table from the occupied symbols (TableBlock::steps, in LDS), by the whole workgroup; begins: the steps that pieces
// threadIdx.x and threadIdx.x + blockDim.x (of eight neighbouring slots) begin in.  First every piece is written as if the
// step it begins in filled it, then every step that starts inside a piece writes its slots of that piece over that: some 60
// instructions per thread of 256 and a barrier, while a search slot by slot (make_piece) takes 200 for each of its two pieces,
// and these tables are made by waves that wait for nothing else.  (The caller's barrier is still to come.)
__device__ __forceinline__ void make_table(const uint32_t *__restrict__ steps, const uint32_t (&begins)[2],
                                           const TableBlock *__restrict__ tb, uint32_t *__restrict__ lut)
{
    const uint32_t tid = threadIdx.x, threads = blockDim.x;
    auto entry = [](uint32_t here, uint32_t there, uint32_t slot) {
        return (here & 0xFFu) | ((((there >> 8) - (here >> 8)) & 0xFFFu) << 8) | ((slot - (here >> 8)) << 20);
    };
    auto fill = [&](uint32_t piece, uint32_t r) {
        const uint32_t e = entry(steps[r], steps[r + 1], piece * 8);
        uint4 *at = reinterpret_cast<uint4 *>(lut) + 2 * piece;
        at[0] = make_uint4(e, e + (1u << 20), e + (2u << 20), e + (3u << 20));
        at[1] = make_uint4(e + (4u << 20), e + (5u << 20), e + (6u << 20), e + (7u << 20));
    };
#pragma unroll
    for (uint32_t r = 0; r < 2; ++r)
        if (tid + r * threads < kM / 8)
            fill(tid + r * threads, begins[r]);
    for (uint32_t piece = tid + 2 * threads; piece < kM / 8; piece += threads)  // (small workgroups)
        fill(piece, tb->step_of[piece]);
    lds_barrier();
    for (uint32_t i = tid; i + 1 < kSteps; i += threads) {
        const uint32_t here = steps[i], there = steps[i + 1];
        const uint32_t from = here >> 8, piece_end = (from + 7) & ~7u;  // (nothing to write where a piece begins with it)
        const uint32_t upto = (there >> 8) < piece_end ? there >> 8 : piece_end;
        for (uint32_t slot = from; slot < upto; ++slot)
            lut[slot] = entry(here, there, slot);
    }
}

// `pieces` such pieces by the workgroup.  The copies are under way when this returns: wait_for_memory_acks, then a barrier.
__device__ __forceinline__ void copy_run_to_lds(const uint4 *from, uint8_t *to, uint32_t pieces)
{
    const uint32_t lane = threadIdx.x & 63u;
    for (uint32_t i = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x & ~63u))); i < pieces;
         i += blockDim.x)
        if (i + lane < pieces)
            copy_to_lds(from + i + lane, to + i * 16);
}

// How a workgroup comes by the tensor's slot table and how many lanes walk a state, settled at compile time: with a
// run-time choice of one or two lanes the other blobs lost 2-5 %, and with a run-time choice of the table (a second
// barrier, 14 registers and 1 KB of LDS that only a made table needs) a binary16 tensor of 58.7 M elements took 61.8 us
// (60.2 now), the k = 3 weights of a Llama-3-8B layer 136.0 (135.0), 20 M elements 24.5 (24.1).
enum DecodeForm {
    kReadTable,  // one lane per state; the slot table is copied from the blob
    kMakeTable,  // one lane per state; the blob is too small to hold the table (its entry points are not used)
    kEntries,    // two lanes per state, from the entry points; the slot table is made
    kReadDirect, // like kReadTable, cached; the words are copied straight into LDS
    kEntriesAlone, // like kEntries, where a SIMD has two waves or so: no branch in the step
};

template <int KB, bool NORM, int MODE, int FORM>
__device__ __forceinline__ void decode_workgroup(const DecodeArgs &a, uint32_t wg, uint32_t *__restrict__ lut,
                                                 uint32_t *__restrict__ steps, uint8_t *__restrict__ stage,
                                                 uint2 *__restrict__ spread)
{
    constexpr bool WIDE = MODE == kWide;
    constexpr bool make_lut = FORM == kMakeTable;
    static_assert(MODE == kPlain || (KB == 7 && !NORM), "binary32 blobs and trained weights are lossless only");
    const uint32_t block = 31u - static_cast<uint32_t>(__clz(static_cast<int>(a.block | 1u)));  // log2 (a power of two)
    const uint16_t *__restrict__ words = a.words;
    const uint8_t *__restrict__ sm = a.sm;
    const uint8_t *__restrict__ coef = a.coef;
    // (blobs of at most 2^24 elements are never beyond the cache, and in a batch that is they are walked whole)
    const bool stream_out = FORM == kMakeTable || (FORM == kReadTable && a.stream_out != 0);
    static_assert(FORM != kEntries && FORM != kEntriesAlone, "see decode_from_entries");
    const uint32_t n_chunks = a.n_chunks;
    const uint32_t tid = threadIdx.x;
    const uint32_t threads = blockDim.x;            // a multiple of 64, at most kDecThreads
    const uint32_t chunks_per_wg = threads / kStates;
    const uint32_t c0 = wg * chunks_per_wg;
    const uint32_t c1 = c0 + chunks_per_wg < n_chunks ? c0 + chunks_per_wg : n_chunks;
    const uint32_t c = c0 + tid / kStates;
    const uint32_t j = tid % kStates;
    const bool live = c < n_chunks;
    const uint32_t id = c * kStates + j;
    const uint64_t base = static_cast<uint64_t>(c) * kChunk;
    const uint32_t m = !live ? 0u : ((a.n - base) < kChunk ? static_cast<uint32_t>(a.n - base) : kChunk);

    // ---- every load that depends on nothing is issued first, so their latencies overlap
    const uint32_t off0 = a.offsets[c0];
    const uint32_t off1 = a.offsets[c1];
    const uint32_t off_c = live ? a.offsets[c] : 0u;
    uint32_t x = live ? a.states[id] : kRansL;
    const uint32_t len = live ? a.lens[id] : 0u;
    const uint32_t lone = a.tb->lone;
    // the tensor's table: its steps (blobs with entry points) or the slot table itself
    const uint4 *table_g = reinterpret_cast<const uint4 *>(make_lut ? a.tb->steps : a.tb->lut);
    constexpr uint32_t table_pieces = make_lut ? kSteps / 4 : kM / 4;  // of 16 bytes
    uint4 *table_to = reinterpret_cast<uint4 *>(make_lut ? steps : lut);
    uint4 table_piece[2];  // the slot table has 1024 pieces: 2 per thread at 512 threads
#pragma unroll
    for (uint32_t r = 0; r < 2; ++r) {
        const uint32_t i = tid + r * threads;
        table_piece[r] = i < table_pieces ? table_g[i] : make_uint4(0, 0, 0, 0);
    }
    uint32_t first_step = 0;  // of this thread's first piece of the slot table
    if constexpr (make_lut)
        first_step = a.tb->step_of[tid];
    TurnsAhead ahead;
#pragma unroll
    for (uint32_t r = 0; r < kTurnsAhead; ++r)
        ahead.fields[r] = !WIDE && m == kChunk && r < (KB == 7 ? kTurnGroupStream : kTurnGroup)  // (the largest group of the width)
                              ? load_turn<KB, NORM>(sm, coef, block, base + r * kTurn + j * kRun)
                              : 0;
    // ---- the word runs of chunks [c0, c1), one contiguous piece of the blob, into LDS
    const uint64_t byte0 = static_cast<uint64_t>(off0) * 2;
    const uint64_t byte1 = static_cast<uint64_t>(off1) * 2;
    const uint64_t aligned0 = byte0 & ~static_cast<uint64_t>(15);
    const uint64_t stage_len = byte1 - aligned0;
    const bool staged = stage_len + 16 <= kStageBytesOf<KB>;  // room for the one-word look-ahead
    const uint4 *from = reinterpret_cast<const uint4 *>(reinterpret_cast<const uint8_t *>(words) + aligned0);
    uint4 *to = reinterpret_cast<uint4 *>(stage);
    auto table_to_lds = [&]() {
#pragma unroll
        for (uint32_t r = 0; r < 2; ++r) {
            const uint32_t i = tid + r * threads;
            if (i < table_pieces)
                table_to[i] = table_piece[r];
        }
        for (uint32_t i = tid + 2 * threads; i < table_pieces; i += threads)  // (small workgroups)
            table_to[i] = table_g[i];
        if constexpr (KB <= 1) {
            for (uint32_t i = tid; i < kSpreadEntries<KB>; i += threads)
                spread[i] = spread_entry<KB>(i);
        }
    };
    if constexpr (FORM == kReadDirect) {
        if (staged)
            copy_run_to_lds(from, stage, static_cast<uint32_t>(stage_len + 15) / 16);
        table_to_lds();
        wait_for_memory_acks();
    } else if constexpr (!make_lut) {
        if (staged) {
            for (uint32_t i = tid; static_cast<uint64_t>(i) * 16 < stage_len; i += threads)
                to[i] = from[i];
        }
        table_to_lds();
    } else {
        // the first three per thread are requested together and stay in registers while the table is made (six, all
        // of a usual workgroup's, were 0.5 % slower)
        constexpr uint32_t kFirst = 3;
        uint4 first[kFirst];
#pragma unroll
        for (uint32_t r = 0; r < kFirst; ++r) {
            const uint32_t i = tid + r * threads;
            first[r] = staged && static_cast<uint64_t>(i) * 16 < stage_len ? from[i] : make_uint4(0, 0, 0, 0);
        }
        table_to_lds();
        __syncthreads();
        if (lone >= 256) {
            make_piece(steps, first_step, tid, lut);
            for (uint32_t piece = tid + threads; piece < kM / 8; piece += threads)  // (small workgroups)
                make_piece(steps, a.tb->step_of[piece], piece, lut);
        }
        if (staged) {
#pragma unroll
            for (uint32_t r = 0; r < kFirst; ++r) {
                const uint32_t i = tid + r * threads;
                if (static_cast<uint64_t>(i) * 16 < stage_len)
                    to[i] = first[r];
            }
            for (uint32_t i = tid + kFirst * threads; static_cast<uint64_t>(i) * 16 < stage_len; i += threads)
                to[i] = from[i];
        }
    }
    __syncthreads();

    // ---- one lane, one state
    if (!live)
        return;
    // start of this state's run: chunk offset + lengths of the states before it (16-lane prefix)
    uint32_t before = len;
#pragma unroll
    for (uint32_t d = 1; d < kStates; d <<= 1) {
        const uint32_t o = __shfl_up(before, d, kStates);
        if (j >= d)
            before += o;
    }
    before -= len;
    const uint64_t run_byte = (static_cast<uint64_t>(off_c) + before) * 2;

    uint32_t wp = 0, wp_begin = 0;
    // (the streaming and the cached store variants are separate instantiations: merged into one
    // loop the compiler drops the non-temporal hint)
    auto walk = [&](auto alone, const auto &src, uint32_t only) {
        constexpr bool LONE = decltype(alone)::value;
        if (stream_out)
            walk_mode<KB, LONE, NORM, true, MODE, false, false>(lut, spread, src, only, x, wp, a, block, ahead, base, m, j, 0u);
        else
            walk_mode<KB, LONE, NORM, false, MODE, false, false>(lut, spread, src, only, x, wp, a, block, ahead, base, m, j, 0u);
    };
    if (lone < 256) {
        walk(std::true_type{}, NoWords{}, lone);
    } else if (staged) {
        wp = wp_begin = static_cast<uint32_t>(run_byte - aligned0);
        walk(std::false_type{}, LdsWords{stage}, 0u);
    } else {
        // the runs of this workgroup's chunks did not fit the LDS window (more than ~4 bits per
        // symbol): read the words straight from the blob
        walk(std::false_type{}, GlobalWords{reinterpret_cast<const uint8_t *>(words) + run_byte}, 0u);
    }
    // a well-formed run is consumed exactly and leaves the state where the encoder started
    if (x != kRansL || wp - wp_begin != 2 * len)
        atomicOr(a.status, 1u);
}

// The same from the entry points: two lanes walk the halves of a state.  A launch of such blobs has a wave or two per SIMD,
// so its time is the workgroup's beginning -- a chain of memory latencies: arguments, tables and offsets, words -- and the
// walk's instructions, one after the other.  So nothing in the beginning is behind a branch (lanes without a chunk read the
// last one's: a masked load made the wave wait for the loads before it), the words go to LDS without passing through
// registers while the slot table is made, and the start of a lane's run is worked out meanwhile.  With the steps of the walk
// without a branch (see rans_get) and the table made by make_table: 4 M elements 13.5 -> 10.7 us, of which the beginning
// 3.9 -> 2.7 and the walk 9.5 -> 7.7, 0.05 M 11.8 -> 9.5, 16.8 M 15.8 -> 14.0, 10 M binary32 elements 20.3 -> 16.4; words
// through registers 11.8 (4 M), 15.5 (16.8 M).
// ALONE: the step without a branch.  A single tensor's launch has two waves per SIMD on average whatever its workgroups' size
// (4096 chunks are 2048 waves), also where they are more than the CUs: weights that have left their kept table, 8 chunks of
// 12-bit symbols to a workgroup, 263 workgroups 14.1 us, with the branch 15.1, 512 16.8 / 17.2; for batches see
// launch_batch_kernel, for tensors that keep the branch all the same runs_in_step.
template <int KB, bool NORM, int MODE, bool ALONE>
__device__ __forceinline__ void decode_from_entries(const DecodeArgs &a, uint32_t wg, uint32_t *__restrict__ lut,
                                                    uint32_t *__restrict__ steps, uint8_t *__restrict__ stage,
                                                    uint2 *__restrict__ spread)
{
    static_assert(MODE == kPlain || (KB == 7 && !NORM), "binary32 blobs and trained weights are lossless only");
    static_assert(kTurns == 2 * kMidTurn, "halves");
    const uint32_t block = 31u - static_cast<uint32_t>(__clz(static_cast<int>(a.block | 1u)));  // log2 (a power of two)
    const uint32_t n_chunks = a.n_chunks, tid = threadIdx.x, threads = blockDim.x;
    const uint32_t chunks_per_wg = threads / (2 * kStates);
    const uint32_t c0 = wg * chunks_per_wg;
    const uint32_t c1 = c0 + chunks_per_wg < n_chunks ? c0 + chunks_per_wg : n_chunks;
    const uint32_t c = c0 + tid / (2 * kStates);
    const uint32_t j = tid % kStates;
    const uint32_t part = (tid / kStates) & 1u;  // before (0) or behind (1) the entry point
    const uint32_t turn0 = part * kMidTurn;
    const bool live = c < n_chunks;
    const uint64_t base = static_cast<uint64_t>(c) * kChunk;
    const uint32_t m = !live ? 0u : ((a.n - base) < kChunk ? static_cast<uint32_t>(a.n - base) : kChunk);

    // ---- every load that depends on nothing
    const uint32_t off0 = a.offsets[c0];
    const uint32_t off1 = a.offsets[c1];
    const uint32_t c_in = live ? c : n_chunks - 1;
    const uint32_t id = c_in * kStates + j;
    const uint32_t off_c = a.offsets[c_in];
    const uint32_t first_x = a.states[id], mid_x = a.mid_states[id];
    const uint32_t len = a.lens[id], mid_len = a.mid_lens[id];
    const uint32_t lone = a.tb->lone;
    const uint4 *steps_g = reinterpret_cast<const uint4 *>(a.tb->steps);
    constexpr uint32_t kStepPieces = kSteps / 4;  // of 16 bytes
    const uint4 step_piece = steps_g[tid < kStepPieces ? tid : kStepPieces - 1];
    // the steps that this thread's first two pieces of the slot table begin in (512 pieces: all, from 256 threads on)
    uint32_t begins[2];
#pragma unroll
    for (uint32_t r = 0; r < 2; ++r)
        begins[r] = a.tb->step_of[min(tid + r * threads, kM / 8 - 1)];
    // the first turns' inputs (addresses stay inside the tensor; a lane without the turn makes no use of what it gets)
    TurnsAhead ahead = {};
    const uint32_t last_run = static_cast<uint32_t>(a.n - 1) & ~(kRun - 1);  // (such tensors have at most 2^24 elements)
    auto request_ahead = [&]() {
#pragma unroll
        for (uint32_t r = 0; r < kTurnsAhead; ++r) {
            const uint32_t at = min(c_in * kChunk + (turn0 + r) * kTurn + j * kRun, last_run);
            if (MODE == kWide || r < kTurnGroup)
                ahead.fields[r] = load_turn<KB, NORM>(a.sm, a.coef, block, at);
            if constexpr (MODE == kWide)
                ahead.lows[r] = *reinterpret_cast<const uint4 *>(a.low + at);
        }
    };
    __builtin_amdgcn_sched_barrier(0);  // (behind what the table is made of, which is waited for first)
    if constexpr (MODE != kWide)
        request_ahead();
    __builtin_amdgcn_sched_barrier(0);
    // ---- the steps, then (as soon as the offsets are there) the word runs of chunks [c0, c1), one contiguous piece of the
    // blob, into LDS
    if (tid < kStepPieces)
        reinterpret_cast<uint4 *>(steps)[tid] = step_piece;
    for (uint32_t i = tid + threads; i < kStepPieces; i += threads)  // (workgroups of one wave)
        reinterpret_cast<uint4 *>(steps)[i] = steps_g[i];
    const uint64_t byte0 = static_cast<uint64_t>(off0) * 2, byte1 = static_cast<uint64_t>(off1) * 2;
    const uint64_t aligned0 = byte0 & ~static_cast<uint64_t>(15);
    const uint64_t stage_len = byte1 - aligned0;
    const bool staged = stage_len + 16 <= kStageBytesOf<KB>;  // room for the one-word look-ahead
    asm volatile("" : "+v"(begins[0]), "+v"(begins[1]));  // (taken here, and not waited for behind the words)
    if (staged)
        copy_run_to_lds(reinterpret_cast<const uint4 *>(reinterpret_cast<const uint8_t *>(a.words) + aligned0), stage,
                        static_cast<uint32_t>(stage_len + 15) / 16);
    if constexpr (KB <= 1) {
        for (uint32_t i = tid; i < kSpreadEntries<KB>; i += threads)
            spread[i] = spread_entry<KB>(i);
    }
    // where this lane begins and ends: the run starts behind those of the states before it in the chunk (a row of 16 lanes)
    const uint32_t before = row_scan_u32(len) - len + (part ? mid_len : 0u);
    const uint64_t run_byte = (static_cast<uint64_t>(off_c) + before) * 2;
    uint32_t x = part ? mid_x : first_x;
    // a well-formed run is consumed exactly and leaves the state where the encoder started; the half before the
    // entry point ends there
    const uint32_t x_end = part ? kRansL : mid_x;
    const uint32_t words_here = part ? len - mid_len : mid_len;
    lds_barrier();
    if (lone >= 256)
        make_table(steps, begins, a.tb, lut);
    wait_for_memory_acks();  // the words
    __syncthreads();
    if (!live)
        return;
    if constexpr (MODE == kWide && ALONE)  // (four times the bytes, which in front of the words are in their way: 10 M elements 18.7 / 18.1 us)
        request_ahead();
    uint32_t wp = 0, wp_begin = 0;
    if (lone < 256) {
        walk_mode<KB, true, NORM, false, MODE, true, ALONE>(lut, spread, NoWords{}, lone, x, wp, a, block, ahead, base, m, j, turn0);
    } else if (staged) {
        wp = wp_begin = static_cast<uint32_t>(run_byte - aligned0);
        walk_mode<KB, false, NORM, false, MODE, true, ALONE>(lut, spread, LdsWords{stage}, 0u, x, wp, a, block, ahead, base, m, j, turn0);
    } else {
        const GlobalWords direct{reinterpret_cast<const uint8_t *>(a.words) + run_byte};
        walk_mode<KB, false, NORM, false, MODE, true, ALONE>(lut, spread, direct, 0u, x, wp, a, block, ahead, base, m, j, turn0);
    }
    if (x != x_end || wp - wp_begin != 2 * words_here)
        atomicOr(a.status, 1u);
}

// The LDS of a workgroup.  The words come first: a direct copy's LDS address has 16 bits.
template <int KB, bool MADE>
struct DecodeLds {
    uint8_t stage[kStageBytesOf<KB>];
    uint32_t lut[kM];
    uint2 spread[kSpreadEntries<KB>];
    uint32_t steps[MADE ? kSteps : 2];
    static_assert(kStageBytesOf<KB> <= 65536 && kStageBytesOf<KB> % 16 == 0, "within reach, and the table behind it aligned");
};

template <int KB, bool NORM, int MODE, bool SPLIT>
__global__ __launch_bounds__(kDecThreads) void decode_kernel(const DecodeArgs a)
{
    __shared__ __align__(16) DecodeLds<KB, SPLIT> lds;
    if constexpr (SPLIT)
        decode_from_entries<KB, NORM, MODE, true>(a, blockIdx.x, lds.lut, lds.steps, lds.stage, lds.spread);
    else
        decode_workgroup<KB, NORM, MODE, kReadTable>(a, blockIdx.x, lds.lut, lds.steps, lds.stage, lds.spread);
}

// The launch whose workgroups all run at once, two on every CU at most (see copies_directly).
template <int KB, bool NORM>
__global__ __launch_bounds__(kDecThreads) void decode_direct_kernel(const DecodeArgs a)
{
    __shared__ __align__(16) DecodeLds<KB, false> lds;
    decode_workgroup<KB, NORM, kPlain, kReadDirect>(a, blockIdx.x, lds.lut, lds.steps, lds.stage, lds.spread);
}

// Several tensors in one launch (a layer's weights): workgroups [t[i-1].wg_end, t[i].wg_end)
// belong to tensor i.  Small tensors, which alone cannot fill the chip, overlap with the others.
struct BatchArgs {
    DecodeArgs t[kBatchMax];
    uint32_t count;
    uint32_t threads;  // (for the host: of a workgroup)
};

// FORM: how the blobs of the batch that have entry points (kEntries, kEntriesAlone) or no slot table (kMakeTable) are walked; the
// others read theirs.
template <int KB, bool NORM, int MODE, int FORM>
__global__ __launch_bounds__(kDecThreads) void decode_batch_kernel(const BatchArgs b)
{
    __shared__ __align__(16) DecodeLds<KB, FORM != kReadTable> lds;
    uint32_t i = 0, first = 0;
    while (i + 1 < b.count && blockIdx.x >= b.t[i].wg_end) {
        first = b.t[i].wg_end;
        ++i;
    }
    const DecodeArgs a = b.t[i];
    if constexpr (FORM == kEntries || FORM == kEntriesAlone) {
        if (a.mid_states) {
            decode_from_entries<KB, NORM, MODE, FORM == kEntriesAlone>(a, blockIdx.x - first, lds.lut, lds.steps, lds.stage, lds.spread);
            return;
        }
    }
    if constexpr (FORM == kMakeTable) {
        if (!holds_table(a.n_chunks)) {
            decode_workgroup<KB, NORM, MODE, kMakeTable>(a, blockIdx.x - first, lds.lut, lds.steps, lds.stage, lds.spread);
            return;
        }
    }
    decode_workgroup<KB, NORM, MODE, kReadTable>(a, blockIdx.x - first, lds.lut, lds.steps, lds.stage, lds.spread);
}

// The entry points of an imported blob: every lane walks its state to them, writing nothing.  A workgroup's words go
// through LDS, as in the decoder (with every word fetched from the blob behind the one before it, the launch was a chain
// of memory latencies: the import of 50 000 elements took 94 us).  A run fed from a damaged container consumes at most
// one word per symbol and stays inside the slack behind the words, here and in the window; the decoder reports it.
constexpr uint32_t kEntryThreads = 256;
constexpr uint32_t kEntryOverrun = (kMidTurn * kRun + 1) * 2;  // bytes a walk can pass the end of its run by

template <class WordSrc>
__device__ __forceinline__ void walk_to_entry(const uint32_t *__restrict__ lut, const WordSrc &src, uint32_t m, uint32_t j,
                                              uint32_t &x, uint32_t &wp)
{
    constexpr bool EAGER = !std::is_same<WordSrc, GlobalWords>::value;
    uint32_t next = src.peek(wp);
    for (uint32_t at = j * kRun; at < m && at < kMidTurn * kTurn; at += kTurn) {
        if (m - at >= kRun) {
#pragma unroll
            for (uint32_t t = 0; t < kRun; ++t)
                rans_get<EAGER>(lut, x, wp, next, src);
        } else {
            for (uint32_t t = 0; t < m - at; ++t)
                rans_get<EAGER>(lut, x, wp, next, src);
        }
    }
}

__global__ __launch_bounds__(kEntryThreads) void entry_points_kernel(const DecodeArgs a, uint32_t *__restrict__ mid_states,
                                                                     uint8_t *__restrict__ mid_lens)
{
    __shared__ __align__(16) uint32_t lut[kM];
    __shared__ __align__(16) uint32_t steps[kSteps];
    __shared__ __align__(16) uint8_t stage[kStageBytes];
    const uint32_t tid = threadIdx.x;
    const uint32_t c0 = blockIdx.x * (kEntryThreads / kStates);
    const uint32_t c1 = c0 + kEntryThreads / kStates < a.n_chunks ? c0 + kEntryThreads / kStates : a.n_chunks;
    const uint64_t byte0 = static_cast<uint64_t>(a.offsets[c0]) * 2, byte1 = static_cast<uint64_t>(a.offsets[c1]) * 2;
    const uint64_t aligned0 = byte0 & ~static_cast<uint64_t>(15);
    const uint64_t stage_len = byte1 - aligned0;
    const bool staged = stage_len + 16 + kEntryOverrun <= kStageBytes;
    const bool lone = a.tb->lone < 256;
    for (uint32_t i = tid; i < kSteps; i += kEntryThreads)
        steps[i] = a.tb->steps[i];
    if (staged) {
        const uint4 *from = reinterpret_cast<const uint4 *>(reinterpret_cast<const uint8_t *>(a.words) + aligned0);
        for (uint32_t i = tid; static_cast<uint64_t>(i) * 16 < stage_len; i += kEntryThreads)
            reinterpret_cast<uint4 *>(stage)[i] = from[i];
    }
    __syncthreads();
    if (!lone)
        for (uint32_t piece = tid; piece < kM / 8; piece += kEntryThreads)
            make_piece(steps, a.tb->step_of[piece], piece, lut);
    __syncthreads();
    const uint32_t c = c0 + tid / kStates, j = tid % kStates, id = c * kStates + j;
    if (c >= a.n_chunks)
        return;
    const uint32_t len = a.lens[id];
    uint32_t before = len;
#pragma unroll
    for (uint32_t d = 1; d < kStates; d <<= 1) {
        const uint32_t o = __shfl_up(before, d, kStates);
        if (j >= d)
            before += o;
    }
    before -= len;
    const uint64_t base = static_cast<uint64_t>(c) * kChunk;
    const uint32_t m = (a.n - base) < kChunk ? static_cast<uint32_t>(a.n - base) : kChunk;
    const uint64_t run_byte = (static_cast<uint64_t>(a.offsets[c]) + before) * 2;
    uint32_t x = a.states[id], wp = 0, wp_begin = 0;
    if (!lone && staged) {
        wp = wp_begin = static_cast<uint32_t>(run_byte - aligned0);
        walk_to_entry(lut, LdsWords{stage}, m, j, x, wp);
    } else if (!lone) {
        walk_to_entry(lut, GlobalWords{reinterpret_cast<const uint8_t *>(a.words) + run_byte}, m, j, x, wp);
    }
    mid_states[id] = x;
    mid_lens[id] = static_cast<uint8_t>((wp - wp_begin) / 2);
}

// ------------------------------------------------------------------------------------------
// Measurement aid: the decoder's memory traffic without its arithmetic, in the decoder's own launch
// shape.  A workgroup of 512 lanes owns 32 chunks of 8 KB of output and holds the decoder's LDS (so the
// same 16 waves per CU are resident); it first copies its share of the "word" input into LDS with
// 128-bit loads behind one barrier; then lane (chunk, state) reads FW bytes of "field" input and writes
// 16 bytes per turn, 256 bytes apart, turns taken four at a time with the next four field loads in
// flight, non-temporal stores for outputs beyond the last-level cache -- the decoder's instructions
// with nothing between them.  What it reaches is the ceiling for a decoder with this access pattern on
// this machine; the decoder's own rate is reported against it.
// ------------------------------------------------------------------------------------------
template <int FW, bool STREAM>
__global__ __launch_bounds__(kDecThreads) void stream_probe_kernel(const uint8_t *__restrict__ fields,
                                                                   const uint4 *__restrict__ words, uint32_t word_vecs_per_wg,
                                                                   uint4 *__restrict__ out, uint32_t n_chunks,
                                                                   uint32_t *__restrict__ sink)
{
    __shared__ __align__(16) uint32_t lut[kM];
    __shared__ __align__(16) uint8_t stage[kStageBytes];
    const uint32_t tid = threadIdx.x, c = blockIdx.x * kDecChunksPerWg + tid / kStates, j = tid % kStates;
    const uint4 *from = words + static_cast<uint64_t>(blockIdx.x) * word_vecs_per_wg;
    for (uint32_t i = tid; i < word_vecs_per_wg; i += kDecThreads)
        reinterpret_cast<uint4 *>(stage)[i % (kStageBytes / 16)] = from[i];
    lut[tid] = tid;
    __syncthreads();
    uint32_t acc = lut[(tid * 7u) % kM] ^ reinterpret_cast<const uint32_t *>(stage)[tid];
    if (c >= n_chunks)
        return;
    typedef typename std::conditional<FW == 8, uint2, typename std::conditional<FW == 4, uint32_t,
            typename std::conditional<FW == 2, uint16_t, uint8_t>::type>::type>::type field_t;
    const field_t *f = reinterpret_cast<const field_t *>(fields + static_cast<uint64_t>(c) * (kTurns * kStates * FW)) + j;
    uint4 *o = out + static_cast<uint64_t>(c) * (kChunk / 8) + j;
    constexpr uint32_t kBurst = kTurnGroupStream;
    field_t now[kBurst];
#pragma unroll
    for (uint32_t r = 0; r < kBurst; ++r)
        now[r] = f[r * kStates];
    for (uint32_t q = 0; q < kTurns; q += kBurst) {
        field_t next[kBurst];
        const uint32_t qn = q + kBurst < kTurns ? q + kBurst : q;
#pragma unroll
        for (uint32_t r = 0; r < kBurst; ++r)
            next[r] = f[(qn + r) * kStates];
#pragma unroll
        for (uint32_t r = 0; r < kBurst; ++r) {
            uint32_t lo, hi;
            if constexpr (FW == 8) {
                lo = now[r].x;
                hi = now[r].y;
            } else {
                lo = now[r];
                hi = q;
            }
            const uint4 w = make_uint4(lo, hi, acc, q + r);
            uint4 *dst = &o[(q + r) * kStates];
            if constexpr (STREAM) {
                __builtin_nontemporal_store(w.x, &dst->x);
                __builtin_nontemporal_store(w.y, &dst->y);
                __builtin_nontemporal_store(w.z, &dst->z);
                __builtin_nontemporal_store(w.w, &dst->w);
            } else {
                *dst = w;
            }
            now[r] = next[r];
        }
    }
    if (acc == 0x9E3779B9u)  // keeps the LDS reads alive; practically never taken
        atomicOr(sink, 1u);
}

}  // namespace nz
