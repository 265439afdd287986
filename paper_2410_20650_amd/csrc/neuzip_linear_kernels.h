// Linear layer on a compressed weight for gfx950: the rANS decoder feeding the matrix cores.
//
// Sec. 2.2, compressed forward pass:  W_hat <- decompress(c_l);  x_l <- W_hat x_{l-1} + b_l.
// Here the two steps are one kernel: the decoded and merged bf16 words of a state's turn (8
// neighbouring weights of one row) are, as they stand in the lane's registers, one lane's share
// of the B operand of v_mfma_f32_16x16x32_bf16, so W_hat is never written to memory.
//
// Operand shapes of that instruction (wave64):  A is 16 x 32 (lane l holds row l % 16,
// k = 8 * (l / 16) .. + 7),  B is 32 x 16 (lane l holds column l % 16, same k),  D is 16 x 16
// float (lane l holds column l % 16, rows 4 * (l / 16) .. + 3).  A = 16 tokens of the
// activations, B = 16 rows of the weight, both over the same 32 input features.
//
// Lane assignment.  A workgroup of 512 threads walks 32 chunks as two groups of 16, or, from the entry
// points, one group of 16 with two waves where there was one, for the two halves of its states.  In a group,
// wave sq (0..3) and lane l own state j = 4 * sq + l / 16 of chunk number l % 16 of the group.
// At turn t that state holds the weights at flat index chunk * 4096 + t * 128 + j * 8 .. + 7, so
// a wave holds, for 16 chunks, the 32 neighbouring input features t * 128 + sq * 32 .. + 31:
// exactly a B operand, provided the 16 chunks sit at the same input-feature offset.  Chunks that
// are `stride` = in_features / gcd(in_features, 4096) apart do (stride * 4096 is a whole number of
// rows), so a group is chunks first + stride * (0..15).
// Every wave accumulates its own share of the input features of a row piece.  Where a row ends inside the
// walk, its partial sums go to y with float atomics (y then starts as the bias, or zero).  At the end of
// the walk the waves of a group add theirs up in LDS first (unless the tokens are few, see
// kLinDirectTokens) and one atomic leaves per sum; and where a chunk is a whole row the sum is complete
// there and is stored with the bias, without atomics and without y set up before.
//
// Two forms, template parameter COLS.  COLS = 16 is the above.  COLS = 32 uses
// v_mfma_f32_32x32x16_bf16 (A 32 x 16, B 16 x 32, lane l: row / column l % 32, k = 8 * (l / 32)
// .. + 7; D: lane l holds column l % 32 and rows (r / 4) * 8 + (l / 32) * 4 + r % 4, r = 0..15):
// the workgroup's 32 chunks form one group, wave w and lane l own state 2 w + l / 32 of chunk
// l % 32.  The weights held per wave and turn are the same 512, but one 128-bit activation load
// per lane now serves 32 tokens instead of 16, which is what limits larger batches.
#pragma once

#include "neuzip_format.h"
#include "neuzip_decode_kernels.h"

namespace nz {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;

// Accumulator tile and matrix instruction of the two forms
template <int COLS>
struct LinearTile;
template <>
struct LinearTile<16> {
    typedef f32x4_t acc_t;
    static constexpr int kRegs = 4;
    static __device__ __forceinline__ acc_t mma(bf16x8_t a, bf16x8_t b, acc_t c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
    // token (row of D) held in register r of lane `lane`
    static __device__ __forceinline__ uint32_t row(uint32_t lane, int r) { return (lane >> 4) * 4 + r; }
};
template <>
struct LinearTile<32> {
    typedef f32x16_t acc_t;
    static constexpr int kRegs = 16;
    static __device__ __forceinline__ acc_t mma(bf16x8_t a, bf16x8_t b, acc_t c)
    {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ uint32_t row(uint32_t lane, int r)
    {
        return (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
    }
};

constexpr uint32_t kLinThreads = 512;
constexpr uint32_t kLinMaxTokens = 64;
// Up to here the waves of a group add their sums to y by themselves (where they are not complete in the
// workgroup): 4096 x 14336, 1 token, 35.6 us, with the sums added up in LDS first 35.8; 8 tokens 36.5 and 35.9, 16
// tokens 43.1 and 38.4.
constexpr uint32_t kLinDirectTokens = 4;

struct LinearArgs {
    const TableBlock *tb;
    const uint32_t *offsets;
    const uint32_t *states;
    const uint8_t *lens;
    const uint32_t *mid_states;  // entry points (nullptr: none)
    const uint8_t *mid_lens;
    const uint16_t *words;
    const uint8_t *sm;
    const uint8_t *coef;   // block coefficients (block-wise normalised blobs only)
    uint32_t block_shift;  // log2 of the block size of the normalisation
    const uint16_t *x;     // [tokens][in_features] bf16
    float *y;              // [tokens][out_features], holds the bias (or zero) on entry unless whole_rows
    uint32_t *status;
    uint64_t n;
    uint32_t n_chunks;
    uint32_t in_features;
    uint32_t out_features;
    uint32_t tokens;
    uint32_t stride;       // chunks between neighbouring columns of a group
    uint32_t n_groups;
    uint32_t split;        // 1: two lanes walk a state's two halves from the entry points
    uint32_t whole_rows;   // a chunk is a row of the weight: sums are complete in the workgroup
    const float *bias;     // whole_rows: added to the sums here (nullptr: none); otherwise y holds it on entry
};

// Several weights applied to the same kind of input in one launch (the q, k and v projections of an
// attention block, say): workgroups [wg_end[i-1], wg_end[i]) belong to weight i.  Weights too small to
// fill the chip on their own overlap with the others.
constexpr uint32_t kLinBatchMax = 4;
struct LinearBatchArgs {
    LinearArgs t[kLinBatchMax];
    uint32_t wg_end[kLinBatchMax];
    uint32_t count;
};
struct LinearInitBatchArgs {
    float *y[kLinBatchMax];
    const float *bias[kLinBatchMax];
    uint32_t out_features[kLinBatchMax];
    uint32_t wg_end[kLinBatchMax];
    uint32_t tokens, count;
};

// y[t][o] = bias[o] (or 0): the accumulation target of the kernel below
__global__ void linear_init_kernel(float *__restrict__ y, const float *__restrict__ bias, uint32_t tokens,
                                   uint32_t out_features)
{
    const uint64_t i = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < static_cast<uint64_t>(tokens) * out_features)
        y[i] = bias ? bias[i % out_features] : 0.0f;
}

__global__ void linear_init_batch_kernel(const LinearInitBatchArgs b)
{
    uint32_t i = 0, first = 0;
    while (i + 1 < b.count && blockIdx.x >= b.wg_end[i]) {
        first = b.wg_end[i];
        ++i;
    }
    const uint64_t at = static_cast<uint64_t>(blockIdx.x - first) * blockDim.x + threadIdx.x;
    if (at < static_cast<uint64_t>(b.tokens) * b.out_features[i])
        b.y[i][at] = b.bias[i] ? b.bias[i][at % b.out_features[i]] : 0.0f;
}

__device__ __forceinline__ void atomic_add_f32(float *p, float v)
{
    // the hardware float add of the memory system (no compare-and-swap loop); y is ordinary
    // device memory, which is what that instruction requires
    unsafeAtomicAdd(p, v);
}

// NORM: the blob is block-wise normalised (Sec. 2.3): the merged words are multiplied by their block's
// coefficient, as in the decoder, before they enter the matrix instruction.
// The partial sums of the last row that the walk touched stay in acc, that row in `row`.
template <int KB, int COLS, int MT, bool LONE, bool NORM, bool EAGER, class WordSrc>
__device__ __forceinline__ void linear_walk(const uint32_t *__restrict__ lut, const WordSrc &src, uint32_t lone,
                                            uint32_t &x, uint32_t &wp, const uint8_t *__restrict__ sm,
                                            const LinearArgs &a, uint64_t base, uint32_t kk, uint32_t turns,
                                            uint32_t all_turns, uint32_t j, uint32_t lane,
                                            typename LinearTile<COLS>::acc_t (&acc)[MT], uint32_t &row)
{
    const uint32_t in = a.in_features, out_features = a.out_features, tokens = a.tokens;
    float *__restrict__ y = a.y;
    typedef LinearTile<COLS> Tile;
    constexpr uint32_t kPerWave = 64 / COLS;         // states of a chunk held by one wave (4 or 2)
    const uint32_t col = lane & (COLS - 1);          // column of B and of D: this lane's chunk
    const uint32_t kq = (j % kPerWave) * 8u;         // this lane's 8 input features inside the wave's 32 or 16
    const uint32_t ksq = (j / kPerWave) * kPerWave * 8u;  // the wave's features inside the turn's 128
    // Position in the matrix: the row is the lane's own (its chunk's); the input-feature offset kk
    // is that of the group's first chunk, which all 16 chunks share -- lanes without a chunk use
    // it too, because every lane supplies activations to A.
    row = static_cast<uint32_t>(base / in);
    // rows of the activations this lane supplies to A (clamped: rows past `tokens` are never stored)
    const uint16_t *xrow[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        uint32_t t = mt * COLS + col;
        t = t < a.tokens ? t : a.tokens - 1;
        xrow[mt] = a.x + static_cast<uint64_t>(t) * in + ksq + kq;
    }
    uint32_t next = LONE ? 0u : src.peek(wp);
    // A turn's inputs are requested once the turn before is done and travel while its own eight symbols are decoded.  (Requested a
    // whole turn earlier, or more, they only take registers and places in the queue: 4096 x 14336, 32 tokens, 43.2 us, with two
    // buffers 48.8; 4096 x 4096, 64 tokens, 25.8 / 26.9; 9000 x 5120, 64 tokens, 86.7 / 89.3.)  A lane without turns of its own
    // reads those of the tensor's first chunk; a turn behind the last reads the last again.  The buffers are written as a
    // rotation of DEPTH of them because of what the compiler makes of it, which is to move the request of the fields alone to
    // the turn's beginning: with one plain buffer it does not (4096 x 4096, 1 token, 16.7 us -> 17.8).  The fields of normalised
    // weights are one value with the coefficient and stay where they are: in the walk of 16 columns they are requested ahead by
    // hand, apart from the coefficient (4096 x 14336, k = 3, blocks of 128, 1 token, 47.8 us -> 43.4, 10937 x 3584, 64 tokens,
    // 134.1 -> 129.8; but not with two tiles of tokens, 32 tokens 79.4 -> 83.7, nor in the walk of 32 columns, 4096 x 14336,
    // k = 0, blocks of 64, 32 tokens, 56.1 -> 58.7).
    constexpr uint32_t DEPTH = 1;
    constexpr bool APART = NORM && COLS == 16 && MT != 2;
    const uint64_t first = (turns > 0 ? base : 0u) + j * kRun;
    const uint32_t last = turns > 0 ? turns - 1 : 0u;
    uint64_t fields[DEPTH];
    uint32_t coef[DEPTH];
    uint4 xa[DEPTH][MT];
    uint32_t ahead = kk;  // the input-feature offset of the turn requested next
    auto request = [&](uint32_t d, uint32_t q) {
        const uint64_t at = first + min(q, last) * kTurn;
        if constexpr (APART)
            coef[d] = a.coef[at >> a.block_shift];
        else
            fields[d] = load_turn<KB, NORM>(sm, a.coef, a.block_shift, at);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
            xa[d][mt] = *reinterpret_cast<const uint4 *>(xrow[mt] + ahead);
        ahead = ahead + kTurn == in ? 0u : ahead + kTurn;
    };
#pragma unroll
    for (uint32_t d = 0; d < DEPTH; ++d) {
        if constexpr (APART)
            fields[d] = load_fields<KB>(sm, first + min(d, last) * kTurn);
        request(d, d);
    }

    // the trip count is the same for every lane of the wave (the matrix instruction needs them
    // all); a lane whose chunk is shorter or absent supplies zeros
    static_assert(kTurns % DEPTH == 0 && kMidTurn % DEPTH == 0, "whole rotations");
    for (uint32_t q0 = 0; q0 < all_turns; q0 += DEPTH) {
#pragma unroll
        for (uint32_t d = 0; d < DEPTH; ++d) {
            const uint32_t q = q0 + d;
            const bool mine = q < turns;
            const uint32_t kk_next = kk + kTurn == in ? 0u : kk + kTurn;
            uint64_t fields_next = 0;
            if constexpr (APART)
                fields_next = load_fields<KB>(sm, first + min(q + DEPTH, last) * kTurn);

            union {
                uint32_t u[4];
                bf16x8_t v;
            } b;
            b.u[0] = b.u[1] = b.u[2] = b.u[3] = 0;
            if (mine) {
                uint32_t e[8];
#pragma unroll
                for (int t = 0; t < 8; ++t)
                    e[t] = LONE ? lone : rans_get<EAGER>(lut, x, wp, next, src);
                b.u[0] = merge_pair<KB>(fields[d], 0, e[0], e[1]);
                b.u[1] = merge_pair<KB>(fields[d], 1, e[2], e[3]);
                b.u[2] = merge_pair<KB>(fields[d], 2, e[4], e[5]);
                b.u[3] = merge_pair<KB>(fields[d], 3, e[6], e[7]);
                if constexpr (NORM) {
                    const float c = coefficient((APART ? coef[d] : static_cast<uint32_t>(fields[d] >> 32)) & 0x7Fu);
#pragma unroll
                    for (int p = 0; p < 4; ++p)
                        b.u[p] = denormalise_pair(b.u[p], c);
                }
            }
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                union {
                    uint4 q4;
                    bf16x8_t v;
                } av;
                av.q4 = xa[d][mt];
                acc[mt] = Tile::mma(av.v, b.v, acc[mt]);
            }
            request(d, q + DEPTH);
            // end of a row of the weight inside the walk: this wave's partial sums leave for y
            if (kk_next == 0 && q + 1 < all_turns) {
                const bool col_live = mine && row < out_features;
                // (one running offset: the compiler would hold an address per register of the tile otherwise, and
                // with them a second workgroup's worth of registers)
                uint64_t at = static_cast<uint64_t>(Tile::row(lane, 0)) * out_features + row;
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
                    for (int r = 0; r < Tile::kRegs; ++r) {
                        const uint32_t t = mt * COLS + Tile::row(lane, r);
                        if (col_live && t < tokens)
                            atomic_add_f32(y + at, acc[mt][r]);
                        acc[mt][r] = 0.0f;
                        const int beyond = r + 1 < Tile::kRegs ? static_cast<int>(Tile::row(0, r + 1) - Tile::row(0, r))
                                                               : COLS - static_cast<int>(Tile::row(0, r));
                        at += static_cast<uint64_t>(beyond) * out_features;
                        asm volatile("" : "+v"(at));
                    }
                }
                ++row;
            }
            kk = kk_next;
            if constexpr (APART)
                fields[d] = fields_next;
        }
    }
}

// READ: every weight of the launch is walked whole and holds its slot table (with the choice of both left to run time
// 4096 x 14336, 1 token, took 36.4 us, 35.7 now, and 8192 x 8192 36.7, 35.9 now).
// EAGER: the step of the walk without a branch (see rans_get).
template <int KB, int COLS, int MT, bool NORM, bool READ, bool EAGER>
__device__ __forceinline__ void linear_workgroup(const LinearArgs &a, uint32_t wg, uint32_t *__restrict__ lut,
                                                 uint32_t *__restrict__ steps, uint8_t *__restrict__ stage)
{
    constexpr uint32_t kLinGroupChunks = COLS;                       // columns of the B operand
    constexpr uint32_t kPerWave = 64 / COLS;                         // states of a chunk per wave: 4 or 2
    const uint32_t split = COLS == 16 && !READ ? a.split : 0u;                // two waves for the halves of a wave's states
    const uint32_t waves_per_group = (kStates / kPerWave) << split;  // 4 (8 with entry points), or 8
    const uint32_t groups_per_wg = kLinThreads / 64 / waves_per_group;
    const uint32_t group_window = kStageBytes / groups_per_wg;       // LDS window of one group's word runs
    const uint32_t cols_per_wave = COLS / waves_per_group;           // columns a wave copies
    const uint32_t tid = threadIdx.x;
    // (the same for all lanes, and told so: what follows from it stays in scalar registers)
    const uint32_t wave = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(tid >> 6)));
    const uint32_t lane = tid & 63u;
    const uint32_t g = wave / waves_per_group, in_group = wave % waves_per_group;
    const uint32_t part = split ? in_group & 1u : 0u;                // before (0) or behind (1) the entry points
    const uint32_t col = lane & (COLS - 1);
    const uint32_t j = (in_group >> split) * kPerWave + lane / COLS;
    const uint32_t group = wg * groups_per_wg + g;
    const bool group_live = group < a.n_groups;
    // group -> its COLS chunks: `stride` groups interleave inside a block of COLS * stride chunks
    const uint32_t block_id = group / a.stride, first_in_block = group % a.stride;
    const uint64_t c64 = static_cast<uint64_t>(block_id) * kLinGroupChunks * a.stride + first_in_block +
                         static_cast<uint64_t>(a.stride) * col;
    const bool live = group_live && c64 < a.n_chunks;
    const uint32_t turn0 = part * kMidTurn, all_turns = split ? kMidTurn : kTurns;
    const uint32_t kk0 = static_cast<uint32_t>(
        ((static_cast<uint64_t>(block_id) * kLinGroupChunks * a.stride + first_in_block) * kChunk + turn0 * kTurn) % a.in_features);
    const uint32_t c = live ? static_cast<uint32_t>(c64) : 0u;
    const uint64_t base = static_cast<uint64_t>(c) * kChunk;
    const uint32_t m = !live ? 0u : ((a.n - base) < kChunk ? static_cast<uint32_t>(a.n - base) : kChunk);
    // in_features is a multiple of 128, so chunks hold whole turns; this lane's share of them
    const uint32_t upto = m / kTurn < turn0 + all_turns ? m / kTurn : turn0 + all_turns;
    const uint32_t turns = upto > turn0 ? upto - turn0 : 0u;

    // ---- loads that depend on nothing
    // (lanes without a chunk read the first one's: no branch, and no wait in front of the loads behind it)
    const uint32_t off_c = a.offsets[c];
    const uint32_t off_c1 = a.offsets[c + 1];
    uint32_t x = a.states[c * kStates + j];
    const uint4 lens16 = *reinterpret_cast<const uint4 *>(a.lens + static_cast<uint64_t>(c) * kStates);
    uint32_t mid_x = kRansL, mid_len = 0;
    if (split) {
        mid_x = a.mid_states[c * kStates + j];
        mid_len = a.mid_lens[c * kStates + j];
    }
    const uint32_t lone = a.tb->lone;
    // the tensor's table: its steps (walked from the entry points, or too small to hold the table) or the slot table itself
    const bool make_lut = !READ && (split || !holds_table(a.n_chunks));
    static_assert(kLinThreads == kM / 8, "one piece of the slot table per thread");
    const uint32_t begins[2] = {make_lut ? a.tb->step_of[tid] : 0u, 0u};  // the step that this thread's piece begins in
    uint4 table_piece[2];
#pragma unroll
    for (uint32_t r = 0; r < 2; ++r) {
        const uint32_t i = tid + r * kLinThreads;
        table_piece[r] = make_uint4(0, 0, 0, 0);
        if (!make_lut)
            table_piece[r] = reinterpret_cast<const uint4 *>(a.tb->lut)[i];
        else if (i < kSteps / 4)
            table_piece[r] = reinterpret_cast<const uint4 *>(a.tb->steps)[i];
    }

    // ---- stage the word runs of the group's chunks: each chunk's piece of the blob, from the
    // 16-byte boundary below its first word, one after the other in the group's window
    const uint64_t byte0 = static_cast<uint64_t>(off_c) * 2, byte1 = static_cast<uint64_t>(off_c1) * 2;
    const uint64_t aligned0 = byte0 & ~static_cast<uint64_t>(15);
    const uint32_t piece = live ? static_cast<uint32_t>((byte1 - aligned0 + 15) & ~static_cast<uint64_t>(15)) : 0u;
    // exclusive prefix over the columns (lanes with equal lane / COLS agree)
    uint32_t place = COLS == 16 ? row_scan_u32(piece) : half_scan_u32(piece);
    const uint32_t group_bytes = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(place), COLS - 1));
    place -= piece;
    const bool staged = group_bytes + 16 <= group_window;
    uint8_t *window = stage + g * group_window;
    // A wave copies cols_per_wave columns straight into LDS (kMostCols, or half as many with entry points), all of them
    // requested together, while the table is made.
    auto of_column = [&](uint32_t v, uint32_t r) {
        return static_cast<uint32_t>(
            __builtin_amdgcn_readlane(static_cast<int>(v), static_cast<int>((in_group * cols_per_wave + r) & 63u)));
    };
    if (make_lut && tid < kSteps / 4)
        reinterpret_cast<uint4 *>(steps)[tid] = table_piece[0];
    asm volatile("" ::"v"(begins[0]));  // (taken here, and not waited for behind the words)
    for (uint32_t r = 0; r < cols_per_wave; ++r) {
        const uint64_t at = of_column(static_cast<uint32_t>(aligned0), r) |
                            (static_cast<uint64_t>(of_column(static_cast<uint32_t>(aligned0 >> 32), r)) << 32);
        const uint32_t len = staged && group_live ? of_column(piece, r) : 0u;
        const uint4 *from = reinterpret_cast<const uint4 *>(reinterpret_cast<const uint8_t *>(a.words) + at);
        uint8_t *to = window + of_column(place, r);
        for (uint32_t i = 0; i * 16 < len; i += 64)
            if ((i + lane) * 16 < len)
                copy_to_lds(from + i + lane, to + i * 16);
    }
    if (make_lut) {
        lds_barrier();
        if (lone >= 256)
            make_table(steps, begins, a.tb, lut);
    } else {
#pragma unroll
        for (uint32_t r = 0; r < 2; ++r)
            reinterpret_cast<uint4 *>(lut)[tid + r * kLinThreads] = table_piece[r];
    }
    wait_for_memory_acks();  // the words
    __syncthreads();
    // ---- start of this state's run: the chunk's offset plus the lengths of the states before it
    const uint32_t lw[4] = {lens16.x, lens16.y, lens16.z, lens16.w};
    uint32_t before = 0, len = 0;
#pragma unroll
    for (uint32_t s = 0; s < kStates; ++s) {
        const uint32_t l8 = (lw[s >> 2] >> (8 * (s & 3u))) & 0xFFu;
        before += s < j ? l8 : 0u;
        len = s == j ? l8 : len;
    }
    // the half before the entry point ends there, the other one where the encoder started
    const uint32_t x_end = split && !part ? mid_x : kRansL;
    const uint32_t words_here = !split ? len : (part ? len - mid_len : mid_len);
    if (part) {
        x = mid_x;
        before += mid_len;
    }
    const uint64_t run_byte = (static_cast<uint64_t>(off_c) + before) * 2;
    const uint64_t from_elem = base + turn0 * kTurn;

    typedef LinearTile<COLS> Tile;
    typename Tile::acc_t acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int r = 0; r < Tile::kRegs; ++r)
            acc[mt][r] = 0.0f;
    uint32_t row = 0;
    if (group_live) {
        uint32_t wp = 0, wp_begin = 0;
        if (lone < 256) {
            linear_walk<KB, COLS, MT, true, NORM, EAGER>(lut, NoWords{}, lone, x, wp, a.sm, a, from_elem, kk0, turns, all_turns, j,
                                                  lane, acc, row);
        } else if (staged) {
            wp = wp_begin = g * group_window + place + static_cast<uint32_t>(run_byte - aligned0);
            linear_walk<KB, COLS, MT, false, NORM, EAGER>(lut, LdsWords{stage}, 0u, x, wp, a.sm, a, from_elem, kk0, turns, all_turns,
                                                   j, lane, acc, row);
        } else {
            const GlobalWords direct{reinterpret_cast<const uint8_t *>(a.words) + run_byte};
            linear_walk<KB, COLS, MT, false, NORM, false>(lut, direct, 0u, x, wp, a.sm, a, from_elem, kk0, turns, all_turns, j, lane,
                                                   acc, row);
        }
        if (live && (x != x_end || wp - wp_begin != 2 * words_here))
            atomicOr(a.status, 1u);
    }

    // ---- the waves that hold partial sums of the same row (those of the group, or of its half when a chunk is not
    // a whole row) add them up in LDS, tile of tokens by tile of tokens, one sum per thread; then they are complete
    // and go to y with the bias, or leave by one atomic per sum instead of one per wave
    constexpr uint32_t kSums = Tile::kRegs * 64;                // of one tile
    const uint32_t half = split && !a.whole_rows ? part : 0u;   // waves of the two halves end in different rows
    const uint32_t sharing = split && !a.whole_rows ? waves_per_group / 2 : waves_per_group;
    const uint32_t place_in = split && !a.whole_rows ? in_group >> 1 : in_group;
    const uint32_t set = split && !a.whole_rows ? g * 2 + half : g;
    static_assert(kLinThreads / 64 * kSums * sizeof(float) <= kStageBytes, "the sums of a tile take the words' place");
    float *sums = reinterpret_cast<float *>(stage) + set * sharing * kSums;
    const uint32_t chunk_turns = m / kTurn;
    const bool row_live = live && chunk_turns > turn0 && row < a.out_features;
    if (MT == 1 && !a.whole_rows && !split && a.tokens <= kLinDirectTokens) {
#pragma unroll
        for (int r = 0; r < Tile::kRegs; ++r)
            if (row_live && Tile::row(lane, r) < a.tokens)
                atomic_add_f32(a.y + static_cast<uint64_t>(Tile::row(lane, r)) * a.out_features + row, acc[0][r]);
        return;
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        __syncthreads();
#pragma unroll
        for (int r = 0; r < Tile::kRegs; ++r)
            sums[place_in * kSums + r * 64 + lane] = acc[mt][r];
        __syncthreads();
        for (uint32_t r = place_in; r < Tile::kRegs; r += sharing) {
            float total = 0.0f;
            for (uint32_t w = 0; w < sharing; ++w)
                total += sums[w * kSums + r * 64 + lane];
            const uint32_t t = mt * COLS + Tile::row(lane, static_cast<int>(r));
            if (row_live && t < a.tokens) {
                float *at = a.y + static_cast<uint64_t>(t) * a.out_features + row;
                if (a.whole_rows)
                    *at = total + (a.bias ? a.bias[row] : 0.0f);
                else
                    atomic_add_f32(at, total);
            }
        }
    }
}

// (Two workgroups of 8 waves share a CU if a lane has at most 128 registers; with the 138 the compiler took
// for 64 tokens it held one.)
template <int KB, int COLS, int MT, bool NORM, bool READ, bool EAGER>
__global__ __launch_bounds__(kLinThreads, 4) void linear_batch_kernel(const LinearBatchArgs b)
{
    __shared__ __align__(16) struct {
        uint8_t stage[kStageBytes];  // first: a direct copy's LDS address has 16 bits
        uint32_t lut[kM];
        uint32_t steps[READ ? 4 : kSteps];
    } lds;
    uint32_t i = 0, first = 0;
    while (i + 1 < b.count && blockIdx.x >= b.wg_end[i]) {
        first = b.wg_end[i];
        ++i;
    }
    linear_workgroup<KB, COLS, MT, NORM, READ, EAGER>(b.t[i], blockIdx.x - first, lds.lut, lds.steps, lds.stage);
}

}  // namespace nz
