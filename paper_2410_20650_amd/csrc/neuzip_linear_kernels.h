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
// points, one group of 16 with two sets of waves, for the two halves of its states.  In a group,
// wave sq (0..3) and lane l own state j = 4 * sq + l / 16 of chunk number l % 16 of the group.
// At turn t that state holds the weights at flat index chunk * 4096 + t * 128 + j * 8 .. + 7, so
// a wave holds, for 16 chunks, the 32 neighbouring input features t * 128 + sq * 32 .. + 31:
// exactly a B operand, provided the 16 chunks sit at the same input-feature offset.  Chunks that
// are `stride` = in_features / gcd(in_features, 4096) apart do (stride * 4096 is a whole number of
// rows), so a group is chunks first + stride * (0..15).
//
// Every wave accumulates its own share of the input features of a row piece.  Where a row ends, inside the walk or at its end,
// the waves of a group add their sums up in LDS and one of them leaves per row and token.  Wave by wave, as float atomics, they
// were 4 or 8 times as many (us, wave by wave / added up: 57344 x 1024, 16 tokens, 61 / 39, 64 tokens 173 / 54; 100000 x 512, 64
// tokens, 588 / 83; 12000 x 4736, 64 tokens, 209 / 93).  Rows that do not pass the end of a chunk are complete then and are stored
// with the bias; the sums of others are added to y, or stored by themselves for a second launch to add up (see LinearArgs).
//
// Two forms, template parameter COLS.  COLS = 16 is the above.  COLS = 32 uses
// v_mfma_f32_32x32x16_bf16 (A 32 x 16, B 16 x 32, lane l: row / column l % 32, k = 8 * (l / 32)
// .. + 7; D: lane l holds column l % 32 and rows (r / 4) * 8 + (l / 32) * 4 + r % 4, r = 0..15):
// the workgroup's 32 chunks form one group, wave w and lane l own state 2 w + l / 32 of chunk
// l % 32.  The weights held per wave and turn are the same 512, but one 128-bit activation load
// per lane now serves 32 tokens instead of 16.
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
// Up to so many sums the waves add those of a row that ends inside the walk to y by themselves: the two barriers of adding them up
// first cost more than the atomics, until these are too many, the sooner the more of a wave's 64 lanes send (by themselves / added up:
// 16000 x 640, 1 token, 16.9 / 17.9 us, 90000 x 640 35.3 / 38.1; 40000 x 640, 2 tokens, 27.7 / 30.5; 15000 x 640, 3 tokens, 18.1 / 18.5,
// 25000 x 640 23.8 / 19.1; 5000 x 1152, 4 tokens, 17.1 / 17.8, 13000 x 640 19.2 / 18.6; 5 tokens: 900 x 384 17.9 / 19.3, 2000 x 1152
// 17.1 / 17.6, 3000 x 640 18.5 / 18.3; 6 tokens: 600 x 1152 17.2 / 18.0, 1000 x 640 18.9 / 18.5; 260 x 384, 10 tokens, 18.1 / 18.9; 500 x
// 384, 8 tokens, 21.5 / 20.1; 120 x 1152, 16 tokens, 15.9 / 17.0, 300 x 640, 12 tokens, 19.1 / 18.4).
constexpr uint32_t direct_sums(uint32_t tokens)
{
    return tokens <= 2 ? 90000 : tokens <= 4 ? 45000 : tokens == 5 ? 10000 : tokens == 6 ? 5000 : 2500;
}

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
    // the activations: bf16, token t's 8 features of state j at t * x_row + j / 2 * x_pair + j % 2 * 16 bytes, x_turn bytes on per turn
    const uint16_t *x;
    uint64_t x_row;
    uint32_t x_pair, x_turn;
    float *y;              // [tokens][out_features], holds the bias (or zero) on entry unless whole_rows
    uint32_t *status;
    uint64_t n;
    uint32_t n_chunks;
    Divisor row_turns;     // in_features / 128
    uint32_t out_features;
    uint32_t tokens;
    Divisor stride;        // chunks between neighbouring columns of a group
    uint32_t columns;      // ... which has this many (at most 16 or 32, as the form has; as many as their words fit the window)
    uint32_t n_groups;
    uint32_t split;        // 1: two lanes walk a state's two halves from the entry points
    // How sums leave: whole, with the bias, where rows do not pass the end of a chunk; or as the sum of one piece (the part of a
    // row inside a chunk or half of one) to pieces[(unit + row) * piece_tokens + token], unit the number of the chunk or half;
    // or they are added to y, which holds the bias or zero on entry.
    uint32_t whole_rows;
    const float *bias;
    float *pieces;
    uint32_t piece_tokens;
};

// Several weights applied to the same kind of input in one launch (the q, k and v projections of an
// attention block, say): workgroups [wg_end[i-1], wg_end[i]) belong to weight i.  Weights too small to
// fill the chip on their own overlap with the others.
constexpr uint32_t kLinBatchMax = 4;
struct LinearBatchArgs {
    uint32_t wg_end[kLinBatchMax];  // (behind the last weight: UINT32_MAX)
    uint32_t count;                 // (for the host)
    LinearArgs t[kLinBatchMax];
};
struct LinearInitArgs {
    float *y[kLinBatchMax];
    const float *bias[kLinBatchMax];
    uint32_t out_features[kLinBatchMax];
    uint32_t wg_end[kLinBatchMax];  // workgroups that set y up (none where the sums are stored whole) ...
    uint32_t set_up;                // ... of all weights
    const uint4 *x;                 // the activations, in pieces of 8 features, and where they go (nullptr: they stay)
    uint4 *scratch;
    uint32_t row_pieces;            // of a token
    uint32_t tokens;
};

// In front of the kernel below, where there is something to do: y[t][o] = bias[o] (or 0), the accumulation target, four tokens of
// 256 outputs to a workgroup; and the activations in the order in which waves read them.
//
// A wave's operand is 32 or 64 bytes of each of 32 or 16 rows of x: as x lies, a request touches as many cache lines, and a CU
// of 16 waves is busy with these requests for longer than with the symbols (64 tokens, x as it lies / every request 1 KB in
// a piece: 4096 x 14336, k = 3, 65 / 47 us, 14336 x 4096 60 / 40, 4096 x 4096 27 / 18).  So, given the room, the tokens of 16
// neighbouring features are laid side by side, 32 bytes each (tile by tile of 64 tokens): whatever 16 or 32 of them a wave
// asks for are then neighbours.
constexpr uint32_t kLinInitThreads = 256, kLinInitTokens = 4;
__host__ __device__ constexpr uint32_t padded_tokens(uint32_t tokens) { return (tokens + 3) / 4 * 4; }  // 128 bytes
__global__ void linear_init_kernel(const LinearInitArgs b)
{
    // which weight's y this workgroup sets up (a grid of outputs x tokens x weights, where this is known without a look at the ends
    // and without a division, gave nothing: 300 x 1152, 9 tokens, 17.7 us either way)
    float *y = nullptr;
    const float *bias = nullptr;
    uint32_t out_features = 1, first = 0;
#pragma unroll
    for (uint32_t i = 0; i < kLinBatchMax; ++i) {
        const uint32_t before = i ? b.wg_end[i - 1] : 0u;
        if (blockIdx.x >= before && blockIdx.x < b.wg_end[i]) {
            y = b.y[i];
            bias = b.bias[i];
            out_features = b.out_features[i];
            first = before;
        }
    }
    if (!y) {  // (behind them all)
        const uint64_t i = static_cast<uint64_t>(blockIdx.x - b.set_up) * kLinInitThreads + threadIdx.x;
        if (i >= static_cast<uint64_t>(b.row_pieces) * b.tokens)
            return;
        // (neighbouring threads take neighbouring places: pieces 2p and 2p + 1 of one token behind those of the token before)
        const uint64_t tile_pieces = static_cast<uint64_t>(b.row_pieces) * kLinMaxTokens;
        const uint32_t tile = b.tokens > kLinMaxTokens ? static_cast<uint32_t>(i / tile_pieces) : 0u;
        const uint64_t in_tile = i - tile * tile_pieces;
        const uint32_t t0 = tile * kLinMaxTokens, tokens = min(b.tokens - t0, kLinMaxTokens), half = i & 1u;
        const uint32_t pair = static_cast<uint32_t>((in_tile >> 1) / tokens), token = static_cast<uint32_t>((in_tile >> 1) - static_cast<uint64_t>(pair) * tokens);
        uint4 *to = b.scratch + tile * tile_pieces;
        to[(static_cast<uint64_t>(pair) * padded_tokens(tokens) + token) * 2 + half] =
            b.x[static_cast<uint64_t>(t0 + token) * b.row_pieces + pair * 2 + half];
        return;
    }
    const uint32_t across = (out_features + kLinInitThreads - 1) / kLinInitThreads;
    const uint32_t o = (blockIdx.x - first) % across * kLinInitThreads + threadIdx.x;
    const uint32_t t0 = (blockIdx.x - first) / across * kLinInitTokens;
    if (o >= out_features)
        return;
    const float v = bias ? bias[o] : 0.0f;
#pragma unroll
    for (uint32_t t = t0; t < t0 + kLinInitTokens; ++t)
        if (t < b.tokens)
            y[static_cast<uint64_t>(t) * out_features + o] = v;
}

// Behind the kernel below, where the sums of pieces are added up: y[t][r] = bias[r] + the pieces of row r.  A workgroup takes 64
// rows; a piece's tokens are read 16 bytes per lane and turned in LDS, so that y is written a row of outputs at a time.
constexpr uint32_t kLinSumThreads = 256, kLinSumRows = 64;
struct LinearSumArgs {
    const float *pieces[kLinBatchMax];
    float *y[kLinBatchMax];
    const float *bias[kLinBatchMax];
    uint32_t out_features[kLinBatchMax];
    uint32_t unit_shift[kLinBatchMax];  // log2 of a unit's elements: a chunk, or half of one
    uint32_t wg_end[kLinBatchMax];
    uint64_t in_features;
    uint32_t tokens, piece_tokens, count;
};
__global__ __launch_bounds__(kLinSumThreads) void linear_sum_kernel(const LinearSumArgs b)
{
    __shared__ float sums[kLinSumRows][kLinMaxTokens + 1];
    uint32_t i = 0, first = 0;
    while (i + 1 < b.count && blockIdx.x >= b.wg_end[i]) {
        first = b.wg_end[i];
        ++i;
    }
    const uint32_t row0 = (blockIdx.x - first) * kLinSumRows, out_features = b.out_features[i], shift = b.unit_shift[i];
    const uint32_t quads = b.piece_tokens / 4;
    for (uint32_t n = threadIdx.x; n < kLinSumRows * quads; n += kLinSumThreads) {
        const uint32_t r = n / quads, t = n % quads * 4;
        const uint64_t row = row0 + r;
        if (row >= out_features)
            break;
        const uint64_t last = ((row + 1) * b.in_features - 1) >> shift;
        float4 sum = make_float4(0, 0, 0, 0);
        for (uint64_t unit = row * b.in_features >> shift; unit <= last; ++unit) {
            const float4 v = *reinterpret_cast<const float4 *>(b.pieces[i] + (unit + row) * b.piece_tokens + t);
            sum.x += v.x;
            sum.y += v.y;
            sum.z += v.z;
            sum.w += v.w;
        }
        sums[r][t] = sum.x;
        sums[r][t + 1] = sum.y;
        sums[r][t + 2] = sum.z;
        sums[r][t + 3] = sum.w;
    }
    __syncthreads();
    const uint32_t r = threadIdx.x % kLinSumRows;
    if (row0 + r >= out_features)
        return;
    const float bias = b.bias[i] ? b.bias[i][row0 + r] : 0.0f;
    for (uint32_t t = threadIdx.x / kLinSumRows; t < b.tokens; t += kLinSumThreads / kLinSumRows)
        b.y[i][static_cast<uint64_t>(t) * out_features + row0 + r] = sums[r][t] + bias;
}

__device__ __forceinline__ void atomic_add_f32(float *p, float v)
{
    // the hardware float add of the memory system (no compare-and-swap loop); y is ordinary
    // device memory, which is what that instruction requires
    unsafeAtomicAdd(p, v);
}

// LDS beside the slot table and the words, for sums on their way out, and what is left for the words (two workgroups share a CU's
// 160 KB).
constexpr uint32_t kLinAreaBytes = 9 * 1024;
constexpr uint32_t kLinStageBytes = 80 * 1024 - kM * 4 - kSteps * 4 - kLinAreaBytes;
static_assert(kLinStageBytes % 32 == 0, "the windows of two groups begin on 16 bytes");

// The arguments that the sums need on their way out, in registers from the beginning on: fetched where they are used, one after
// the other, they are 0.6 us at the end of a launch.
struct LinearOut {
    // (pointers that an asm statement has passed on have to say themselves that they are global: a flat store makes every wait
    // for a load one for all)
    typedef __attribute__((address_space(1))) float global_float_t;
    global_float_t *y, *pieces;
    const global_float_t *bias;
    uint32_t out_features, tokens, whole_rows, piece_tokens;
    __device__ __forceinline__ explicit LinearOut(const LinearArgs &a)
        : y((global_float_t *)a.y), pieces((global_float_t *)a.pieces), bias((const global_float_t *)a.bias), out_features(a.out_features), tokens(a.tokens), whole_rows(a.whole_rows),
          piece_tokens(a.piece_tokens)
    {
        asm volatile("" : "+s"(y), "+s"(pieces), "+s"(bias), "+s"(out_features), "+s"(tokens), "+s"(whole_rows), "+s"(piece_tokens));
    }
};

// How the sums of a tile of tokens leave.  The waves of a set (16 columns: four; 32: the workgroup's eight) hold partial sums of
// the same rows and tokens, over the input features of their own states.
template <int COLS, int MT>
struct LinearSums {
    typedef LinearTile<COLS> Tile;
    static constexpr uint32_t kWaves = COLS == 16 ? 4 : 8;
    static constexpr uint32_t kAll = MT * Tile::kRegs;  // registers of a wave's sums
    // ... that go through LDS at a time: at the end of a row inside the walk four, at its end, where the words are done with, more
    static constexpr uint32_t kFew = 4, kMany = kAll < 16 ? kAll : 16;
    // Floats between the registers of a wave in LDS: a lane's column and the tokens of four registers are also read tokens first.
    static constexpr uint32_t kApart = COLS == 16 ? 68 : 72;
    static_assert(kLinThreads / 64 * kFew * kApart * sizeof(float) <= kLinAreaBytes, "the area holds a pass of all waves");
    static_assert(kLinThreads / 64 * kMany * kApart * sizeof(float) <= kLinStageBytes, "... and the words' place one of the last");

    // They add them up in LDS, one sum per thread, which leaves from there.  joint: the sums of both sets belong together (whole
    // rows only).  has: this wave's set hands over; the barriers are for the whole workgroup, whose waves all come here.  live:
    // the lane's column has a row to hand over, `row`, in unit `unit`.  The area is free before and after.
    template <uint32_t PASS>
    static __device__ __forceinline__ void add_up(const typename Tile::acc_t (&acc)[MT], const LinearOut &a, float *area,
                                                  uint32_t set, uint32_t place, uint32_t lane, bool joint, bool has, bool live,
                                                  uint32_t row, uint32_t unit)
    {
        // (opaque here, so that no address of this is worked out before the walk and held in registers through it)
        asm volatile("" : "+v"(lane));
        constexpr uint32_t kSet = kWaves * PASS * kApart;
        constexpr uint32_t kTokens = 4 * (64 / COLS);  // of four registers: 16 or 8
        float *own = area + set * kSet;
        const uint32_t waves = joint ? 2 * kWaves : kWaves, first = joint ? set * kWaves + place : place;
        const uint32_t piece = live ? unit + row : ~0u;
#pragma unroll
        for (uint32_t p = 0; p < kAll; p += PASS) {
            // (the first token of four registers is that of the first of them in lane 0)
            const uint32_t t0 = p / Tile::kRegs * COLS + Tile::row(0, static_cast<int>(p % Tile::kRegs));
            if (t0 >= a.tokens)
                break;
            if (has) {
#pragma unroll
                for (uint32_t r = 0; r < PASS; ++r)
                    own[(place * PASS + r) * kApart + lane] = acc[(p + r) / Tile::kRegs][(p + r) % Tile::kRegs];
            }
            lds_barrier();
            if (has && a.pieces) {
                // neighbouring threads take neighbouring tokens of a piece: 256 sums for four registers
                for (uint32_t i = place * 64 + lane; i < PASS * 64; i += kWaves * 64) {
                    const uint32_t r = i / 256 * 4, token = i % kTokens, col = i % 256 / kTokens;
                    const float *from = own + (r + token % 4) * kApart + token / 4 * COLS + col;
                    float total = 0.0f;
#pragma unroll
                    for (uint32_t w = 0; w < kWaves; ++w)
                        total += from[w * PASS * kApart];
                    const uint32_t at = __shfl(piece, static_cast<int>(col));
                    const uint32_t t = (p + r) / Tile::kRegs * COLS + Tile::row(0, static_cast<int>((p + r) % Tile::kRegs)) + token;
                    if (at != ~0u && t < a.tokens)
                        a.pieces[static_cast<uint64_t>(at) * a.piece_tokens + t] = total;
                }
            } else if (has) {
                // ... neighbouring columns of a token
                for (uint32_t r = first; r < PASS; r += waves) {
                    const float *from = (joint ? area : own) + r * kApart + lane;
                    float total = 0.0f;
                    for (uint32_t w = 0; w < waves; ++w)
                        total += from[w * PASS * kApart];
                    const uint32_t t = (p + r) / Tile::kRegs * COLS + Tile::row(lane, static_cast<int>((p + r) % Tile::kRegs));
                    auto *at = a.y + static_cast<uint64_t>(t) * a.out_features + row;
                    if (live && t < a.tokens) {
                        if (a.whole_rows)
                            *at = total + (a.bias ? a.bias[row] : 0.0f);
                        else
                            atomic_add_f32((float *)at, total);
                    }
                }
            }
            lds_barrier();
        }
    }
};

// Where a wave stands in its workgroup.
struct LinearPlace {
    uint32_t set, in_set, lane, j;
    uint32_t unit;           // the chunk, or half of one, of the lane's column
    uint32_t row;            // the row of the weight that it begins in
    uint32_t row_turns;      // turns of a row
    uint32_t row_turn;       // the turn of a row that the walk begins with
    float *area;             // the workgroup's (see LinearSums)
    uint32_t turns_to_end;   // from the walk's beginning to the end of the row, of this set ...
    uint32_t other_to_end;   // ... and of the other one
};

// NORM: the blob is block-wise normalised (Sec. 2.3): the merged words are multiplied by their block's
// coefficient, as in the decoder, before they enter the matrix instruction.
// The partial sums of the last row that the walk touched stay in acc, that row in `row`.  All waves of a workgroup come here
// and take the same turns: they meet at barriers.
template <int KB, int COLS, int MT, bool LONE, bool NORM, bool EAGER, class WordSrc>
__device__ __forceinline__ void linear_walk(const uint32_t *__restrict__ lut, const WordSrc &src, uint32_t lone,
                                            uint32_t &x, uint32_t &wp, const uint8_t *__restrict__ sm,
                                            const LinearArgs &a, const LinearOut &to, const LinearPlace &at, uint64_t base, uint32_t turns,
                                            uint32_t all_turns, typename LinearTile<COLS>::acc_t (&acc)[MT], uint32_t &row)
{
    const uint32_t out_features = to.out_features, tokens = to.tokens, lane = at.lane, j = at.j;
    typedef LinearTile<COLS> Tile;
    // Position in the matrix: the row is the lane's own (its chunk's); the turn of the row is that of the group's first chunk,
    // which all its chunks share -- lanes without a chunk use it too, because every lane supplies activations to A.
    row = at.row;
    // the rows of the activations that this lane supplies to A, state j's 8 features of a turn (clamped: rows past `tokens` are
    // never stored)
    const uint8_t *xrow[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const uint32_t t = mt * COLS + (lane & (COLS - 1));
        xrow[mt] = reinterpret_cast<const uint8_t *>(a.x) + static_cast<uint64_t>(t < tokens ? t : tokens - 1) * a.x_row +
                   (j / 2) * a.x_pair + (j % 2) * (kRun * 2);
    }
    uint32_t next = LONE ? 0u : src.peek(wp);
    // A turn's activations are requested at its beginning and travel while its eight symbols are decoded; its fields a turn ahead.
    // (Activations requested behind the matrix instruction of the turn before, into the registers that it reads: 14336 x 4096, 17
    // tokens, 36.5 us, 35.4 now, 4096 x 4096, 8 tokens, 15.9 / 15.6; whole turns ahead they take registers and places in the queue:
    // 4096 x 14336, 32 tokens, 43 -> 49.  Fields requested with them: 4096 x 4096, 1 token, 16.7 us -> 17.8.)  A lane without turns
    // of its own reads those of the tensor's first chunk; a turn behind the last reads the last again.  The coefficient of
    // normalised weights is requested behind the turn before, and their fields a turn ahead in the walk of 16 columns only (4096 x 14336,
    // k = 3, blocks of 128, 1 token, 47.8 us -> 43.4; but not with two tiles of tokens, nor in the walk of 32 columns, 4096 x
    // 14336, k = 0, blocks of 64, 32 tokens, 56.1 -> 58.7).
    const uint32_t row_turns = at.row_turns;
    constexpr bool EARLY = !NORM || (COLS == 16 && MT != 2);
    const uint64_t first = (turns > 0 ? base : 0u) + j * kRun;
    const uint32_t last = turns > 0 ? turns - 1 : 0u;
    uint64_t fields = 0;
    uint32_t coef = 0;
    bf16x8_t xa[MT];
    uint32_t ahead = at.row_turn;                                // the turn of the row that is requested next ...
    uint64_t ahead_at = static_cast<uint64_t>(ahead) * a.x_turn;  // ... and where its activations are in a token's
    uint32_t x_turn = a.x_turn;
    asm volatile("" : "+s"(x_turn));
    auto request_fields = [&](uint32_t q) { fields = load_fields<KB>(sm, first + min(q, last) * kTurn); };
    auto request_coef = [&](uint32_t q) {
        if constexpr (NORM)
            coef = a.coef[(first + min(q, last) * kTurn) >> a.block_shift];
        if constexpr (!EARLY)
            request_fields(q);
    };
    auto request_x = [&]() {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
            xa[mt] = *reinterpret_cast<const bf16x8_t *>(xrow[mt] + ahead_at);
        const bool wraps = ++ahead == row_turns;
        ahead = wraps ? 0u : ahead;
        ahead_at = wraps ? 0u : ahead_at + x_turn;
    };
    if constexpr (EARLY)
        request_fields(0);
    request_coef(0);

    // The trip counts are the same for every lane of the wave (the matrix instruction needs them all); a lane whose chunk is
    // shorter or absent supplies zeros.  The walk goes from one end of a row of the weight to the next, of either set, the turns
    // between them in a loop of their own: with the end of a row as a branch inside one loop of turns, the compiler moved the
    // whole tile of sums from register to register in every turn, behind a wait for the matrix instruction (4096 x 14336, 1 token,
    // 38.0 -> 36.9 us, 64 tokens 67.9 -> 65.0).
    const bool direct = COLS == 16 && MT == 1 && out_features <= direct_sums(tokens) / tokens && !to.whole_rows && !to.pieces;
    // (sums that leave by themselves meet at no barrier: the other set's ends are nothing to this one)
    uint32_t q = 0, own_end = at.turns_to_end, other_end = direct ? ~0u : at.other_to_end;
    // The fields of the turn behind an end are waited for in front of it.  Behind it, it would be for the acknowledgements of the sums
    // that leave there, too, at every end (300 x 640, 4 tokens, 17.4 us, 16.1 now; 260 x 384, 5 tokens, 18.5 / 16.7; 2000 x 640, 6
    // tokens, 19.2 / 18.5; 57344 x 1024, 16 tokens, 36.0 / 35.2).  The compiler waits behind it if there is a way there without.
    if constexpr (EARLY)
        settle(fields);
    for (;;) {
        const uint32_t next_end = min(all_turns, min(own_end, other_end));
        for (; q < next_end; ++q) {
            request_x();
            const uint64_t f = fields;
            if constexpr (EARLY)
                request_fields(q + 1);

            union {
                uint32_t u[4];
                bf16x8_t v;
            } b;
            b.u[0] = b.u[1] = b.u[2] = b.u[3] = 0;
            if (q < turns) {
                uint32_t e[8];
#pragma unroll
                for (int t = 0; t < 8; ++t)
                    e[t] = LONE ? lone : rans_get<EAGER>(lut, x, wp, next, src);
                b.u[0] = merge_pair<KB>(f, 0, e[0], e[1]);
                b.u[1] = merge_pair<KB>(f, 1, e[2], e[3]);
                b.u[2] = merge_pair<KB>(f, 2, e[4], e[5]);
                b.u[3] = merge_pair<KB>(f, 3, e[6], e[7]);
                if constexpr (NORM) {
                    const float c = coefficient(coef & 0x7Fu);
#pragma unroll
                    for (int p = 0; p < 4; ++p)
                        b.u[p] = denormalise_pair(b.u[p], c);
                }
            }
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                acc[mt] = Tile::mma(xa[mt], b.v, acc[mt]);
            request_coef(q + 1);
        }
        if constexpr (EARLY)
            settle(fields);
        if (q == all_turns)
            break;
        // the end of a row of the weight inside the walk: its sums leave for y
        const bool ends = q == own_end;
        const bool col_live = q - 1 < turns && row < out_features;
        if (direct) {
            if (ends && col_live)
#pragma unroll
                for (int r = 0; r < Tile::kRegs; ++r)
                    if (Tile::row(lane, r) < tokens)
                        atomic_add_f32((float *)(to.y + static_cast<uint64_t>(Tile::row(lane, r)) * out_features + row), acc[0][r]);
        } else
            LinearSums<COLS, MT>::template add_up<LinearSums<COLS, MT>::kFew>(acc, to, at.area, at.set, at.in_set, lane, false, ends, col_live, row, at.unit);
        if (ends) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int r = 0; r < Tile::kRegs; ++r)
                    acc[mt][r] = 0.0f;
            ++row;
            own_end += row_turns;
        }
        if (q == other_end)
            other_end += row_turns;
    }
}

// READ: every weight of the launch is walked whole and holds its slot table (with the choice of both left to run time
// 4096 x 14336, 1 token, took 36.4 us, 35.7 now, and 8192 x 8192 36.7, 35.9 now).
// EAGER: the step of the walk without a branch (see rans_get).
template <int KB, int COLS, int MT, bool NORM, bool READ, bool EAGER>
__device__ __forceinline__ void linear_workgroup(const LinearArgs &a, uint32_t wg, uint32_t *__restrict__ lut,
                                                 uint32_t *__restrict__ steps, uint8_t *__restrict__ stage,
                                                 float *__restrict__ area)
{
    const LinearOut to(a);
    constexpr uint32_t kPerWave = 64 / COLS;                         // states of a chunk per wave: 4 or 2
    constexpr uint32_t kSetWaves = kStates / kPerWave;               // 4 or 8
    const uint32_t split = COLS == 16 && !READ ? a.split : 0u;                // two sets for the halves of a group's states
    const uint32_t waves_per_group = kSetWaves << split;             // 4 (8 with entry points), or 8
    const uint32_t groups_per_wg = kLinThreads / 64 / waves_per_group;
    const uint32_t group_window = kLinStageBytes / groups_per_wg;       // LDS window of one group's word runs
    const uint32_t cols_per_wave = COLS / waves_per_group;           // columns a wave copies
    const uint32_t tid = threadIdx.x;
    // (the same for all lanes, and told so: what follows from it stays in scalar registers)
    const uint32_t wave = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(tid >> 6)));
    const uint32_t lane = tid & 63u;
    const uint32_t g = wave / waves_per_group, in_group = wave % waves_per_group;
    const uint32_t part = split ? in_group / kSetWaves : 0u;                // before (0) or behind (1) the entry points
    const uint32_t set = wave / kSetWaves, in_set = wave % kSetWaves;
    const uint32_t col = lane & (COLS - 1);
    const uint32_t j = in_set * kPerWave + lane / COLS;
    // group -> its chunks: `stride` groups interleave inside a block of columns * stride chunks; the first of them
    // (32-bit numbers: chunks and turns.  In 64-bit bytes and elements the three divisions of the beginning took 1.2 us.)
    auto first_chunk = [&](uint32_t group) { return group + a.stride.quotient(group) * (a.columns - 1) * a.stride.by; };
    const uint32_t group = wg * groups_per_wg + g;
    const bool group_live = group < a.n_groups;
    const uint32_t c_of = first_chunk(group) + a.stride.by * col;
    const bool live = group_live && col < a.columns && c_of < a.n_chunks;
    const uint32_t turn0 = part * kMidTurn, all_turns = split ? kMidTurn : kTurns;
    const uint32_t row_turns = a.row_turns.by, row_turn = a.row_turns.rest(first_chunk(group) * kTurns + turn0);
    // (the other set of the workgroup: the other half of this group, or the other group)
    const uint32_t other_turn = groups_per_wg == 1 && !split
                                    ? row_turn
                                    : a.row_turns.rest(first_chunk(split ? group : group ^ 1u) * kTurns + (split ? kMidTurn - turn0 : 0u));
    const uint32_t c = live ? c_of : 0u;
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
    const LinearPlace at = {set, in_set, lane, j, split ? 2 * c + part : c, a.row_turns.quotient(c * kTurns + turn0), row_turns,
                            row_turn, area, row_turns - row_turn, row_turns - other_turn};
    uint32_t wp = 0, wp_begin = 0;
    if (lone < 256) {
        linear_walk<KB, COLS, MT, true, NORM, EAGER>(lut, NoWords{}, lone, x, wp, a.sm, a, to, at, from_elem, turns, all_turns, acc,
                                                     row);
    } else if (staged) {
        wp = wp_begin = g * group_window + place + static_cast<uint32_t>(run_byte - aligned0);
        linear_walk<KB, COLS, MT, false, NORM, EAGER>(lut, LdsWords{stage}, 0u, x, wp, a.sm, a, to, at, from_elem, turns, all_turns,
                                                      acc, row);
    } else {
        const GlobalWords direct{reinterpret_cast<const uint8_t *>(a.words) + run_byte};
        linear_walk<KB, COLS, MT, false, NORM, false>(lut, direct, 0u, x, wp, a.sm, a, to, at, from_elem, turns, all_turns, acc, row);
    }
    if (live && (x != x_end || wp - wp_begin != 2 * words_here))
        atomicOr(a.status, 1u);

    // ---- what is left of the last row: the row's sum if rows do not pass the end of a chunk, or of its half (the two halves of a
    // chunk that is one row end in the same one)
    const uint32_t chunk_turns = m / kTurn;
    const bool row_live = live && chunk_turns > turn0 && row < to.out_features;
    lds_barrier();  // (the sums take the words' place)
    LinearSums<COLS, MT>::template add_up<LinearSums<COLS, MT>::kMany>(acc, to, reinterpret_cast<float *>(stage), set, in_set, lane,
                                                                       split && row_turns == kTurns, true, row_live, row, at.unit);
}

// (Two workgroups of 8 waves share a CU if a lane has at most 128 registers; with the 138 the compiler took
// for 64 tokens it held one.)
template <int KB, int COLS, int MT, bool NORM, bool READ, bool EAGER>
__global__ __launch_bounds__(kLinThreads, 4) void linear_batch_kernel(const LinearBatchArgs b)
{
    __shared__ __align__(16) struct {
        uint8_t stage[kLinStageBytes];  // first: a direct copy's LDS address has 16 bits
        uint32_t lut[kM];
        float area[kLinAreaBytes / 4];
        uint32_t steps[READ ? 4 : kSteps];
    } lds;
    // (the first weight's, with the ends, which lie in its first line; workgroups of the others wait for theirs as they come to them)
    fetch_arguments(b.t[0]);
    uint32_t i = 0, first = 0;
#pragma unroll
    for (uint32_t n = 0; n + 1 < kLinBatchMax; ++n) {  // (behind the last weight: no workgroup has these numbers)
        if (blockIdx.x >= b.wg_end[n]) {
            i = n + 1;
            first = b.wg_end[n];
        }
    }
    linear_workgroup<KB, COLS, MT, NORM, READ, EAGER>(b.t[i], blockIdx.x - first, lds.lut, lds.steps, lds.stage, lds.area);
}

}  // namespace nz
