// Dense product of the quantiser on the matrix cores:  C[r][c] = sum_k A[k][r] * B[k][c]  (not public).
//
// A is [K][R] with pitch lda, B is [K][C] with pitch ldb, binary32, "k-major" (both pitches and R, C multiples of 4,
// all pointers 16-byte aligned).  What happens to the finished tile is the mode:
//   kQuadForm   part[tile column][r] = sum over the tile's columns c of C'[r][c] * E[c][r], where C' takes B[k][c] with the
//               weight 1 for k < c, 1/2 for k = c and 0 for k > c: half of the quadratic form of a symmetric B if
//               E = A.  The k range of a tile stops at its last column.  (out is [tile column][ldo], E has pitch ldo)
//   kQuadFormSplit   kQuadForm with A split beforehand (see ProductArgs)
//   kAddTwiceSymmetric   out[r][c] += 2 C[r][c], B = A: only the tiles on and above the diagonal are computed and each
//               element is added to both out[r][c] and out[c][r]
//   kSubtract   out[r][c] -= C[r][c];   kSubtractLower   the same for the tiles on and below the diagonal only
//   kStore      out[r][c] = C[r][c]; with triangular_b B[k][c] = 0 for k > c
//   kStoreNegated   out[r][c] = -C[r][c], A[k][r] = 0 for k < r
//
// Arithmetic.  The binary32 matrix instruction (v_mfma_f32_32x32x2_f32) runs at 1/16 of the rate of the binary16 ones
// (v_mfma_f32_16x16x32_f16).  So every operand value x is split, after scaling by a power of two s that belongs to its
// row or column of the product, into two binary16 numbers, hi = rne16(s x) and lo = rne16(s x - hi), and the product is
// lo hi' + hi lo' + hi hi', three instructions that accumulate in binary32.  Where |s x| >= 1/4, |s x - hi - lo| is at most
// 2^-23 |s x| (three significands in four are exact); below that it is at most 2^-25, half the smallest step of a binary16
// number.  The dropped lo lo' is at most 2^-22 of the term.  The accumulator is rounded three times per 16 values of k
// (measured: the instruction over 32 values rounds twice) instead of 16 times, which outweighs that: 2-norm error of
// 2 X^T X with standard normal X against binary64, binary32 instruction / this, 16 samples 7.4e-8 / 8.4e-8, 24 samples 8.9e-8 /
// 8.6e-8, 256 samples 2.8e-7 / 1.8e-7, 2048 samples 6.6e-7 / 4.1e-7.  Up to 20 values of k the binary32 instruction is used.
// The scales: binary16 reaches from 2^-24 to 2^16, and values far below the largest of their row or column should keep their
// bits, because what they are multiplied by may be as much larger.  So s is chosen from the largest magnitude in the first 32
// values of the row or column, which it puts at 2^8..2^9: full precision down to 2^-10 of it, and later values may be at
// least 117 times larger.  Where more is known, more is used:
//   quadratic forms   d is bounded by its row's range, and the values of a positive semidefinite B by its diagonal, which
//                 together with the largest of all puts them at most at 2^15;
//   triangular operands, zero in the first 32 values   the diagonal;
//   errors of the GPTQ pass   they have been divided by the diagonal of U, whose smallest value in reach is known (ProductArgs::least).
//                 They and the rows of U grow more on the way than data do and start at 2^5, which leaves a factor of at least 937;
//   the factor    its matrix is scaled so that all channels are of one size (bcq_quant.hip).
// The largest magnitude of all values is tracked on the way; a tile with a guess that was too low, or more than 2^6 too high, is
// computed once more with s from the true maximum, at 2^14.  (Scales that change on the way, by a flag in LDS per step that
// all waves look at, cost 11 % of a large Hessian and 24 % of a small one.)
// Inverse-Hessian factor, error per column of U against binary64, binary32 instruction / this, four channels 2^10 (2^12) times as
// loud at the start of every block of 128 channels: 2.0e-7 / 1.7e-7 (5.1e-7 / 4.3e-7); before its channels were scaled, and with a
// first guess at 2^4, 9e-7 (1.4e-5).  Search with four of 7168 channels 2^13 times as loud: 59.0 ms when the tiles of H had to be
// computed twice, now 31 as with any other.
// A value that is not finite makes every sum it enters not finite.
//
// Work split.  A workgroup of four waves owns a 128 x 128 tile of C, a wave a 64 x 64 quarter as 4 x 4 accumulators of
// 16 x 16; a step takes 32 values of k.  Wave w brings the eight rows 8 w .. 8 w + 7 of the step, lane l the columns 2 l
// and 2 l + 1 of both operands (eight 8-byte loads each, the rows of a wave contiguous), splits them in registers (2.5
// vector instructions per value) and stores one 16-byte octet of k values per column and half: the layout in which the
// matrix instruction takes its operands.  Two stages in LDS (64 KB) with one barrier per step; two workgroups per
// compute unit, so that one's loads and splits run under the other's matrix instructions.  The loop has no branch around
// its loads (buffer descriptors end at the k range), so that the compiler interleaves the vector instructions with the
// matrix instructions: with branches the same loop was 25 % slower.
// What bounds it: 110 vector instructions (440 clocks) and 48 matrix instructions (768 clocks) per wave and step, two waves per
// SIMD.  Counters: 2 X^T X over 14336 samples of 7168 channels matrix pipe busy 36 % of the time, vector ALU 21 %, LDS 36 %
// (a third of it bank conflicts: not the reads, so the 16-byte stores), waves at a wait 42 % of their cycles; the quadratic form
// with A split beforehand 47 %, 16 %, 32 % (a quarter conflicts), 36 %.  Measured (binary32 instruction before / now): quadratic form of a 7168 x
// 7168 layer 3.32 / 1.38 ms per candidate, 1.19 with A split beforehand (kQuadFormSplit: 930 TFLOP/s of binary16 products; a
// large library product of that type reaches 1230 on this card), 2 X^T X over 4 x 2048 samples of 7168 channels 7.17 / 1.80 ms.
// An octet of column c sits at position c ^ ((c >> 4) & 1): the 16 lanes that a 16-byte LDS read serves together then
// touch 16 different 16-byte columns.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "bcq_device.h"

namespace bcq {

typedef _Float16 prod_f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 prod_f16x2 __attribute__((ext_vector_type(2)));
typedef unsigned prod_u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned prod_u32x2 __attribute__((ext_vector_type(2)));
typedef float prod_f32x2 __attribute__((ext_vector_type(2)));
typedef float prod_f32x4 __attribute__((ext_vector_type(4)));

#define PROD_INLINE __attribute__((always_inline))

enum ProductMode { kQuadForm = 0, kSubtract = 1, kAddTwiceSymmetric = 2, kStore = 3, kStoreNegated = 4, kSubtractLower = 5, kQuadFormSplit = 6 };

constexpr int kProdTile = 128, kProdStep = 32, kProdBlock = 4;  // tile edge, k values per step, tiles per block edge
constexpr int kProdTarget = 8;                                  // a first guess puts its magnitude at 2^8 .. 2^9
constexpr int kProdFew = 20;                                    // up to so many values of k in binary32 instructions
constexpr float kProdMost = 60000.0f, kProdLeast = 4.0f;        // where scaled maxima have to lie, see above

struct ProductArgs {
    const float *A, *B, *E;
    float *out;
    int lda, R, ldb, C, K, ldo;
    int triangular_b;  // kStore: B[k][c] = 0 for k > c
    const uint16_t *split;  // kQuadFormSplit: A in two halves, [hi, lo][k / 8][row (pitch ldo)][8 values of k]; K a multiple of 8
    size_t split_plane;     // values per half
    const int *split_shift; // quadratic forms: exponent of each row's scale
    const float *diag_max;  // quadratic forms: largest value on B's diagonal
    const float *least;     // kSubtract, errors of the GPTQ pass: smallest divisor of the 128 rows of block k / 128 of B and of its
                            // first 32, at least[2 (k / 128)], for up to four blocks; or null
    // several products of one shape in a launch (blockIdx.y): operands and result of product y lie y * stride floats on; the
    // last one may have fewer columns, columns_end - y * columns_step of them, and with k_is_columns as many values of k
    size_t stride;
    int columns_end, columns_step, k_is_columns;
    const int *rows;  // kQuadFormSplit: number of rows that are there, in device memory, or null: R
};

// Number of workgroups, and the tile of one.  Tiles are taken block by block of 4 x 4 so that the workgroups that share an L2 at a
// time share their operand panels (workgroup numbers go round the eight XCDs).
// Where all tiles cost the same (the symmetric sum, on and above the diagonal, and the subtractions) they are numbered block row by
// block row, only those that exist, and each XCD takes an eighth of the numbers, from their end: by whole blocks the XCD with the most
// tiles had 9 % more than its share at 7168 channels.  Up to eight tiles are one XCD's, as they share the lines at their edges.  us, whole
// blocks / numbers / numbers from their end, H += 2 X^T X: 7168 channels, 2048 samples 436 / 421 / 424, 256 samples 105 / 108 / 107; 4096
// channels 204 / 192 / 190 and 49.7 / 54.1 / 50.4, one sample 29.8 / 32.6 / 28.9; 132 channels, one sample 9.5 / 10.4 / (one XCD) 9.7.  The factor
// and the GPTQ pass take the same time with all three.  Otherwise each XCD takes every eighth block, for the quadratic
// forms and the products with a triangular right operand column by column from the last one, whose columns have the longest k range.
// Several products of a launch (kStore, kStoreNegated) go on where the one before ended, after `before` blocks: starting each at the first XCD left all
// blocks of small products to it (7168 channels, us: 14 pairs of 256 channels 38 + 32 -> 20 + 19, 7 of 512 channels 64 + 50 -> 24 + 25, the longest columns of
// 4096 first 212 -> 164).  In these two modes every other eight blocks go to the XCDs in reverse, so that none has all the longer ones of a triangular operand.
template <int MODE>
constexpr bool kProdEven = MODE == kAddTwiceSymmetric || MODE == kSubtract || MODE == kSubtractLower;

template <int MODE>
static inline int product_groups(int R, int C)
{
    const int ntr = (R + kProdTile - 1) / kProdTile, ntc = (C + kProdTile - 1) / kProdTile;
    const long long tiles = MODE == kSubtract ? (long long)ntr * ntc : (long long)ntr * (ntr + 1) / 2;
    const int br = (ntr + kProdBlock - 1) / kProdBlock, bc = (ntc + kProdBlock - 1) / kProdBlock;
    return kProdEven<MODE> ? (tiles <= 8 ? 64 : (int)((tiles + 7) / 8 * 8)) : (br * bc + 7) / 8 * 8 * kProdBlock * kProdBlock;
}

template <int MODE>
__device__ __forceinline__ bool product_tile(int wg, int wgs, int R, int C, int before, int *tile_row, int *tile_col)
{
    const int ntr = (R + kProdTile - 1) / kProdTile, ntc = (C + kProdTile - 1) / kProdTile;
    const int xcd = wg & 7, j = wg >> 3;
    if constexpr (kProdEven<MODE>) {
        constexpr bool kTriangle = MODE != kSubtract;
        int t = xcd * (wgs >> 3) + (wgs >> 3) - 1 - j, b_row = 0, rows, first;
        for (;; ++b_row) {  // the block row, its first column and its number of tiles
            if (b_row * kProdBlock >= ntr) return false;
            rows = ntr - b_row * kProdBlock < kProdBlock ? ntr - b_row * kProdBlock : kProdBlock;
            first = kTriangle ? b_row * kProdBlock : 0;
            const int count = rows * (ntc - first) - (kTriangle ? rows * (rows - 1) / 2 : 0);
            if (t < count) break;
            t -= count;
        }
        int r, c;
        if (kTriangle && t < rows * (rows + 1) / 2) {  // its block on the diagonal
            for (r = 0; t >= rows - r; ++r) t -= rows - r;
            c = first + r + t;
        } else {
            if (kTriangle) {
                t -= rows * (rows + 1) / 2;
                first += rows;
            }
            const int block = t / (rows * kProdBlock), width = ntc - first - block * kProdBlock;
            t -= block * rows * kProdBlock;
            const int cols = width < kProdBlock ? width : kProdBlock;
            r = t / cols;
            c = first + block * kProdBlock + t % cols;
        }
        r += b_row * kProdBlock;
        *tile_row = MODE == kSubtractLower ? c : r;
        *tile_col = MODE == kSubtractLower ? r : c;
        return true;
    } else {
        const int br = (ntr + kProdBlock - 1) / kProdBlock, bc = (ntc + kProdBlock - 1) / kProdBlock;
        const int t = j & (kProdBlock * kProdBlock - 1), round = j / (kProdBlock * kProdBlock), at = (xcd - before) & 7;
        constexpr bool kTurns = MODE == kStore || MODE == kStoreNegated;
        const int s = round * 8 + (kTurns && (round & 1) ? 7 - at : at);
        if (s >= br * bc) return false;
        const bool by_column = MODE == kQuadForm || MODE == kQuadFormSplit || MODE == kStore;
        const int b_row = by_column ? s % br : s / bc, b_col = by_column ? bc - 1 - s / br : s % bc;
        *tile_row = b_row * kProdBlock + t / kProdBlock;
        *tile_col = b_col * kProdBlock + t % kProdBlock;
        return *tile_row < ntr && *tile_col < ntc;
    }
}

// Exponent of the power of two that puts a magnitude (as float bits) at 2^target .. 2^(target + 1), kept to those a
// normal binary32 number can hold.
__device__ __forceinline__ int product_shift(unsigned magnitude, int target)
{
    const int e = target - ((int)(magnitude >> 23) - 127);
    return e < -126 ? -126 : (e > 126 ? 126 : e);
}

// LDS of a workgroup
typedef uint8_t ProductStage[2][4][kProdTile * 16];  // [hi, lo][octet][column]
typedef unsigned ProductLargest[2][kProdTile];
typedef int ProductShift[2][kProdTile];
struct ProductShared {
    ProductStage stage_a0, stage_a1, stage_b[2];
    ProductLargest largest;
    unsigned largest_of_tile[2];
    ProductShift shift;
};

// Tile of workgroup wg of wgs.  stage_a0 .. stage_b: the two stages of both operands; largest: largest magnitude per row of A's
// tile, column of B's tile (float bits); shift: exponents of the scales.
template <int MODE>
__device__ __forceinline__ void product_tile_of(ProductArgs p, int wg, int wgs, ProductStage &stage_a0, ProductStage &stage_a1,
                                                ProductStage (&stage_b)[2], ProductLargest &largest, unsigned (&largest_of_tile)[2],
                                                ProductShift &shift)
{
    constexpr bool kQuad = MODE == kQuadForm || MODE == kQuadFormSplit, kSplitA = MODE == kQuadFormSplit;
    constexpr int kFirst = kSplitA ? 1 : 0;  // first operand that comes in binary32
    constexpr int kGuess = kQuad ? 1 : 0;    // first operand whose scales are guessed
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lo = lane & 15, hi = lane >> 4, wr = wave >> 1, wc = wave & 1;
    int before = 0;  // blocks of the launch's products before this one (only the last one may have fewer columns)
    if (MODE == kStore || MODE == kStoreNegated) {
        constexpr int kEdge = kProdTile * kProdBlock;
        before = (int)blockIdx.y * ((p.R + kEdge - 1) / kEdge) * ((p.C + kEdge - 1) / kEdge);
        p.A += blockIdx.y * p.stride;
        p.B += blockIdx.y * p.stride;
        p.out += blockIdx.y * p.stride;
        const int left = p.columns_end - (int)blockIdx.y * p.columns_step;
        if (left < p.C) p.C = left;
        if (p.k_is_columns) p.K = p.C;
    }
    int tile_row, tile_col;
    if (!product_tile<MODE>(wg, wgs, p.R, p.C, before, &tile_row, &tile_col)) return;
    const int r0 = tile_row * kProdTile, c0 = tile_col * kProdTile;
    if (kSplitA && p.rows && r0 >= *p.rows) return;

    // k range of the tile: what a triangular operand leaves
    int k_begin = 0, k_end = p.K;
    if (kQuad && k_end > c0 + kProdTile) k_end = c0 + kProdTile;
    if (MODE == kStore && p.triangular_b && k_end > c0 + kProdTile) k_end = c0 + kProdTile;
    if (MODE == kStoreNegated) k_begin = r0;
    const int steps = (k_end - k_begin + kProdStep - 1) / kProdStep;

    // Rows k .. k + 7 of an operand's panel as a buffer: reads beyond the k range come back as zeros without touching
    // memory, so the loads need no branch.  Columns beyond the operand read the row that follows (inside the buffer, whose
    // end is the last valid value of the last row) and only reach results that are dropped.
    const float *const panel[2] = {p.A + r0, p.B + c0};
    const int pitch[2] = {p.lda, p.ldb}, width[2] = {p.R - r0, p.C - c0};
    prod_u32x2 raw[2][8];
    auto load = [&](int step) PROD_INLINE {
        const int k = k_begin + step * kProdStep + 8 * wave;
        const int rows = k_end - k < 0 ? 0 : (k_end - k < 8 ? k_end - k : 8);
#pragma unroll
        for (int o = kFirst; o < 2; ++o) {
            const unsigned bytes = rows ? 4u * ((unsigned)(rows - 1) * (unsigned)pitch[o] + (unsigned)width[o]) : 0u;
            const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<float *>(panel[o] + (size_t)(rows ? k : k_begin) * pitch[o]), 0, (int)bytes, kRawBufferFlags);
#pragma unroll
            for (int j = 0; j < 8; ++j)
                raw[o][j] = __builtin_amdgcn_raw_buffer_load_b64(rsrc, 8 * lane, __builtin_amdgcn_readfirstlane(4 * j * pitch[o]), 0);
        }
    };
    auto weigh = [&](int step) PROD_INLINE {  // kQuadForm: B on and beyond its diagonal
        const int k0 = k_begin + step * kProdStep + 8 * wave;
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int c = c0 + 2 * lane + e;
                const float v = __uint_as_float(raw[1][j][e]);
                raw[1][j][e] = __float_as_uint(k0 + j < c ? v : (k0 + j == c ? 0.5f * v : 0.0f));
            }
    };
    float top[2][2] = {{0.f, 0.f}, {0.f, 0.f}};  // largest magnitudes seen by this lane
    auto track = [&]() PROD_INLINE {
#pragma unroll
        for (int o = kGuess; o < 2; ++o)
#pragma unroll
            for (int j = 0; j < 8; ++j)
#pragma unroll
                for (int e = 0; e < 2; ++e) top[o][e] = fmaxf(top[o][e], fabsf(__uint_as_float(raw[o][j][e])));
    };
    auto publish = [&]() PROD_INLINE {  // the lanes' maxima into `largest`
#pragma unroll
        for (int o = kGuess; o < 2; ++o)
#pragma unroll
            for (int e = 0; e < 2; ++e) atomicMax(&largest[o][2 * lane + e], __float_as_uint(top[o][e]));
    };
    float s[2][2];
    const int at = (2 * lane) ^ ((lane >> 3) & 1);  // position of the lane's first column; the second one's is at ^ 1
    auto split_store = [&](auto buf) PROD_INLINE {
        const int b = buf;
#pragma unroll
        for (int o = kFirst; o < 2; ++o)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                prod_u32x4 h, l;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float v0 = __uint_as_float(raw[o][2 * j][e]), v1 = __uint_as_float(raw[o][2 * j + 1][e]);
                    unsigned pair = __builtin_bit_cast(unsigned, prod_f16x2{(_Float16)(v0 * s[o][e]), (_Float16)(v1 * s[o][e])});
                    asm("" : "+v"(pair));  // one packed conversion serves both uses
                    h[j] = pair;
                    const prod_f16x2 hp = __builtin_bit_cast(prod_f16x2, pair);
                    l[j] = __builtin_bit_cast(unsigned, prod_f16x2{(_Float16)fmaf(v0, s[o][e], -(float)hp[0]),
                                                                  (_Float16)fmaf(v1, s[o][e], -(float)hp[1])});
                }
                auto &st = o ? stage_b[b] : (b ? stage_a1 : stage_a0);
                *reinterpret_cast<prod_u32x4 *>(&st[0][wave][(at ^ e) * 16]) = h;
                *reinterpret_cast<prod_u32x4 *>(&st[1][wave][(at ^ e) * 16]) = l;
            }
    };

    prod_f32x4 acc[4][4];
    auto clear = [&]() PROD_INLINE {
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b) acc[a][b] = prod_f32x4{0.f, 0.f, 0.f, 0.f};
    };
    // kQuadFormSplit: A's halves are in the operand layout already and are copied by buffer loads with an LDS destination;
    // wave w brings the octets 2 (w % 2) and 2 (w % 2) + 1 of half w / 2.
    auto copy_a = [&](auto buf, int step) PROD_INLINE {
        const int b = buf;
        auto &st = b ? stage_a1 : stage_a0;
        const int rows = width[0] < kProdTile ? width[0] : kProdTile, half = wave >> 1;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int octet = 2 * (wave & 1) + q, k8 = 4 * step + octet;
            const bool in = 8 * k8 < k_end;
            const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<uint16_t *>(p.split + half * p.split_plane + ((size_t)(in ? k8 : 0) * p.ldo + r0) * 8), 0,
                in ? 16 * rows : 0, kRawBufferFlags);
#pragma unroll
            for (int x = 0; x < 2; ++x)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(
                    rsrc, (__attribute__((address_space(3))) void *)&st[half][octet][64 * x * 16], 16,
                    16 * (64 * x + (lane ^ ((lane >> 4) & 1))), 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);  // (the waits count the loads that follow)
    };
    constexpr int kLoads = 8 * (2 - kFirst);  // per wave and step
    auto barrier = [&]() PROD_INLINE {
        if (kSplitA) {
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(kLoads) : "memory");
            __builtin_amdgcn_sched_barrier(0);
        } else {
            __syncthreads();
        }
    };
    auto multiply = [&](auto buf) PROD_INLINE {
        const int bf = buf;
        auto &sa = bf ? stage_a1 : stage_a0;
        auto &sb = stage_b[bf];
        prod_f16x8 a[2][4], b[2][4];  // [hi, lo][tile]
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                a[x][t] = *reinterpret_cast<const prod_f16x8 *>(&sa[x][hi][(wr * 64 + t * 16 + (lo ^ (t & 1))) * 16]);
                b[x][t] = *reinterpret_cast<const prod_f16x8 *>(&sb[x][hi][(wc * 64 + t * 16 + (lo ^ (t & 1))) * 16]);
            }
#pragma unroll
        for (int x = 0; x < 3; ++x)  // lo hi', hi lo', hi hi'
#pragma unroll
            for (int ta = 0; ta < 4; ++ta)
#pragma unroll
                for (int tb = 0; tb < 4; ++tb)
                    acc[ta][tb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[x == 0][ta], b[x == 1][tb], acc[ta][tb], 0, 0, 0);
    };
    // Up to kProdFew values of k (not a quadratic form): with so few terms the roundings of the operands do not average out, and
    // finding scales takes longer than multiplying.  Such a product is the binary32 instruction's, from one copy of both panels
    // [k][column ^ 16 (k % 4)] in the place of a stage.  512 channels, 8 samples 14.4 -> 12.4 us.
    auto multiply_few = [&]() PROD_INLINE {
        load(0);
        float *const panels[2] = {reinterpret_cast<float *>(&stage_a0[0][0][0]), reinterpret_cast<float *>(&stage_b[0][0][0][0])};
#pragma unroll
        for (int o = 0; o < 2; ++o)
#pragma unroll
            for (int j = 0; j < 8; ++j)
                *reinterpret_cast<prod_u32x2 *>(panels[o] + (8 * wave + j) * kProdTile + ((2 * lane) ^ (16 * (j & 3)))) = raw[o][j];
        shift[tid >> 7][tid & 127] = 0;
        __syncthreads();
        for (int k = 0; k < k_end - k_begin; k += 4) {
            float a[4], b[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                a[t] = panels[0][(k + hi) * kProdTile + ((wr * 64 + t * 16 + lo) ^ (16 * hi))];
                b[t] = panels[1][(k + hi) * kProdTile + ((wc * 64 + t * 16 + lo) ^ (16 * hi))];
            }
#pragma unroll
            for (int ta = 0; ta < 4; ++ta)
#pragma unroll
                for (int tb = 0; tb < 4; ++tb) acc[ta][tb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[ta], b[tb], acc[ta][tb], 0, 0, 0);
        }
    };
    // Steps [from, to): while a step is multiplied, the next one is split and stored to the other stage and the one
    // after it is requested.
    auto one = [&](auto buf, auto other, int step, auto weighed) PROD_INLINE {
        if (kSplitA) copy_a(other, step + 1);
        multiply(buf);
        if (decltype(weighed)::value) weigh(step + 1);
        track();
        split_store(other);
        load(step + 2);
        barrier();  // the other stage is complete, and everyone is done reading this one
    };
    constexpr std::integral_constant<int, 0> even{};
    constexpr std::integral_constant<int, 1> odd{};
    auto run = [&](int from, int to, auto weighed) PROD_INLINE {  // kSplitA: `from` is even, and the stages are constants
        if constexpr (kSplitA) {
            int step = from;
            for (; step + 1 < to; step += 2) {
                one(even, odd, step, weighed);
                one(odd, even, step + 1, weighed);
            }
            if (step < to) one(even, odd, step, weighed);  // the last of all
        } else {
            for (int step = from; step < to; ++step) one(step & 1, (step & 1) ^ 1, step, weighed);
        }
    };
    // kQuadForm: the accumulators' contribution to the quadratic form, and a fresh start.  Once per 1024 values of k: the
    // shorter sums lose less to rounding.
    prod_f32x4 sum[4];
    auto contract = [&]() PROD_INLINE {
        const int columns = width[1] < kProdTile ? width[1] : kProdTile;
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float *>(p.E + (size_t)c0 * p.ldo + r0), 0, 4 * ((columns - 1) * p.ldo + width[0]), kRawBufferFlags);
#pragma unroll
        for (int tb = 0; tb < 4; ++tb) {
            const int cl = wc * 64 + tb * 16 + lo;
            prod_f32x4 e[4];
#pragma unroll
            for (int ta = 0; ta < 4; ++ta)
                e[ta] = __builtin_bit_cast(prod_f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                                           rsrc, 4 * (cl * p.ldo + wr * 64 + ta * 16 + 4 * hi), 0, 0));
            if (cl < columns) {
                const int shift_c = -shift[1][cl];
#pragma unroll
                for (int ta = 0; ta < 4; ++ta)
#pragma unroll
                    for (int i = 0; i < 4; ++i) sum[ta][i] = fmaf(ldexpf(acc[ta][tb][i], shift_c), e[ta][i], sum[ta][i]);
            }
        }
        clear();
    };
    // All steps under one set of scales, and once more with all magnitudes known if a guess was too low or too high.
    const bool few = !kQuad && k_end - k_begin <= kProdFew;
    if constexpr (!kQuad) {
        if (few) {
            clear();
            multiply_few();
        }
    }
    for (int attempt = 0; !few; ++attempt) {
        const int o = tid >> 7, i = tid & 127;  // this thread's row of A's tile, column of B's
        // A magnitude that the first step need not show: the diagonal of a symmetric or triangular operand.
        float hint = 0.0f, ratio = 1.0f;
        if (attempt == 0) {
            if (MODE == kSubtract && p.least) {
                float all = INFINITY, of_block[8];
#pragma unroll
                for (int b = 0; b < 8; ++b) of_block[b] = p.least[b];  // (all requested together)
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    if (b * kProdTile < p.K) all = fminf(all, of_block[2 * b]);
                ratio = of_block[1] / all;
            }
            if (kQuad && o == 1 && c0 + i < p.C) {
                hint = p.B[(size_t)(c0 + i) * p.ldb + c0 + i];
                ratio = *p.diag_max;
            }
            if ((MODE == kStore || MODE == kStoreNegated) && o == 0 && r0 + i < p.R && r0 + i < p.K)
                hint = fabsf(p.A[(size_t)(r0 + i) * p.lda + r0 + i]);
        }
        if (kSplitA) copy_a(even, 0);
        load(0);
        if (kQuad && c0 < kProdStep) weigh(0);
        track();
        if (attempt == 0) {
            largest[o][i] = 0u;
            if (tid < 2) largest_of_tile[tid] = 0u;
            __syncthreads();
            publish();
#pragma unroll
            for (int x = kGuess; x < 2; ++x) {
                float m = fmaxf(top[x][0], top[x][1]);
#pragma unroll
                for (int d = 32; d > 0; d >>= 1) m = fmaxf(m, __shfl_xor(m, d));
                if (lane == 0) atomicMax(&largest_of_tile[x], __float_as_uint(m));
            }
            __syncthreads();
        }
        {
            unsigned m = largest[o][i];
            int to = 14;
            if (attempt == 0) {  // (a row or column without any guess takes the tile's)
                if (!kQuad && hint < INFINITY) m = __float_as_uint(fmaxf(hint, __uint_as_float(m)));
                if (m == 0u) m = largest_of_tile[o];
                if (!kQuad) to = kProdTarget;
                if (MODE == kSubtract && p.least) to = 5;  // errors and rows of U grow more on the way than data do
            }
            int now = product_shift(m, to);
            if (MODE == kSubtract && p.least && o == 1 && attempt == 0) {  // and errors divided by smaller numbers are as much larger
                const float grown = __uint_as_float(m) * ratio;
                if (grown < INFINITY) now = min(now, product_shift(__float_as_uint(grown), 12));
            }
            // Quadratic form: with a positive semidefinite B no value of column c is above sqrt(max_k B[k][k] B[c][c]): that, or
            // 2^15 B[c][c] if it is less, goes to 2^15 (by exponents).
            const int e_diag = (int)(__float_as_uint(hint) >> 23) - 127, e_max = (int)(__float_as_uint(ratio) >> 23) - 127;
            if (kQuad && attempt == 0 && e_diag > -127 && e_diag < 128) now = min(now, 15 - min((e_max + e_diag + 3) >> 1, e_diag + 15));
            shift[o][i] = now;
            if (kQuad && o == 0) shift[0][i] = i < width[0] ? p.split_shift[r0 + i] : 0;
        }
        __syncthreads();
#pragma unroll
        for (int x = kFirst; x < 2; ++x)
#pragma unroll
            for (int e = 0; e < 2; ++e) s[x][e] = ldexpf(1.0f, shift[x][2 * lane + e]);
        clear();
        split_store(even);
        load(1);
        barrier();
        if constexpr (kQuad) {
            // the last steps, which reach the diagonal, are weighed one step ahead (and, to keep the number of the others even,
            // the one before them, which changes nothing in it)
            const int plain = c0 / kProdStep - 2;
            constexpr int kChunk = 1024 / kProdStep;
#pragma unroll
            for (int ta = 0; ta < 4; ++ta) sum[ta] = prod_f32x4{0.f, 0.f, 0.f, 0.f};
            int step = 0;
            while (step < plain) {
                const int to = plain - step < kChunk ? plain : step + kChunk;
                run(step, to, std::false_type{});
                if (to < plain) contract();
                step = to;
            }
            run(step, steps, std::true_type{});
        } else {
            run(0, steps - 1, std::false_type{});
            multiply((steps - 1) & 1);  // nothing follows it that had to be split
        }
        if (attempt) break;
        publish();
        __syncthreads();
        const float most = ldexpf(__uint_as_float(largest[tid >> 7][tid & 127]), shift[tid >> 7][tid & 127]);
        const bool bad = tid >> 7 >= kGuess && (tid & 127) < width[tid >> 7] &&
                         (!(most <= kProdMost) || (most < (kQuad ? 0.25f : MODE == kSubtract && p.least ? 0x1p-6f : kProdLeast) && most > 0.0f));
        if (!__syncthreads_or(bad)) break;
    }

    // Element i of a 16 x 16 accumulator: row 4 hi + i, column lo; the scales are taken out again.  Through a descriptor of
    // the tile, elements that do not exist out of range, so that the 16 old values of a column group are requested together
    // (one at a time, each behind the store of the one before, they were a third of a short product: K = 128, 384 x 3584
    // on average, 21.6 -> 12.7 us, 12.1 since the last step no longer splits a step that does not exist).
    if constexpr (!kQuad) {
        constexpr unsigned kNone = 0xfffffff0u;
        constexpr bool kSymmetric = MODE == kAddTwiceSymmetric, kRead = MODE == kSubtract || MODE == kSubtractLower || kSymmetric;
        const int rows = width[0] < kProdTile ? width[0] : kProdTile, columns = width[1] < kProdTile ? width[1] : kProdTile;
        const __amdgpu_buffer_rsrc_t tile = __builtin_amdgcn_make_buffer_rsrc(
            p.out + (size_t)r0 * p.ldo + c0, 0, 4 * ((rows - 1) * p.ldo + columns), kRawBufferFlags);
        // kAddTwiceSymmetric: element (r, c) with r < c also goes to (c, r)
        const __amdgpu_buffer_rsrc_t mirror = __builtin_amdgcn_make_buffer_rsrc(
            p.out + (size_t)c0 * p.ldo + r0, 0, kSymmetric ? 4 * ((columns - 1) * p.ldo + rows) : 0, kRawBufferFlags);
        const bool diagonal = kSymmetric && r0 == c0;
#pragma unroll
        for (int tb = 0; tb < 4; ++tb) {
            const int cl = wc * 64 + tb * 16 + lo;
            const int shift_c = shift[1][cl];
            float v[4][4];
            prod_u32x4 there[4];
            unsigned old[4][4];
#pragma unroll
            for (int ta = 0; ta < 4; ++ta) {
                const int rl = wr * 64 + ta * 16 + 4 * hi;  // rows and columns are multiples of 4
                const bool in = rl < rows && cl < columns;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (kRead)
                        old[ta][i] = __builtin_amdgcn_raw_buffer_load_b32(
                            tile, in && !(diagonal && rl + i > cl) ? 4u * (rl * p.ldo + cl) : kNone, 4 * i * p.ldo, 0);
                if (kSymmetric && !diagonal)
                    there[ta] = __builtin_amdgcn_raw_buffer_load_b128(mirror, in ? 4u * (cl * p.ldo + rl) : kNone, 0, 0);
                if (kSymmetric && diagonal) {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        there[ta][i] = __builtin_amdgcn_raw_buffer_load_b32(
                            mirror, in && rl + i < cl ? 4u * (cl * p.ldo + rl + i) : kNone, 0, 0);
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) v[ta][i] = ldexpf(acc[ta][tb][i], -(shift[0][rl + i] + shift_c));
            }
#pragma unroll
            for (int ta = 0; ta < 4; ++ta) {
                const int rl = wr * 64 + ta * 16 + 4 * hi;
                const bool in = rl < rows && cl < columns;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float w = v[ta][i];
                    if (MODE == kStoreNegated) w = -w;
                    if (MODE == kSubtract || MODE == kSubtractLower) w = __uint_as_float(old[ta][i]) - w;
                    if (kSymmetric) w = __uint_as_float(old[ta][i]) + 2.0f * w;
                    __builtin_amdgcn_raw_buffer_store_b32(
                        __float_as_uint(w), tile, in && !(diagonal && rl + i > cl) ? 4u * (rl * p.ldo + cl) : kNone, 4 * i * p.ldo, 0);
                    if (kSymmetric) there[ta][i] = __float_as_uint(__uint_as_float(there[ta][i]) + 2.0f * v[ta][i]);
                    if (kSymmetric && diagonal)
                        __builtin_amdgcn_raw_buffer_store_b32(there[ta][i], mirror,
                                                              in && rl + i < cl ? 4u * (cl * p.ldo + rl + i) : kNone, 0, 0);
                }
                if (kSymmetric && !diagonal)
                    __builtin_amdgcn_raw_buffer_store_b128(there[ta], mirror, in ? 4u * (cl * p.ldo + rl) : kNone, 0, 0);
            }
        }
    } else {
        float *red = reinterpret_cast<float *>(&stage_b[0][0][0][0]);  // [2 column halves][128 rows], free after the loop's last barrier
        contract();
#pragma unroll
        for (int ta = 0; ta < 4; ++ta)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int rl = wr * 64 + ta * 16 + 4 * hi + i;
                float all = sum[ta][i];
#pragma unroll
                for (int d = 1; d < 16; d <<= 1) all += __shfl_xor(all, d);
                if (lo == 0) red[wc * kProdTile + rl] = ldexpf(all, -shift[0][rl]);
            }
        __syncthreads();
        if (tid < kProdTile && r0 + tid < p.R) p.out[(size_t)tile_col * p.ldo + r0 + tid] = red[tid] + red[kProdTile + tid];
    }
}

// The tiles of a launch are those from `first` (a multiple of 8) on of `all`.
template <int MODE>
__device__ __forceinline__ void product_tiles(const ProductArgs &p, int first, int all)
{
    // (A's stages are two objects so that the compiler can tell the copies into one, of kQuadFormSplit, from the reads of the other)
    __shared__ __attribute__((aligned(16))) ProductStage stage_a0;
    __shared__ __attribute__((aligned(16))) ProductStage stage_a1;
    __shared__ __attribute__((aligned(16))) ProductStage stage_b[2];
    __shared__ ProductLargest largest;
    __shared__ unsigned largest_of_tile[2];
    __shared__ ProductShift shift;
    product_tile_of<MODE>(p, first + (int)blockIdx.x, all, stage_a0, stage_a1, stage_b, largest, largest_of_tile, shift);
}

template <int MODE>
__global__ __launch_bounds__(256, 2) void product_kernel(ProductArgs p)
{
    product_tiles<MODE>(p, 0, gridDim.x);
}

template <int MODE>
__global__ __launch_bounds__(256, 2) void product_part_kernel(ProductArgs p, int first, int all)
{
    product_tiles<MODE>(p, first, all);
}

static ProductArgs product_args(const float *A, int lda, int R, const float *B, int ldb, int C, int K, float *out, int ldo,
                                const float *least = nullptr)
{
    return {A, B, nullptr, out, lda, R, ldb, C, K, ldo, 0, nullptr, 0, nullptr, nullptr, least, 0, C, 0, 0, nullptr};
}

template <int MODE>
static void launch_product(hipStream_t stream, const float *A, int lda, int R, const float *B, int ldb, int C, int K, float *out, int ldo)
{
    const ProductArgs p = product_args(A, lda, R, B, ldb, C, K, out, ldo);
    hipLaunchKernelGGL((product_kernel<MODE>), dim3((unsigned)product_groups<MODE>(R, C)), dim3(256), 0, stream, p);
}

// `count` products kStore (with B[k][c] = 0 for k > c) or kStoreNegated of size x size x size, see ProductArgs.
template <int MODE>
static void launch_products(hipStream_t stream, int count, size_t stride, int columns_end, const float *A, const float *B, float *out,
                            int pitch, int size)
{
    ProductArgs p = {A, B, nullptr, out, pitch, size, pitch, size, size, pitch, MODE == kStore ? 1 : 0, nullptr, 0, nullptr, nullptr, nullptr,
                     stride, columns_end, 2 * size, MODE == kStore ? 1 : 0, nullptr};
    const int groups = product_groups<MODE>(size, size);
    hipLaunchKernelGGL((product_kernel<MODE>), dim3((unsigned)groups, (unsigned)count), dim3(256), 0, stream, p);
}

// The quadratic forms of the rows of D: kQuadForm splits them as it reads them, for kQuadFormSplit they come as `split` too
// (see ProductArgs).
template <int MODE>
static void launch_quad_form(hipStream_t stream, const uint16_t *split, size_t plane, const int *shift, const float *D, int R, const float *B,
                             int ldb, const float *diag_max, int C, float *out, int ldo, const int *rows = nullptr)
{
    ProductArgs p = {D, B, D, out, ldo, R, ldb, C, C, ldo, 0, split, plane, shift, diag_max, nullptr, 0, C, 0, 0, rows};
    const int groups = product_groups<MODE>(R, C);
    hipLaunchKernelGGL((product_kernel<MODE>), dim3((unsigned)groups), dim3(256), 0, stream, p);
}

}  // namespace bcq
