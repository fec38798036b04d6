// Activations as signed bytes for the integer matrix instruction (bcq_few.hip).  Not public.
//
// A plane's sign bits become matrix operands with one v_and_b32 per four signs: bit b of a byte, masked where it stands, is the
// signed byte 2^b (-128 for b = 7), and the column's activation enters times 2^(7 - b) (negated for b = 7), so that every
// product is 2^7 times the activation where the bit is set.  An activation is taken relative to the largest one of its
// 128-column block: v = rint(x * 2^k) with |v| <= 2^22, which is exact for a binary16 number from 2^-11 of that largest one
// up and at most 2^-22 of it off otherwise (what a binary32 sum of the block loses); times 2^(7 - b) it has 30 bits and is cut
// into four signed bytes ("digits").  All sums are exact in 32 bits.  With the products' sum T = 2^7 sum(bit v), the sum over
// the signs is 2^6 sum(+-v) = T - 2^6 sum(v): the accumulators start at the digits of -2^6 sum(v).
#pragma once
#include "bcq_device.h"

namespace bcq {

typedef int i32x4 __attribute__((ext_vector_type(4)));

template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xf, 0xf, true);
}

constexpr int kRor4 = 0x124, kRor8 = 0x128;  // rotations of 16 lanes
constexpr int kXor1 = 0xb1, kXor2 = 0x4e;    // exchanges inside four lanes

// f(f(..)) over the 16 lanes of a block, in every one of them; f commutes.
template <class F>
__device__ __forceinline__ uint32_t over_block(uint32_t v, F f)
{
    v = f(v, dpp<kXor1>(v));
    v = f(v, dpp<kXor2>(v));
    v = f(v, dpp<kRor4>(v));
    return f(v, dpp<kRor8>(v));
}

// Eight activations of a lane (one chunk; the 16 lanes of a block together) for V vectors: digits[v][b] = the digits of column
// b's integer as bytes 0 (lowest) to 3, sum = the block's sum of the integers, scale = what 2^6 sum(+-v) is multiplied by.  In a block with
// infinities only they count and the scale is infinite; with a NaN the scale is one.  The vectors go through each stage together,
// without a branch between them: one after the other they cost 0.4 us each.
template <int V>
__device__ __forceinline__ void block_digits(const u32x4 (&x)[V], uint32_t (&digits)[V][8], int (&sum)[V], float (&scale)[V])
{
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
    constexpr uint32_t kBase = 0x4b400000u;  // 1.5 * 2^23, whose low bits take the integer
    uint32_t f[V][8], m[V];
    bool finite = true;
#pragma unroll
    for (int v = 0; v < V; ++v) {
        u16x2 most = {0, 0};
#pragma unroll
        for (int k = 0; k < 4; ++k) most = __builtin_elementwise_max(most, __builtin_bit_cast(u16x2, x[v][k] & 0x7fff7fffu));
        m[v] = over_block(max((uint32_t)most.x, (uint32_t)most.y), [](uint32_t a, uint32_t b) { return max(a, b); });
        finite = finite && m[v] < 0x7c00u;
        const int e = max((int)(m[v] >> 10), 1);                           // |x| < 2^(e - 14)
        const float up = __uint_as_float((uint32_t)(127 + 36 - e) << 23);  // integers up to 2^22
        scale[v] = __uint_as_float((uint32_t)(127 - 36 - 6 + e) << 23);
#pragma unroll
        for (int k = 0; k < 8; ++k) {  // (the last column's negated)
            const uint32_t bits = (k & 1) ? x[v][k >> 1] >> 16 : x[v][k >> 1] & 0xffffu;
            f[v][k] = __float_as_uint(fmaf(half_bits_to_float(bits), k == 7 ? -up : up, 12582912.0f));
        }
    }
    if (__builtin_amdgcn_ballot_w64(!finite)) {  // (uniform)
#pragma unroll
        for (int v = 0; v < V; ++v) {
            if (m[v] < 0x7c00u) continue;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const uint32_t bits = (k & 1) ? x[v][k >> 1] >> 16 : x[v][k >> 1] & 0xffffu;
                const bool minus = ((bits & 0x8000u) != 0) != (k == 7);
                f[v][k] = (bits & 0x7fffu) < 0x7c00u ? kBase : minus ? kBase - (1u << 22) : kBase + (1u << 22);
            }
            scale[v] = __uint_as_float(m[v] == 0x7c00u ? 0x7f800000u : 0x7fc00000u);
        }
    }
#pragma unroll
    for (int v = 0; v < V; ++v) {
        sum[v] = (int)over_block((((f[v][0] + f[v][1]) + (f[v][2] + f[v][3])) + ((f[v][4] + f[v][5]) + f[v][6])) - f[v][7] - 6u * kBase,
                                 [](uint32_t a, uint32_t b) { return a + b; });
#pragma unroll
        for (int b = 0; b < 8; ++b) digits[v][b] = ((f[v][b] << (7 - b)) + (0x00808080u - (kBase << (7 - b)))) ^ 0x00808080u;
    }
}

// Byte d of the lanes 0..3 of each four, in lane d: a 4 x 4 byte transpose.
__device__ __forceinline__ uint32_t transpose_quad(uint32_t u, int lane)
{
    const uint32_t p = dpp<kXor1>(u);
    const uint32_t t = __builtin_amdgcn_perm(p, u, (lane & 1) ? 0x03070105u : 0x06020400u);
    const uint32_t q = dpp<kXor2>(t);
    return __builtin_amdgcn_perm(q, t, (lane & 2) ? 0x03020706u : 0x05040100u);
}

// What the accumulators of a block start at: digits of -2^6 sum, |sum| <= 2^29.
__device__ __forceinline__ i32x4 start_digits(int sum)
{
    return i32x4{-((sum & 3) << 6), -((sum >> 2) & 255), -((sum >> 10) & 255), -(sum >> 18)};
}

// sum_d 2^(8 d) acc[d] in binary32.  |acc[d]| <= 2^21 (128 columns of bytes) and |acc[3]| <= 2^14, so both halves are exact integers and the first is
// exact in binary32 too.
__device__ __forceinline__ float digit_value(const i32x4 &acc)
{
    const int hi = (acc[3] << 8) + acc[2], lo = (acc[1] << 8) + acc[0];
    return fmaf((float)hi, 65536.0f, (float)lo);
}

// Bits 4 half .. 4 half + 3 of every byte of w, each where it stands.
__device__ __forceinline__ i32x4 masked_signs(uint32_t w, int half)
{
    i32x4 a;
#pragma unroll
    for (int t = 0; t < 4; ++t) a[t] = (int)(w & (0x01010101u << (4 * half + t)));
    return a;
}

}  // namespace bcq
