// Activations as signed bytes for the integer matrix instruction (bcq_few.hip).  Not public.
//
// A plane's sign bits become matrix operands with one v_and_b32 per four signs: bit t of a nibble, masked where it stands (the upper
// nibbles after one shift of the dword), is the signed byte 2^t.  The column's activation enters as the integer I = rint(x 2^(31 - p - t)),
// an even one for t = 0, so that every product is 2^t I = x 2^(31 - p) where the bit is set; 2^p is the power of two above the largest
// magnitude of the (128-column block, vector), or twice that if it is within 2^-8 of it: I has 31 bits and a sign and is cut into four signed bytes
// ("digits").  All sums are exact in 32 bits, and with T = sum(bit 2^t I), S = sum(2^t I) the sum over the signs is
// sum(+-x) = 2^(p - 31) (2 T - S): the accumulators start at the digits of -S / 2.
//
// What is rounded: a binary16 number from 2^(p - 18) up is exact; others are at most 2^(p - 29) off (t = 3; 2^(p - 30) for t = 2, 2^(p - 31) below), where an
// addition in binary32 to a sum that holds the largest one loses up to 2^(p - 25).
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

// floor(f + 1/2) in one instruction.  (f has 11 significant bits: the addition is exact where it matters, whatever it is done in.)
__device__ __forceinline__ int nearest(float f)
{
    int i;
    asm("v_cvt_rpi_i32_f32 %0, %1" : "=v"(i) : "v"(f));
    return i;
}

// Eight activations of a lane (one chunk; the 16 lanes of a block together) for V vectors: digits[v][b] = the digits of column
// b's integer (t = b mod 4) as bytes 0 (lowest) to 3, scale = 2^(p - 30).  In a block with infinities only they count and the
// scale is infinite; with a NaN it is a NaN.  The vectors go through each stage together, without a branch between them: one after the
// other they cost 0.4 us each.
template <int V>
__device__ __forceinline__ void block_digits(const u32x4 (&x)[V], uint32_t (&digits)[V][8], float (&scale)[V])
{
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
    int I[V][8];  // halves of them for t = 0
    uint32_t m[V];
    bool finite = true;
#pragma unroll
    for (int v = 0; v < V; ++v) {
        u16x2 most = {0, 0};
#pragma unroll
        for (int k = 0; k < 4; ++k) most = __builtin_elementwise_max(most, __builtin_bit_cast(u16x2, x[v][k] & 0x7fff7fffu));
        m[v] = over_block(max((uint32_t)most.x, (uint32_t)most.y), [](uint32_t a, uint32_t b) { return max(a, b); });
        finite = finite && m[v] < 0x7c00u;
        // p = e - 14: 1015 / 1024 and less above a power of two stays below the largest four signed bytes, 127 (1 + 2^8 + 2^16 + 2^24)
        const int e = max((int)((m[v] + 8) >> 10), 1);
        scale[v] = __uint_as_float((uint32_t)(127 - 44 + e) << 23);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const uint32_t bits = (b & 1) ? x[v][b >> 1] >> 16 : x[v][b >> 1] & 0xffffu;
            const float up = __uint_as_float((uint32_t)(127 + 45 - e - max(b & 3, 1)) << 23);
            I[v][b] = nearest(fmaf(half_bits_to_float(bits), up, 0.0f));
        }
    }
    if (__builtin_amdgcn_ballot_w64(!finite)) {  // (uniform)
#pragma unroll
        for (int v = 0; v < V; ++v) {
            if (m[v] < 0x7c00u) continue;
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const uint32_t bits = (b & 1) ? x[v][b >> 1] >> 16 : x[v][b >> 1] & 0xffffu;
                const int one = 1 << (30 - max(b & 3, 1));
                I[v][b] = (bits & 0x7fffu) < 0x7c00u ? 0 : (bits & 0x8000u) ? -one : one;
            }
            scale[v] = __uint_as_float(m[v] == 0x7c00u ? 0x7f800000u : 0x7fc00000u);
        }
    }
#pragma unroll
    for (int v = 0; v < V; ++v)
#pragma unroll
        for (int b = 0; b < 8; ++b) digits[v][b] = (((uint32_t)I[v][b] << (b & 3 ? 0 : 1)) + 0x00808080u) ^ 0x00808080u;
}

// Byte d of the lanes 0..3 of each four, in lane d: a 4 x 4 byte transpose.
__device__ __forceinline__ uint32_t transpose_quad(uint32_t u, int lane)
{
    const uint32_t p = dpp<kXor1>(u);
    const uint32_t t = __builtin_amdgcn_perm(p, u, (lane & 1) ? 0x03070105u : 0x06020400u);
    const uint32_t q = dpp<kXor2>(t);
    return __builtin_amdgcn_perm(q, t, (lane & 2) ? 0x03020706u : 0x05040100u);
}

// What the accumulators of a block start at: digits of -S / 2 from the sums of digits.  A digit's odd half is 128 of the one below;
// the lowest is even (t = 0).
__device__ __forceinline__ i32x4 start_digits(const i32x4 &S)
{
    return i32x4{-((S[0] >> 1) + ((S[1] & 1) << 7)), -((S[1] >> 1) + ((S[2] & 1) << 7)), -((S[2] >> 1) + ((S[3] & 1) << 7)), -(S[3] >> 1)};
}

// sum_d 2^(8 d) acc[d] in binary32.  |acc[d]| <= 128 * 32 * (1 + 2 + 4 + 8) = 61440 (of sums over signs half of that, and 129), so both halves are below
// 2^24 and exact in binary32 too.
__device__ __forceinline__ float digit_value(const i32x4 &acc)
{
    const int hi = (acc[3] << 8) + acc[2], lo = (acc[1] << 8) + acc[0];
    return fmaf((float)hi, 65536.0f, (float)lo);
}

// The bits of every byte's lower nibble in w, each where it stands.
__device__ __forceinline__ i32x4 masked_signs(uint32_t w)
{
    i32x4 a;
#pragma unroll
    for (int t = 0; t < 4; ++t) a[t] = (int)(w & (0x01010101u << t));
    return a;
}

}  // namespace bcq
