// Shared by the matrix-core kernels for several activation vectors (bcq_skinny.hip, bcq_wide.hip).  Not public.
#pragma once
#include "bcq_internal.h"
#include "bcq_device.h"

namespace bcq {

struct SkinnyParams {
    const uint8_t *blob;
    const uint16_t *X;
    uint16_t *Y;
    unsigned long long *accum;  // [batch][Mp]
    int M, N, Mp, batch, ldx, ldy;
    int ntile, nslice, ntg;  // ntg = ceil(ntile / 4) tile groups (the four row tiles of a workgroup)
    int units;               // ntg * nslice work units, cut into one contiguous range per workgroup:
    int unit_base, unit_rem; // units div / mod the number of workgroups (first_unit, owner_of_unit in bcq_device.h)
    unsigned tile_bytes;
    int scale_lane_mask;     // 63: one scale record per lane; 15: one per row (group = N)
#ifdef BCQ_TRACE
    unsigned *trace;         // [workgroup][wave][kTraceSlots] time stamps (the tracing build only)
    int trace_groups;        // workgroups the buffer has room for
#endif
};

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

// Undo the per-row byte permutation of the blob (chunk_of_byte): on return byte s of the
// 128-bit value is chunk s.
template <int SUB>
__device__ __forceinline__ void unrotate(u32x4 &w, int r)
{
    if (SUB == 1) {
        // chunk = (byte + r) mod 16: rotate the 128-bit ring left by r bytes, i.e. right by k = (16 - r) mod 16:
        // byte j of the result is byte j + k of w.  Dword step first (two rounds of selects), then one
        // v_alignbyte_b32 per dword for the k mod 4 bytes that cross dwords.
        const int k = (16 - r) & 15;
        const bool s1 = k & 4, s2 = k & 8;
        const uint32_t b = k & 3;
        uint32_t t0 = w.x, t1 = w.y, t2 = w.z, t3 = w.w;
        const uint32_t u0 = s1 ? t1 : t0, u1 = s1 ? t2 : t1, u2 = s1 ? t3 : t2, u3 = s1 ? t0 : t3;
        t0 = s2 ? u2 : u0; t1 = s2 ? u3 : u1; t2 = s2 ? u0 : u2; t3 = s2 ? u1 : u3;
        w.x = __builtin_amdgcn_alignbyte(t1, t0, b);
        w.y = __builtin_amdgcn_alignbyte(t2, t1, b);
        w.z = __builtin_amdgcn_alignbyte(t3, t2, b);
        w.w = __builtin_amdgcn_alignbyte(t0, t3, b);
    } else if (SUB == 2) {  // rotate each 64-bit half left by r mod 8 bytes, swap the halves if r >= 8
        unsigned long long lo = ((unsigned long long)w.y << 32) | w.x, hi = ((unsigned long long)w.w << 32) | w.z;
        lo = __builtin_rotateleft64(lo, 8 * (r & 7));
        hi = __builtin_rotateleft64(hi, 8 * (r & 7));
        const unsigned long long a = (r & 8) ? hi : lo, b = (r & 8) ? lo : hi;
        w.x = (uint32_t)a; w.y = (uint32_t)(a >> 32); w.z = (uint32_t)b; w.w = (uint32_t)(b >> 32);
    } else {  // rotate each dword left by r mod 4 bytes, dword d goes to d xor (r div 4)
        const unsigned sh = 8 * (r & 3);
        uint32_t t0 = __builtin_rotateleft32(w.x, sh), t1 = __builtin_rotateleft32(w.y, sh);
        uint32_t t2 = __builtin_rotateleft32(w.z, sh), t3 = __builtin_rotateleft32(w.w, sh);
        // masked exchanges (written without selects so that they stay in registers)
        const uint32_t m4 = (r & 4) ? 0xffffffffu : 0u, m8 = (r & 8) ? 0xffffffffu : 0u;
        uint32_t d01 = (t0 ^ t1) & m4, d23 = (t2 ^ t3) & m4;
        t0 ^= d01; t1 ^= d01; t2 ^= d23; t3 ^= d23;
        uint32_t d02 = (t0 ^ t2) & m8, d13 = (t1 ^ t3) & m8;
        t0 ^= d02; t2 ^= d02; t1 ^= d13; t3 ^= d13;
        w.x = t0; w.y = t1; w.z = t2; w.w = t3;
    }
}

// Sign table: entry b holds 8 binary16 values, +1.0 for a set bit: pair d = (bit d, bit d + 4) of b (the element order
// that the X staged through registers uses), or with IN_ORDER (bit 2 d, bit 2 d + 1); copy c of entry b sits at (TC b + c) * 16 and lane l reads copy
// l mod TC.  With TC = 16 copies (64 KB) the 16 lanes that a ds_read_b128 serves together always read 16
// different bank columns whatever their bytes are; with 8 copies (32 KB) two of them share a column and
// collide unless their bytes are equal, which costs the table reads about half their rate.
template <int TC> constexpr int kTabBytes = 256 * TC * 16;

template <int NT, int TC, bool IN_ORDER = false>
__device__ __forceinline__ void build_sign_table(uint8_t *tab, int tid)
{
#pragma unroll
    for (int k = 0; k < 256 * TC / NT; ++k) {
        const int idx = tid + NT * k, b = idx / TC;
        u32x4 e;
#pragma unroll
        for (int d = 0; d < 4; ++d)
            e[d] = (((b >> (IN_ORDER ? 2 * d : d)) & 1) ? 0x3c00u : 0xbc00u) |
                   ((((b >> (IN_ORDER ? 2 * d + 1 : d + 4)) & 1) ? 0x3c00u : 0xbc00u) << 16);
        *reinterpret_cast<u32x4 *>(tab + idx * 16) = e;
    }
}

// The kernel for many activation vectors: batch columns it takes per pass, and one pass (p describes exactly its columns).
int wide_columns(const Geom &g);
hipError_t launch_wide(const Geom &g, const SkinnyParams &p, const GemvTuning &tuning, hipStream_t stream);

}  // namespace bcq
