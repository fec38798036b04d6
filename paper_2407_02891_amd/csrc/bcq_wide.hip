// Binary-coding product with many activation vectors (paper Eq. 11) for gfx950: Y[j][m] = sum_k W_q[m][k] X[j][k], up to
// 16 NB vectors per pass over the weights.
//
// The arithmetic is the table kernel's of bcq_skinny.hip: the four lanes that hold the four blocks of a row exchange
// dwords, after which one v_mfma_f32_16x16x32_f16 contracts 32 columns of a single block with +-1.0 operands from a
// 256-entry table in LDS, and the binary32 sums of a scaling group are multiplied by its alpha.  Every sign operand serves
// NB matrix instructions, so from two column groups on these are the largest part of a pass and everything else has to stay
// out of their way.  Counters at 64 columns of 7168 x 28672, q = 3 (83 us): matrix pipe busy 37 % of the time, vector ALU 19 %, LDS
// 23 % (no bank conflicts), waves at a wait 40 % of their cycles: what bounds it is that two waves per SIMD in lock step per
// stage do not keep the matrix pipe fed.
//
//  * Two waves per SIMD (eight per workgroup, one workgroup per compute unit) in 256 registers: the two row halves of a
//    tile are taken one after the other, so that only one half's block sums and operands are live.
//  * X is copied to LDS by the memory system itself (buffer loads with an LDS destination), no registers and no vector
//    instructions: a stage is one 128-column block of 16 NB vectors per K group, two stages, one barrier per stage.  A lane's
//    16 bytes go where the instruction puts them, so the layout is made by the source addresses: the chunks of a row are
//    stored at position chunk ^ g(row), g(r) = r ^ ((r & 4) << 1), with which the 16 lanes that a ds_read_b128 serves
//    together ({0-3, 12-15, 20-23, 24-27}, {4-7, 8-11, 16-19, 28-31} and + 32) touch 16 different 16-byte columns.
//  * A workgroup covers four row tiles (128 rows) and two neighbouring column slices at a time: waves 0-3 take the even
//    slice of a pair, waves 4-7 the odd one (K groups), and the two partial sums of a row tile meet in LDS when the
//    workgroup leaves it.  Half the rows per workgroup means half the split-K atomics of eight row tiles for the same number
//    of workgroups, and they are what the kernel before this one paid most for besides the matrix instructions.
//  * Groups of 32 or 64 columns per scale have a kernel of their own (bcq_wide_groups_kernel).  The bytes of a scaling group are put in order in
//    registers (alignbyte, a 4 x 4 byte transpose) and the dwords exchanged through a wave's own piece of LDS, 12 instructions and an LDS round trip
//    per 16 bytes where lane swaps took 40; the scales lie there too, where the lane that needs a group finds them without selects.  A block's X
//    operands are in registers, read once for both row halves: while the second half is computed each is replaced by the next block's, so a
//    stage is free again in the middle of the block that it was filled for, where the barrier stands.  The sums of a finished group are scaled plane by
//    plane between the matrix instructions that start the next one.  us, before and after: 10855 x 26304 q = 3 groups of 32, 17 columns 113 -> 97,
//    64 columns 228 -> 197; 13102 x 18880 q = 2 with offset, groups of 64, 45 columns 78 -> 71, 64 columns 98 -> 89; 5000 x 7232 27 columns 19.5 -> 18.7;
//    q = 1 4755 x 5312 17.8 -> 17.1, 2193 x 17600 19.0 -> 19.5.  With one group per block that way of holding X gains nothing (28672 x 8192, 64 columns 80.7 / 80.8;
//    24524 x 5824, 32 columns 35.9 / 38.1), so the kernel there reads X for each half.
//  * Workgroups per row group: a whole number unless that leaves too much of the chip idle (plan_wide), so that no workgroup
//    holds parts of two row groups; a single one writes its outputs without atomics.
#include <atomic>

#include "bcq_internal.h"
#include "bcq_device.h"
#include "bcq_skinny.h"

namespace bcq {

struct WideParams {
    SkinnyParams s;
    int pairs;             // pairs of column slices
    int parts;             // > 0: workgroups per row group, each an even share of its pairs; 0: contiguous ranges over all
};

constexpr int kWideRowTiles = 4, kWideWaves = 8;

// Adds one half of a row tile (16 rows) to the outputs: acc[nb][j] = (batch column 16 nb + h + 4 j, row r) in lane 16 h + r.
// All atomics are in flight at once: one round trip to memory per flush.
template <int NB>
__device__ __forceinline__ void wide_store(const SkinnyParams &p, int cols, const f32x4 (&acc)[NB], int row, int h, int arrivals)
{
    if (arrivals == 1) {
#pragma unroll
        for (int k = 0; k < 4 * NB; ++k) {
            const int col = 16 * (k >> 2) + h + 4 * (k & 3);
            if (col < cols && row < p.M) p.Y[(size_t)col * p.ldy + row] = float_to_half_bits(acc[k >> 2][k & 3]);
        }
        return;
    }
    unsigned long long mine[4 * NB], old[4 * NB];
#pragma unroll
    for (int k = 0; k < 4 * NB; ++k) {
        const int col = 16 * (k >> 2) + h + 4 * (k & 3);
        mine[k] = old[k] = 0;  // (no arrival: such a column is not completed below)
        if (col < cols) {
            mine[k] = encode_partial_f32(acc[k >> 2][k & 3]);
            old[k] = __hip_atomic_fetch_add(p.accum + (size_t)col * p.Mp + row, mine[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
#pragma unroll
    for (int k = 0; k < 4 * NB; ++k) {
        const int col = 16 * (k >> 2) + h + 4 * (k & 3);
        const unsigned long long total = old[k] + mine[k];
        if (arrivals_of(total) == (unsigned)arrivals) {
            if (row < p.M) p.Y[(size_t)col * p.ldy + row] = float_to_half_bits(decode_total(total));
            __hip_atomic_store(p.accum + (size_t)col * p.Mp + row, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// One scaling group per block.
template <int Q, int Z, int NB>
__global__ __launch_bounds__(64 * kWideWaves, 2) void bcq_wide_kernel(WideParams wp)
{
    constexpr int kRows = 16 * NB;                 // staged vectors
    constexpr int kStage = 2 * kRows * 256;        // one stage: [K group][vector][16 chunks of 16 bytes]
    constexpr int kCopies = kStage / 1024 / kWideWaves;  // copy instructions per wave and stage (each moves four rows)
    constexpr int kRec = Q + Z;                    // dwords of a scale record
    static_assert(kCopies >= 1, "a wave copies at least four rows");
    __shared__ __attribute__((aligned(16))) uint8_t stage0[kStage];
    __shared__ __attribute__((aligned(16))) uint8_t stage1[kStage];
    __shared__ __attribute__((aligned(16))) uint8_t tab[kTabBytes<16>];
    const SkinnyParams &p = wp.s;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, h = lane >> 4;
    const int kg = wave >> 2, rt = wave & 3;

    // this workgroup's units (row group, pair of slices), row group first
    int u_begin, u_end;
    const int groups = gridDim.x;
    if (wp.parts) {
        const int rg = blockIdx.x / wp.parts, part = blockIdx.x - rg * wp.parts;
        u_begin = rg * wp.pairs + (int)(((long long)part * wp.pairs) / wp.parts);
        u_end = rg * wp.pairs + (int)(((long long)(part + 1) * wp.pairs) / wp.parts);
    } else {
        u_begin = first_unit<true>(blockIdx.x, p.units, groups, p.unit_base, p.unit_rem);
        u_end = first_unit<true>(blockIdx.x + 1, p.units, groups, p.unit_base, p.unit_rem);
    }
    if (u_begin >= u_end) return;  // uniform for the workgroup, before any barrier

    // ---- copying X: instruction c of this wave fills the four rows 4 (wave kCopies + c) .. + 3 of the stage ----
    const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t *>(p.X), 0, (int)(2u * ((uint32_t)(p.batch - 1) * (uint32_t)p.ldx + (uint32_t)p.N)), kRawBufferFlags);
    uint32_t src[kCopies];   // byte offset of the lane's chunk in block 0 of slice 0
    int chunk8[kCopies];     // first column of that chunk inside a block; beyond all columns for a row without a vector
#pragma unroll
    for (int c = 0; c < kCopies; ++c) {
        const int row = (4 * (wave * kCopies + c) + (lane >> 4)) % kRows;  // the same rows for both K groups
        const int rho = row & 15, g = rho ^ ((rho & 4) << 1);
        const int col = (row & ~15) + (rho >> 2) + 4 * (rho & 3);  // staged row 4 h + j holds column h + 4 j (see wide_store)
        chunk8[c] = col < p.batch ? 8 * ((lane & 15) ^ g) : p.N;
        src[c] = 2u * ((uint32_t)col * (uint32_t)p.ldx + (uint32_t)chunk8[c]);
    }
    auto copy_stage = [&](uint8_t *stage, int pair, int B) {
        int first = wave * kCopies;
        asm volatile("" : "+s"(first));  // (the destinations are worked out here, not kept in scalar registers)
#pragma unroll
        for (int c = 0; c < kCopies; ++c) {
            const int group = (first + c) / (kRows / 4);  // K group of these rows
            const int col0 = kTileCols * (2 * pair + group) + kBlockCols * B;
            const uint32_t off = col0 + chunk8[c] < p.N ? src[c] + 2u * (uint32_t)col0 : 0xfffffff0u;  // beyond N: zeros
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                xrsrc, (__attribute__((address_space(3))) void *)(stage + 1024 * (first + c)), 16, (int)off, 0, 0, 0);
        }
    };

    int rg = u_begin / wp.pairs, pair = u_begin - rg * wp.pairs;
    auto tile_rsrc = [&](int rgroup, int pr, bool wanted) {
        const int t = kWideRowTiles * rgroup + rt, sl = 2 * pr + kg;
        const bool ok = wanted && t < p.ntile && sl < p.nslice;
        return __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint8_t *>(p.blob + (ok ? ((size_t)sl * p.ntile + t) * p.tile_bytes : 0)), 0, ok ? (int)p.tile_bytes : 0,
            kRawBufferFlags);
    };
    TileRegs<Q, Z, 1> cur;
    const int scale_lane = lane & p.scale_lane_mask;
    copy_stage(stage0, pair, 0);
    load_tile_buf<Q, Z, 1>(cur, tile_rsrc(rg, pair, true), lane, scale_lane);
    build_sign_table<64 * kWideWaves, 16, true>(tab, tid);
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");

    const uint32_t copy_bits = (lane & 15) * 16;  // this lane's copy of the sign table
    // staged rows of K group kg: row r of a column group, chunk 4 h + s at position (4 h + s) ^ g(r)
    const int g_r = r ^ ((r & 4) << 1);
    const int xrow = kg * kRows * 256 + r * 256;
    const u32x4 ones = {0x3c003c00u, 0x3c003c00u, 0x3c003c00u, 0x3c003c00u};
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};

    int u = u_begin;
    while (u < u_end) {
        const int seg_end = min(u_end, (rg + 1) * wp.pairs), seg_rg = rg;
        f32x4 acc[NB][2];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[nb][0] = acc[nb][1] = zero;
        for (; u < seg_end; ++u) {
            const bool more = u + 1 < u_end;
            int n_pair = pair + 1, n_rg = rg;
            if (n_pair == wp.pairs) { n_pair = 0; n_rg = rg + 1; }
            const __amdgpu_buffer_rsrc_t n_rsrc = tile_rsrc(n_rg, n_pair, more);
            TileRegs<Q, Z, 1> nxt;

            // chunk order, then the 4 x 4 dword transpose across the lanes r, r + 16, r + 32, r + 48:
            // wb[t][i][B] = chunks 4 h .. 4 h + 3 of (row 16 t + r, block B, plane i)
            uint32_t wb[2][Q][4];
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    u32x4 w = cur.planes[t][i];
                    unrotate<1>(w, r);
                    const auto e01 = __builtin_amdgcn_permlane16_swap(w.x, w.y, false, false);
                    const auto e23 = __builtin_amdgcn_permlane16_swap(w.z, w.w, false, false);
                    const auto f02 = __builtin_amdgcn_permlane32_swap(e01[0], e23[0], false, false);
                    const auto f13 = __builtin_amdgcn_permlane32_swap(e01[1], e23[1], false, false);
                    wb[t][i][0] = f02[0]; wb[t][i][1] = f13[0]; wb[t][i][2] = f02[1]; wb[t][i][3] = f13[1];
                }
            uint32_t rec[kRec];
#pragma unroll
            for (int e = 0; e < kRec; ++e) rec[e] = cur.scales[e];

#pragma unroll
            for (int B = 0; B < 4; ++B) {
                const uint8_t *const xs = (B & 1) ? stage1 : stage0;
                // requests: the next stage's X first (the wait at the end of this stage counts what follows), then a piece
                // of the next unit's tile
                __builtin_amdgcn_sched_barrier(0);
                if (B < 3) copy_stage((B & 1) ? stage0 : stage1, pair, B + 1);
                else copy_stage(stage0, more ? n_pair : wp.pairs, 0);  // (beyond the last slice: zeros)
                asm volatile("" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
                if (B < 2) {
#pragma unroll
                    for (int i = 0; i < Q; ++i) load_tile_piece<Q, Z, 1>(nxt, n_rsrc, lane, scale_lane, B * Q + i);
                } else if (B == 2) {
                    load_tile_piece<Q, Z, 1>(nxt, n_rsrc, lane, scale_lane, 2 * Q);
                }
                __builtin_amdgcn_sched_barrier(0);
                // this block's scale record, from the lane group that owns it
                uint32_t sc[kRec];
#pragma unroll
                for (int e = 0; e < kRec; ++e) sc[e] = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * (16 * B + r), (int)rec[e]);

                auto fetch = [&](int q8, f16x8 (&a)[Q], f16x8 (&bx)[NB]) {
                    const int t = q8 >> 2, s = q8 & 3;
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
                        bx[nb] = *reinterpret_cast<const f16x8 *>(xs + xrow + nb * 4096 + (((4 * h + s) ^ g_r) * 16));
#pragma unroll
                    for (int i = 0; i < Q; ++i) {
                        asm volatile("" : "+v"(wb[t][i][B]));  // keeps the address arithmetic of later steps out of this one
                        const uint32_t off = __builtin_amdgcn_perm(wb[t][i][B], copy_bits, 0x0c0c0400u | ((uint32_t)s << 8));
                        a[i] = *reinterpret_cast<const f16x8 *>(tab + off);
                    }
                };
                f16x8 abuf[2][Q], bbuf[2][NB];
                fetch(0, abuf[0], bbuf[0]);
                f32x4 C[NB][Q];
                f32x4 Cz[Z ? NB : 1];
#pragma unroll
                for (int q8 = 0; q8 < 8; ++q8) {
                    const int t = q8 >> 2, s = q8 & 3, cb = q8 & 1;
                    const bool start = s == 0, done = s == 3;
                    __builtin_amdgcn_sched_barrier(0);
                    if (q8 + 1 < 8) fetch(q8 + 1, abuf[cb ^ 1], bbuf[cb ^ 1]);
                    float v[Q + Z];
                    if (done) {
                        // scales of the block, which is finished by this step
#pragma unroll
                        for (int e = 0; e < kRec; ++e) asm volatile("" : "+v"(sc[e]));  // (not earlier)
#pragma unroll
                        for (int c = 0; c < Q + Z; ++c) {
                            const int e = t * (Q + Z) + c;
                            v[c] = half_bits_to_float((e & 1) ? (sc[e >> 1] >> 16) : (sc[e >> 1] & 0xffffu));
                        }
                    }
                    auto mul = [&](int nb, int i) {
                        C[nb][i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(bbuf[cb][nb], abuf[cb][i], start ? zero : C[nb][i], 0, 0, 0);
                    };
                    auto sums = [&](int nb) {
                        if (Z && t == 0)  // column sums of X, the same for both row halves
                            Cz[Z ? nb : 0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(bbuf[cb][nb], __builtin_bit_cast(f16x8, ones),
                                                                                    start ? zero : Cz[Z ? nb : 0], 0, 0, 0);
                    };
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) {
#pragma unroll
                        for (int i = 0; i < Q; ++i) mul(nb, i);
                        sums(nb);
                    }
                    if (done) {
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb) {
#pragma unroll
                            for (int c = 0; c < Q + Z; ++c)
#pragma unroll
                                for (int j = 0; j < 4; ++j)
                                    acc[nb][t][j] = fmaf(v[c], c == Q ? Cz[Z ? nb : 0][j] : C[nb][c < Q ? c : 0][j], acc[nb][t][j]);
                            // the sums exist here: left alone the compiler moves the scaling of all blocks to the end of the
                            // unit and keeps every block's sums until then
                            asm volatile("" : "+v"(acc[nb][t]));
                        }
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
                // the next stage's X has arrived (what was requested after it may still be under way); everyone is done with
                // this stage
                if (B < 2) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(Q) : "memory");
                // (the compiler may join the scale loads, four dwords to an instruction at most)
                else if (B == 2) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((kRec + 3) / 4) : "memory");
                else asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
            }
            if (more) cur = nxt;
            rg = n_rg; pair = n_pair;
        }
        // Flush.  The two K groups of a row tile meet in the second stage's buffer, which nobody uses until the next unit's
        // first stage has been computed: wave kg keeps row half kg and hands the other half over.
        // (The lane index goes through an empty asm so that the per-lane addresses of the flush are not kept in registers
        // during the units.)
        int fl = lane;
        asm volatile("" : "+v"(fl));
        int cols = p.batch;
        asm volatile("" : "+s"(cols));
        float *const meet = reinterpret_cast<float *>(stage1) + rt * (NB * 2 * 4 * 64) + fl;  // [K group][column group][j][lane]
        float *const here = meet + kg * (NB * 4 * 64), *const there = meet + (kg ^ 1) * (NB * 4 * 64);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float give = kg ? acc[nb][0][j] : acc[nb][1][j];
                here[(4 * nb + j) * 64] = give;
            }
        __syncthreads();
        // number of workgroups that contribute to this row group
        int arrivals = wp.parts;
        if (arrivals == 0)
            arrivals = owner_of_unit<true>((seg_rg + 1) * wp.pairs - 1, p.units, groups, p.unit_base, p.unit_rem) -
                       owner_of_unit<true>(seg_rg * wp.pairs, p.units, groups, p.unit_base, p.unit_rem) + 1;
        const int row = (kWideRowTiles * seg_rg + rt) * kTileRows + 16 * kg + (fl & 15);
        if (kWideRowTiles * seg_rg + rt < p.ntile) {  // uniform for the wave
            f32x4 v[NB];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    v[nb][j] = (kg ? acc[nb][1][j] : acc[nb][0][j]) + there[(4 * nb + j) * 64];
            wide_store<NB>(p, cols, v, row, fl >> 4, arrivals);
        }
        __syncthreads();  // the buffer is free again
    }
}

// A tile's share of a lane, with the scale record in a vector type: as an array some instances keep it in memory.
typedef uint32_t u32x16 __attribute__((ext_vector_type(16)));

template <int Q>
struct WideTile {
    u32x4 planes[2][Q];
    u32x16 scales;
};

template <int Q, int Z, int SUB>
__device__ __forceinline__ void wide_load_scales(WideTile<Q> &r, __amdgpu_buffer_rsrc_t rsrc, int scale_lane)
{
    const uint32_t so = 2u * Q * 1024u + 4u * (Q + Z) * SUB * scale_lane;
#pragma unroll
    for (int c = 0; c < (Q + Z) * SUB; ++c) r.scales[c] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, so + 4u * c, 0, 2);
}

template <int Q>
__device__ __forceinline__ void wide_load_plane(WideTile<Q> &r, __amdgpu_buffer_rsrc_t rsrc, int lane, int t, int i)
{
    r.planes[t][i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, 16u * lane + (t * Q + i) * 1024u, 0, 2);
}

// A lane's scales to LDS, [row half][byte range] 64 BYTES apart.
template <int Q, int Z, int SUB, int BYTES>
__device__ __forceinline__ void store_scales(const u32x16 &r, uint8_t *dst)
{
#pragma unroll
    for (int g = 0; g < 2 * SUB; ++g) {
        uint32_t o[4] = {0, 0, 0, 0};
#pragma unroll
        for (int c = 0; c < Q + Z; ++c) {
            const int e = g * (Q + Z) + c;
            o[c] = (e & 1) ? r[e >> 1] >> 16 : r[e >> 1] & 0xffffu;
        }
        if constexpr (BYTES == 4) *reinterpret_cast<uint32_t *>(dst + 64 * BYTES * g) = o[0] | o[1] << 16;
        else *reinterpret_cast<u32x2 *>(dst + 64 * BYTES * g) = u32x2{o[0] | o[1] << 16, o[2] | o[3] << 16};
    }
}

// Two or four scaling groups per block.
template <int Q, int Z, int SUB, int NB>
__global__ __launch_bounds__(64 * kWideWaves, 2) void bcq_wide_groups_kernel(WideParams wp)
{
    constexpr int kRows = 16 * NB;                 // staged vectors
    constexpr int kStage = 2 * kRows * 256;        // one stage: [K group][vector][16 chunks of 16 bytes]
    constexpr int kCopies = kStage / 1024 / kWideWaves;  // copy instructions per wave and stage (each moves four rows)
    constexpr int kRec = (Q + Z) * SUB;            // dwords of a scale record
    constexpr int kPer = 4 / SUB;                  // steps per scaling group
    constexpr int kScaleBytes = Q + Z <= 2 ? 4 : 8;  // the scales of a (row, block, byte range), in LDS
    constexpr int kAhead = 1, kBufs = kAhead + 1;  // steps that sign operands are requested ahead
    static_assert((SUB == 2 || SUB == 4) && Q + Z <= 4, "scaling groups per block, scales per record");
    static_assert(kCopies >= 1, "a wave copies at least four rows");
    __shared__ __attribute__((aligned(16))) uint8_t stages[2 * kStage];
    __shared__ __attribute__((aligned(16))) uint8_t tab[kTabBytes<16>];
    // a wave's own piece: sign words on their way between lanes, then the scales of the unit
    constexpr int kOwn = Q * 1024 > 2 * SUB * 64 * kScaleBytes ? Q * 1024 : 2 * SUB * 64 * kScaleBytes;
    __shared__ __attribute__((aligned(16))) uint8_t owns[kWideWaves * kOwn];
    static_assert(sizeof(stages) + sizeof(tab) + sizeof(owns) <= 160 * 1024, "one workgroup per compute unit");
    const SkinnyParams &p = wp.s;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, h = lane >> 4;
    const int kg = wave >> 2, rt = wave & 3;

    // this workgroup's units (row group, pair of slices), row group first
    int u_begin, u_end;
    const int groups = gridDim.x;
    if (wp.parts) {
        const int rg = blockIdx.x / wp.parts, part = blockIdx.x - rg * wp.parts;
        u_begin = rg * wp.pairs + (int)(((long long)part * wp.pairs) / wp.parts);
        u_end = rg * wp.pairs + (int)(((long long)(part + 1) * wp.pairs) / wp.parts);
    } else {
        u_begin = first_unit<true>(blockIdx.x, p.units, groups, p.unit_base, p.unit_rem);
        u_end = first_unit<true>(blockIdx.x + 1, p.units, groups, p.unit_base, p.unit_rem);
    }
    if (u_begin >= u_end) return;  // uniform for the workgroup, before any barrier

    // ---- copying X: instruction c of this wave fills the four rows 4 (wave kCopies + c) .. + 3 of the stage ----
    const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t *>(p.X), 0, (int)(2u * ((uint32_t)(p.batch - 1) * (uint32_t)p.ldx + (uint32_t)p.N)), kRawBufferFlags);
    uint32_t src[kCopies];   // byte offset of the lane's chunk in block 0 of slice 0
    int chunk8[kCopies];     // first column of that chunk inside a block; beyond all columns for a row without a vector
#pragma unroll
    for (int c = 0; c < kCopies; ++c) {
        const int row = (4 * (wave * kCopies + c) + (lane >> 4)) % kRows;  // the same rows for both K groups
        const int rho = row & 15, g = rho ^ ((rho & 4) << 1);
        const int col = (row & ~15) + (rho >> 2) + 4 * (rho & 3);  // staged row 4 h + j holds column h + 4 j (see wide_store)
        chunk8[c] = col < p.batch ? 8 * ((lane & 15) ^ g) : p.N;
        src[c] = 2u * ((uint32_t)col * (uint32_t)p.ldx + (uint32_t)chunk8[c]);
    }
    auto copy_stage = [&](int which, int pair, int B) {
        int first = wave * kCopies;
        asm volatile("" : "+s"(first));  // (the destinations are worked out here, not kept in scalar registers)
#pragma unroll
        for (int c = 0; c < kCopies; ++c) {
            const int group = (first + c) / (kRows / 4);  // K group of these rows
            const int col0 = kTileCols * (2 * pair + group) + kBlockCols * B;
            const uint32_t off = col0 + chunk8[c] < p.N ? src[c] + 2u * (uint32_t)col0 : 0xfffffff0u;  // beyond N: zeros
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                xrsrc, (__attribute__((address_space(3))) void *)(stages + which * kStage + 1024 * (first + c)), 16, (int)off, 0, 0, 0);
        }
    };

    int rg = u_begin / wp.pairs, pair = u_begin - rg * wp.pairs;
    auto tile_rsrc = [&](int rgroup, int pr, bool wanted) {
        const int t = kWideRowTiles * rgroup + rt, sl = 2 * pr + kg;
        const bool ok = wanted && t < p.ntile && sl < p.nslice;
        return __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint8_t *>(p.blob + (ok ? ((size_t)sl * p.ntile + t) * p.tile_bytes : 0)), 0, ok ? (int)p.tile_bytes : 0,
            kRawBufferFlags);
    };
    WideTile<Q> nxt;
    const int scale_lane = lane & p.scale_lane_mask;
    copy_stage(0, pair, 0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    {
        const __amdgpu_buffer_rsrc_t rsrc = tile_rsrc(rg, pair, true);
#pragma unroll
        for (int k = 0; k < 2 * Q; ++k) wide_load_plane<Q>(nxt, rsrc, lane, k / Q, k % Q);
        wide_load_scales<Q, Z, SUB>(nxt, rsrc, scale_lane);
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    copy_stage(1, pair, 1);  // (waited for in the middle of the first block)
    build_sign_table<64 * kWideWaves, 16, true>(tab, tid);
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(kCopies) : "memory");

    const uint32_t copy_bits = (lane & 15) * 16;  // this lane's copy of the sign table
    // staged rows of K group kg: row r of a column group, chunk 4 s + h at position (4 s + h) ^ g(r)
    const int g_r = r ^ ((r & 4) << 1);
    const uint8_t *const xrow = stages + kg * kRows * 256 + r * 256;
    const u32x4 ones = {0x3c003c00u, 0x3c003c00u, 0x3c003c00u, 0x3c003c00u};
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f16x8 X[4][NB];  // the operands of the block at hand
    auto read_x = [&](int which, int s) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
            X[s][nb] = *reinterpret_cast<const f16x8 *>(xrow + which * kStage + nb * 4096 + (((4 * s + h) ^ g_r) * 16));
    };
#pragma unroll
    for (int s = 0; s < 4; ++s) read_x(0, s);

    uint8_t *const slot = owns + wave * kOwn;
    const uint32_t turn = (4 - (r & 3)) & 3;
    // byte s of an outgoing dword comes from dword s xor `group`, which puts the block's scaling groups in order
    const uint32_t group = SUB == 2 ? (uint32_t)(((8 - (r & 7)) & 7) >> 2 | (r >> 3) << 1) : (uint32_t)(r >> 2);
    uint32_t sel0 = 0, sel1 = 0;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const uint32_t d = (uint32_t)s ^ group;  // dword whose byte goes to position s; a0/b0 hold dwords (0,1)/(2,3)
        const uint32_t lowb = (d & 1) + ((d & 2) ? 4u : 0u);
        sel0 |= lowb << (8 * s);
        sel1 |= (lowb + 2u) << (8 * s);
    }

    const uint32_t own_scale = (subgroup_of_range(0, r, SUB) * 64 + r) * kScaleBytes;

    int u = u_begin;
    while (u < u_end) {
        const int seg_end = min(u_end, (rg + 1) * wp.pairs), seg_rg = rg;
        f32x4 acc[NB][2];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[nb][0] = acc[nb][1] = zero;
        for (; u < seg_end; ++u) {
            const bool more = u + 1 < u_end;
            int n_pair = pair + 1, n_rg = rg;
            if (n_pair == wp.pairs) { n_pair = 0; n_rg = rg + 1; }
            const __amdgpu_buffer_rsrc_t n_rsrc = tile_rsrc(n_rg, n_pair, more);

            // wb[t][i][B]: byte s = chunk 4 s + h of (row 16 t + r, block B, plane i)
            uint32_t wb[2][Q][4];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    const u32x4 w = nxt.planes[t][i];
                    // bytes in order inside a scaling group, then byte s of every dword from dword s (groups in order: sel0, sel1) and
                    // the dwords of the four lanes exchanged through LDS
                    u32x4 v;
                    if constexpr (SUB == 2) {
                        v = u32x4{__builtin_amdgcn_alignbyte(w.y, w.x, turn), __builtin_amdgcn_alignbyte(w.x, w.y, turn),
                                  __builtin_amdgcn_alignbyte(w.w, w.z, turn), __builtin_amdgcn_alignbyte(w.z, w.w, turn)};
                    } else {
                        v = u32x4{__builtin_amdgcn_alignbyte(w.x, w.x, turn), __builtin_amdgcn_alignbyte(w.y, w.y, turn),
                                  __builtin_amdgcn_alignbyte(w.z, w.z, turn), __builtin_amdgcn_alignbyte(w.w, w.w, turn)};
                    }
                    const uint32_t a0 = __builtin_amdgcn_perm(v.y, v.x, 0x05010400u), a1 = __builtin_amdgcn_perm(v.y, v.x, 0x07030602u);
                    const uint32_t b0 = __builtin_amdgcn_perm(v.w, v.z, 0x05010400u), b1 = __builtin_amdgcn_perm(v.w, v.z, 0x07030602u);
                    *reinterpret_cast<u32x4 *>(slot + i * 1024 + lane * 16) =
                        u32x4{__builtin_amdgcn_perm(b0, a0, sel0), __builtin_amdgcn_perm(b0, a0, sel1), __builtin_amdgcn_perm(b1, a1, sel0),
                              __builtin_amdgcn_perm(b1, a1, sel1)};
#pragma unroll
                    for (int B = 0; B < 4; ++B) wb[t][i][B] = *reinterpret_cast<const uint32_t *>(slot + i * 1024 + 256 * B + 16 * r + 4 * h);
                }
            }
            store_scales<Q, Z, SUB, kScaleBytes>(nxt.scales, slot + lane * kScaleBytes);  // (the sign words are in registers)

            f16x8 abuf[kBufs][Q];
            auto fetch = [&](int q) {  // sign operands of step q = 8 B + 4 t + s
                const int B = q >> 3, t = (q >> 2) & 1, s = q & 3;
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    const uint32_t off = __builtin_amdgcn_perm(wb[t][i][B], copy_bits, 0x0c0c0400u | ((uint32_t)s << 8));
                    abuf[q % kBufs][i] = *reinterpret_cast<const f16x8 *>(tab + off);
                }
            };
#pragma unroll
            for (int q = 0; q < kAhead; ++q) fetch(q);

            f32x4 C[NB][Q + Z];
            float v[Q + Z];
            // adds term c of the group that has just been finished for row half t
            auto apply = [&](int t, int c) {
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        acc[nb][t][j] = fmaf(v[c], C[nb][c][j], acc[nb][t][j]);
            };
#pragma unroll
            for (int q = 0; q < 32; ++q) {
                const int B = q >> 3, t = (q >> 2) & 1, s = q & 3, cb = q % kBufs;
                const bool start = s % kPer == 0, done = s % kPer == kPer - 1;
                if ((q & 7) == 4) {
                    // the next block's X has arrived (what was requested after it may still be under way), and everyone's reads of this
                    // block's have returned (lgkmcnt: nothing else waits for them before the barrier, and a refill does not wait for
                    // reads that are queued): its stage can be filled again
                    if (B == 0) asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
                    else if (B < 3) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(Q) : "memory");
                    else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((kRec + 3) / 4) : "memory");
                    __builtin_amdgcn_sched_barrier(0);
                    if (B < 2) copy_stage(B & 1, pair, B + 2);
                    else copy_stage(B & 1, more ? n_pair : wp.pairs, B - 2);  // (beyond the last slice: zeros)
                    asm volatile("" ::: "memory");
                    __builtin_amdgcn_sched_barrier(0);
                    if (B < 2) {
#pragma unroll
                        for (int i = 0; i < Q; ++i) wide_load_plane<Q>(nxt, n_rsrc, lane, B, i);
                    } else if (B == 2) {
                        wide_load_scales<Q, Z, SUB>(nxt, n_rsrc, scale_lane);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (q + kAhead < 32) fetch(q + kAhead);
                const int tp = ((q + 31) >> 2) & 1;  // row half of the step before
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    if (start && q > 0) apply(tp, i);
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
                        C[nb][i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(X[s][nb], abuf[cb][i], start ? zero : C[nb][i], 0, 0, 0);
                }
                if (Z) {
                    if (start && q > 0) apply(tp, Q);
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)  // column sums of X
                        C[nb][Q + Z - 1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(X[s][nb], __builtin_bit_cast(f16x8, ones),
                                                                                  start ? zero : C[nb][Q + Z - 1], 0, 0, 0);
                }
                if (t == 1) read_x((B & 1) ^ 1, s);  // the next block's
                if (done) {
                    // scales of the group that is finished by this step, from the lane and the byte range that hold it
                    const uint8_t *const own = slot + (own_scale ^ ((s / kPer) * 64 * kScaleBytes)) + (t * SUB * 64 + 16 * B) * kScaleBytes;
                    uint32_t o[2] = {0, 0};
                    if constexpr (kScaleBytes == 4) {
                        o[0] = *reinterpret_cast<const uint32_t *>(own);
                    } else {
                        const u32x2 both = *reinterpret_cast<const u32x2 *>(own);
                        o[0] = both.x;
                        o[1] = both.y;
                    }
#pragma unroll
                    for (int c = 0; c < Q + Z; ++c) v[c] = half_bits_to_float((c & 1) ? o[c >> 1] >> 16 : o[c >> 1] & 0xffffu);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int c = 0; c < Q + Z; ++c) apply(1, c);
            rg = n_rg; pair = n_pair;
        }
        // Flush.  The two K groups of a row tile meet in the first stage's buffer, whose block is in everyone's registers: wave kg keeps
        // row half kg and hands the other half over.
        // (The lane index goes through an empty asm so that the per-lane addresses of the flush are not kept in registers
        // during the units.)
        int fl = lane;
        asm volatile("" : "+v"(fl));
        int cols = p.batch;
        asm volatile("" : "+s"(cols));
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        float *const meet = reinterpret_cast<float *>(stages) + rt * (NB * 2 * 4 * 64) + fl;  // [K group][column group][j][lane]
        float *const here = meet + kg * (NB * 4 * 64), *const there = meet + (kg ^ 1) * (NB * 4 * 64);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float give = kg ? acc[nb][0][j] : acc[nb][1][j];
                here[(4 * nb + j) * 64] = give;
            }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        // number of workgroups that contribute to this row group
        int arrivals = wp.parts;
        if (arrivals == 0)
            arrivals = owner_of_unit<true>((seg_rg + 1) * wp.pairs - 1, p.units, groups, p.unit_base, p.unit_rem) -
                       owner_of_unit<true>(seg_rg * wp.pairs, p.units, groups, p.unit_base, p.unit_rem) + 1;
        const int row = (kWideRowTiles * seg_rg + rt) * kTileRows + 16 * kg + (fl & 15);
        if (kWideRowTiles * seg_rg + rt < p.ntile) {  // uniform for the wave
            f32x4 v[NB];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    v[nb][j] = (kg ? acc[nb][1][j] : acc[nb][0][j]) + there[(4 * nb + j) * 64];
            wide_store<NB>(p, cols, v, row, fl >> 4, arrivals);
        }
        // (what the others hand over is read before they reach the next barrier, and the buffer is not filled before that)
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // nothing is on its way to LDS when a wave ends
}

// ---------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------
int compute_units()
{
    constexpr int kMaxDevices = 64;
    static std::atomic<int> cached[kMaxDevices];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 256;
    int cus = cached[dev].load(std::memory_order_relaxed);
    if (cus == 0) {
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) cus = 256;
        cached[dev].store(cus, std::memory_order_relaxed);
    }
    return cus;
}

// Workgroups: a whole number (`parts`) per row group, or one contiguous range of units each.  A range may end inside a row
// group, and then two row groups are added to the outputs, which costs about as much as half a unit; against a single
// workgroup per row group, which adds nothing but stores, about two units.  So ranges are taken if they have that much less
// for the workgroup with the most units (us, whole / ranges; units in parentheses).  One per row group, 8192 columns, 64
// vectors: 16512 rows 73.9 / 66.6 (8 / 5), 23040 rows 76.6 / 75.8 (8 / 6), 25600 rows 79.9 / 85.5 (8 / 7), 16512 x 4096 39.3 /
// 46.6 (4 / 3).  Several: 11008 x 8192 49.9 / 45.2 (4 / 3), 11008 x 28672, 32 vectors 85.2 / 71.2 (14 / 10), 8960 x 8192 41.7 / 48.1
// (3 / 3), 7168 x 28672 83.3 / 82.5 (7 / 7).
static void plan_wide(WideParams &wp, bool single_slice, int forced, int *groups)
{
    const int cus = compute_units(), rgs = wp.s.ntg;
    const long long units = (long long)rgs * wp.pairs;
    wp.s.units = (int)units;
    wp.parts = 0;
    const int parts = single_slice || rgs > cus ? 1 : (cus / rgs < wp.pairs ? cus / rgs : wp.pairs);
    const long long most_whole = (wp.pairs + parts - 1) / parts, most_ranges = (units + cus - 1) / cus;
    if (forced > 0) {
        *groups = (int)(forced < units ? forced : units);
    } else if (single_slice || (rgs <= cus && most_ranges + (parts == 1 ? 2 : 1) > most_whole)) {
        wp.parts = parts;
        *groups = rgs * parts;
    } else {
        *groups = (int)(cus < units ? cus : units);
    }
    wp.s.unit_base = (int)(units / *groups);
    wp.s.unit_rem = (int)(units % *groups);
}

template <int Q, int Z, int SUB, int NB>
static hipError_t launch_one(const WideParams &wp, int groups, hipStream_t stream)
{
    if constexpr (SUB == 1)
        hipLaunchKernelGGL((bcq_wide_kernel<Q, Z, NB>), dim3((unsigned)groups), dim3(64 * kWideWaves), 0, stream, wp);
    else
        hipLaunchKernelGGL((bcq_wide_groups_kernel<Q, Z, SUB, NB>), dim3((unsigned)groups), dim3(64 * kWideWaves), 0, stream, wp);
    return hipGetLastError();
}

// Column groups per pass: what fits 256 registers without spilling (0: less than two, not worth a pass).
constexpr int wide_most(int q, int z, int sub)
{
    if (q <= 2) return q == 2 && z == 1 && sub == 4 ? 3 : 4;
    if (q == 3) return z == 0 ? (sub == 1 ? 4 : 3) : (sub == 4 ? 2 : 3);
    return sub == 1 || (sub == 2 && z == 0) ? 2 : 0;
}

int wide_columns(const Geom &g) { return 16 * wide_most(g.q, g.z, g.sub); }

template <int Q, int Z, int SUB>
static hipError_t launch_sub(const WideParams &wp, int nb, int groups, hipStream_t stream)
{
    if constexpr (wide_most(Q, Z, SUB) >= 4) {
        if (nb == 4) return launch_one<Q, Z, SUB, 4>(wp, groups, stream);
    }
    if constexpr (wide_most(Q, Z, SUB) >= 3) {
        if (nb == 3) return launch_one<Q, Z, SUB, 3>(wp, groups, stream);
    }
    if constexpr (wide_most(Q, Z, SUB) >= 2) {
        if (nb == 2) return launch_one<Q, Z, SUB, 2>(wp, groups, stream);
    }
    return hipErrorInvalidValue;
}

template <int Q, int Z>
static hipError_t launch_qz(const WideParams &wp, int nb, int sub, int groups, hipStream_t stream)
{
    return sub == 1 ? launch_sub<Q, Z, 1>(wp, nb, groups, stream)
         : sub == 2 ? launch_sub<Q, Z, 2>(wp, nb, groups, stream) : launch_sub<Q, Z, 4>(wp, nb, groups, stream);
}

// p describes 17 to wide_columns() batch columns; workspace may be absent only for a single column slice.
hipError_t launch_wide(const Geom &g, const SkinnyParams &p, const GemvTuning &tuning, hipStream_t stream)
{
    WideParams wp;
    wp.s = p;
    wp.pairs = (g.nslice + 1) / 2;
    wp.s.ntg = (g.ntile + kWideRowTiles - 1) / kWideRowTiles;
    if ((long long)wp.s.ntg * wp.pairs > 0x7fffffffLL) return hipErrorInvalidValue;
    int groups;
    const int forced = tuning.skinny_parts > 0 ? tuning.skinny_parts * wp.s.ntg : tuning.workgroups;
    plan_wide(wp, p.accum == nullptr, p.accum == nullptr ? 0 : forced, &groups);
    const int nb = (p.batch + 15) / 16;
    switch (g.q * 2 + g.z) {
        case 2: return launch_qz<1, 0>(wp, nb, g.sub, groups, stream);
        case 3: return launch_qz<1, 1>(wp, nb, g.sub, groups, stream);
        case 4: return launch_qz<2, 0>(wp, nb, g.sub, groups, stream);
        case 5: return launch_qz<2, 1>(wp, nb, g.sub, groups, stream);
        case 6: return launch_qz<3, 0>(wp, nb, g.sub, groups, stream);
        case 7: return launch_qz<3, 1>(wp, nb, g.sub, groups, stream);
        case 8: return launch_qz<4, 0>(wp, nb, g.sub, groups, stream);
        case 9: return launch_qz<4, 1>(wp, nb, g.sub, groups, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace bcq
