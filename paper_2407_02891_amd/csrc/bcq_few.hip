// Binary-coding product with two to four activation vectors (paper Eq. 11) for gfx950, one scaling group per 128-column block.
//
//   y_v[m] = sum_blocks sum_i alpha_i[m,blk] * S_i,v[m,blk]  (+ z[m,blk] * X_v[blk])
//
// The sums over the signs are formed by the 8-bit integer matrix instruction, exactly: v_mfma_i32_16x16x64_i8 with the sign bits
// masked in place as one operand and the activations' digits as the other (bcq_digits.h, which says what the digits round).  Four vectors of
// four digits are the sixteen rows of that operand, and lane 16 h + r of the result holds the four digits of vector h's sum for weight row r:
// two additions, two conversions and an FMA make it a binary32 number.  A sign costs 9/32 of a vector instruction and no table.
//
//  * A wave owns one column slice of 512: its activations are made into digits once and stay in 48 registers, and it streams
//    the slice's row tiles, which are contiguous in the blob, a tile ahead.  There is no barrier in that stream.
//  * The four lanes that hold the four blocks of a row exchange dwords through a wave-private piece of LDS (one 16-byte
//    write and four 4-byte reads per plane and row half), which undoes the dword part of the blob's byte rotation on the way:
//    four vector instructions where selects and lane swaps take sixteen (9216 x 36864, q = 3: 31.5 -> 30.6 us).
//  * A workgroup has up to twelve waves (168 registers: three per SIMD; a lone wave issues a vector instruction every 8 clocks, two or
//    three one every 4): neighbouring slices of the same rows, and where these are few, several groups of rows.  Their sums of
//    8 or 16 half tiles (few_chunk) meet in LDS; what leaves the workgroup is one number per row and vector, stored if the workgroup has all slices,
//    else added to the row's fixed-point accumulator (encode_partial_f32), whose last contributor stores it.
//  * What a launch costs besides its steps is the digits (about 120 vector instructions per vector and wave), so how many waves share the
//    work is a compromise (plan_few).
//
// Bound: vector instructions (about 215 per half tile with three planes, 24 matrix instructions; with the loads taken out of the loop a launch
// on 7168 x 28672 is 2 us shorter, of 22).  Measured against the kernels that took these calls before (us, four vectors, graph replay): 9216 x 36864
// q = 3 38.8 -> 32.6, 7168 x 28672 25.9 -> 21.8, 28672 x 7168 26.0 -> 24.8, 28083 x 10208 with a scale per row 33.6 -> 29.2, 7168 x 7168 11.6 -> 10.4,
// 2048 x 4096 q = 2 5.9 -> 4.9, 512 x 512 4.9 -> 4.3; two vectors 4096 x 4096 7.1 -> 5.8, 512 x 512 4.8 -> 3.8.  All eight signs of a byte masked without a
// shift is 0 to 2 % faster (9216 x 36864 32.2, 7168 x 7168 10.1), but takes 2^7 from the digits' range instead of 2^3: with 22 bits of activations
// the error where a loud column cancels was ten times that of a sum in binary32, and is a quarter of it now.  Tried: signs from a table of 8-byte entries in LDS with three digits and a third fewer
// vector instructions: 40.4 / 27.2 us on the two large layers (30.6 / 22.1 this way, eager); eight vectors per wave: 34 against 28 us there; the activations
// of a lane strided so that the digits need no exchange between lanes: 1 to 3 % slower; the additions of two or four half tiles of a wave's share of a meeting
// under way at once: 7168 x 28672 the same, small layers 3 to 20 % slower (registers go to scratch).
#include <atomic>

#include "bcq_internal.h"
#include "bcq_skinny.h"
#include "bcq_digits.h"

namespace bcq {

namespace {

constexpr int kFewWaves = 12, kFewBatch = 4;
constexpr int kFewX = 8192;            // bytes of a slice's digits: [block][half of the bits][lane] 16 bytes

struct FewParams {
    const uint8_t *blob;
    const uint16_t *X;
    uint16_t *Y;
    unsigned long long *accum;  // [batch][Mp]
    int M, N, Mp, batch, ldx, ldy;
    int ntile, nslice;
    int ranges;                 // workgroups that share a row
    int slices;                 // slices of a workgroup (one may be missing); its waves are whole groups of that many
    int part_base, part_rem;    // half tiles per group of waves: part_base, the first part_rem one more
    unsigned tile_bytes;
    int scale_lane_mask;        // 63: one scale record per lane; 15: one per row (group = N)
};

// Half tiles between two meetings of a workgroup's waves, of at most `most`.  With more than four waves there is one workgroup per compute
// unit, which stands still meanwhile (8 / 16, us, four vectors: 7168 x 28672 23.1 / 21.7, 9216 x 36864 33.0 / 31.9, 28672 x 8192 q = 2 with offset 20.2 / 19.3);
// several of them fill each other's pauses, and their additions are better spread (28672 x 7168 25.5 / 25.9).
constexpr int few_chunk(int waves, int most) { return waves > 4 && most > 8 ? 16 : 8; }
// LDS of a workgroup of `waves` waves; a scale per (wave, block, vector), static, beside it.
constexpr size_t few_lds_bytes(int waves, int chunk) { return (size_t)waves * (kFewX + chunk * 256); }
static_assert(few_lds_bytes(kFewWaves, 16) + kFewWaves * 64 <= 160 * 1024, "one workgroup per compute unit");

}  // namespace

// V: vectors made into digits, 2 or 4; the operand's other rows are not looked at.  CHUNK: half tiles between two meetings of the waves.
template <int Q, int Z, int V, int CHUNK>
__global__ __launch_bounds__(64 * kFewWaves) void bcq_few_kernel(FewParams p)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t few_lds[];
    __shared__ float block_scale[kFewWaves][4][4];  // [wave][block][vector]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int waves = blockDim.x >> 6;
    const int r = lane & 15, h = lane >> 4;
    uint8_t *const xs = few_lds + wave * kFewX;
    float *const partial = reinterpret_cast<float *>(few_lds + waves * kFewX);

    // this wave: slice `slice`, half tiles [h_begin, h_end)
    const int range = blockIdx.x % p.ranges, row_groups = waves / p.slices, first_part = blockIdx.x / p.ranges * row_groups;
    const int s_begin = (int)((long long)range * p.nslice / p.ranges), s_end = (int)((long long)(range + 1) * p.nslice / p.ranges);
    const int slice = s_begin + wave % p.slices;
    const bool mine = slice < s_end;
    const auto first_half = [&](int part) { return part * p.part_base + min(part, p.part_rem); };
    const int h_begin = first_half(first_part + wave / p.slices), h_end = first_half(first_part + wave / p.slices + 1);
    const int most = p.part_base + (first_part < p.part_rem ? 1 : 0);  // of the workgroup's waves
    const int scale_lane = lane & p.scale_lane_mask;

    // ---- activations requested, then the first tile ----
    const int col = slice * kTileCols + kChunkCols * lane;  // lane = chunk
    const bool have = mine && col < p.N;
    u32x4 xr[V];
#pragma unroll
    for (int v = 0; v < V; ++v)
        xr[v] = *reinterpret_cast<const u32x4 *>(p.X + (size_t)(v < p.batch ? v : 0) * p.ldx + (have ? col : 0));
    const uint8_t *const column = p.blob + (size_t)(mine ? slice : 0) * p.ntile * p.tile_bytes;
    u32x4 raw[2][Q];
    uint32_t rec[2][Q + Z];
    // a half tile's signs and its tile's scale record, or zeros without touching memory
    const auto request = [&](int half, u32x4 (&w)[Q], uint32_t (&e)[Q + Z]) {
        constexpr int kNonTemporal = 2;
        const bool ok = mine && half < h_end;
        uint8_t *const tile = const_cast<uint8_t *>(column) + (size_t)(ok ? half >> 1 : 0) * p.tile_bytes;
        const __amdgpu_buffer_rsrc_t signs =
            __builtin_amdgcn_make_buffer_rsrc(tile + (half & 1) * (Q * 1024), 0, ok ? Q * 1024 : 0, kRawBufferFlags);
        const __amdgpu_buffer_rsrc_t scales =
            __builtin_amdgcn_make_buffer_rsrc(tile + 2 * Q * 1024, 0, ok ? (int)(p.tile_bytes - 2 * Q * 1024) : 0, kRawBufferFlags);
#pragma unroll
        for (int i = 0; i < Q; ++i) w[i] = __builtin_amdgcn_raw_buffer_load_b128(signs, 16u * lane + i * 1024u, 0, kNonTemporal);
#pragma unroll
        for (int c = 0; c < Q + Z; ++c)
            e[c] = __builtin_amdgcn_raw_buffer_load_b32(scales, 4u * (Q + Z) * scale_lane + 4u * c, 0, kNonTemporal);
    };
    request(h_begin, raw[0], rec[0]);
    request(h_begin + 1, raw[1], rec[1]);

    // ---- digits: lane (block h, chunk r) writes, for vector v, what lane group r div 4 of X row 4 v + r mod 4 reads ----
    uint32_t digits[V][8];
    float own_scale[V];
#pragma unroll
    for (int v = 0; v < V; ++v)
        if (!have || v >= p.batch) xr[v] = u32x4{0u, 0u, 0u, 0u};
    block_digits<V>(xr, digits, own_scale);
#pragma unroll
    for (int v = 0; v < V; ++v) {
        uint8_t *const dst = xs + (h * 128 + (r >> 2) * 16 + 4 * v + (r & 3)) * 16;
#pragma unroll
        for (int b = 0; b < 8; ++b) digits[v][b] = transpose_quad(digits[v][b], lane);
        *reinterpret_cast<u32x4 *>(dst) = u32x4{digits[v][0], digits[v][1], digits[v][2], digits[v][3]};
        *reinterpret_cast<u32x4 *>(dst + 1024) = u32x4{digits[v][4], digits[v][5], digits[v][6], digits[v][7]};
    }
    if (r == 0) {
#pragma unroll
        for (int v = 0; v < V; ++v) block_scale[wave][h][v] = own_scale[v];
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // (one wave wrote and reads all of it)
    // this lane's vector is h
    i32x4 X[4][2], start[4];
    float scale[4], xsum[Z ? 4 : 1];
#pragma unroll
    for (int B = 0; B < 4; ++B) {
        scale[B] = block_scale[wave][B][h];
        X[B][0] = *reinterpret_cast<const i32x4 *>(xs + (B * 128 + lane) * 16);
        X[B][1] = *reinterpret_cast<const i32x4 *>(xs + (B * 128 + 64 + lane) * 16);
    }
#pragma unroll
    for (int B = 0; B < 4; ++B) {  // all bits set: the digits of S
        const i32x4 all = masked_signs(0x0f0f0f0fu);
        i32x4 S = __builtin_amdgcn_mfma_i32_16x16x64_i8(X[B][0], all, i32x4{0, 0, 0, 0}, 0, 0, 0);
        S = __builtin_amdgcn_mfma_i32_16x16x64_i8(X[B][1], all, S, 0, 0, 0);
        start[B] = start_digits(S);
        if (Z) xsum[Z ? B : 0] = 0.5f * digit_value(S);
    }

    // The blob's rotation (chunk_of_byte): chunk c of the block is byte (c - r) mod 16, so dword d in chunk order is dword (d + k div 4) mod 4 of the
    // 16 bytes turned by k mod 4, k = -r mod 16.
    const int k = (16 - r) & 15;
    const uint32_t turn = k & 3;
    const int from = r * 16 + ((h + (k >> 2)) & 3) * 4;

    for (int done = 0; done < most; done += CHUNK) {
        const int c_end = min(h_end, h_begin + done + CHUNK);
        for (int half = h_begin + done; half < c_end; half += 2) {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                if (half + t >= c_end) break;
                // scales of this half, one copy of every lane group's in every lane group
                uint32_t sc[4][(Q + Z + 1) / 2];
                {
                    uint32_t own[Q + Z + 1];
                    own[Q + Z] = 0;
#pragma unroll
                    for (int c = 0; c < Q + Z; ++c) {
                        const int e0 = c, e1 = (Q + Z) + c;
                        const uint32_t first = (e0 & 1) ? rec[t][e0 >> 1] >> 16 : rec[t][e0 >> 1] & 0xffffu;
                        const uint32_t second = (e1 & 1) ? rec[t][e1 >> 1] >> 16 : rec[t][e1 >> 1] & 0xffffu;
                        own[c] = ((half + t) & 1) ? second : first;
                    }
#pragma unroll
                    for (int k = 0; k < (Q + Z + 1) / 2; ++k) {
                        const uint32_t v = own[2 * k] | (own[2 * k + 1] << 16);
                        const auto lo_hi = __builtin_amdgcn_permlane32_swap(v, v, false, false);
                        const unsigned lo = lo_hi[0], hi = lo_hi[1];
                        const auto g01 = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
                        const auto g23 = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
                        sc[0][k] = g01[0]; sc[1][k] = g01[1]; sc[2][k] = g23[0]; sc[3][k] = g23[1];
                    }
                }
                // wb[i][B] = chunks 4 h .. 4 h + 3 of (row r of the half, block B, plane i)
                uint32_t wb[Q][4];
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    const u32x4 w = raw[t][i];
                    uint8_t *const slot = xs + (t * Q + i) * 1024;  // (the digits are in registers)
                    *reinterpret_cast<u32x4 *>(slot + lane * 16) =
                        u32x4{__builtin_amdgcn_alignbyte(w.y, w.x, turn), __builtin_amdgcn_alignbyte(w.z, w.y, turn),
                              __builtin_amdgcn_alignbyte(w.w, w.z, turn), __builtin_amdgcn_alignbyte(w.x, w.w, turn)};
#pragma unroll
                    for (int B = 0; B < 4; ++B) wb[i][B] = *reinterpret_cast<const uint32_t *>(slot + 256 * B + from);
                }
                request(half + t + 2, raw[t], rec[t]);
                float y = 0.0f;
#pragma unroll
                for (int B = 0; B < 4; ++B) {
                    i32x4 acc[Q];
#pragma unroll
                    for (int bits = 0; bits < 2; ++bits)
#pragma unroll
                        for (int i = 0; i < Q; ++i)
                            acc[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(X[B][bits], masked_signs(bits ? wb[i][B] >> 4 : wb[i][B]),
                                                                          bits == 0 ? start[B] : acc[i], 0, 0, 0);
                    float yb = 0.0f;
#pragma unroll
                    for (int c = 0; c < Q + Z; ++c) {
                        const uint32_t pair = sc[B][c >> 1];
                        const float a = half_bits_to_float((c & 1) ? pair >> 16 : pair & 0xffffu);
                        yb = fmaf(a, c < Q ? digit_value(acc[c < Q ? c : 0]) : xsum[Z ? B : 0], yb);
                    }
                    y = fmaf(yb, scale[B], y);
                }
                partial[((half + t - h_begin - done) * waves + wave) * 64 + lane] = y;
            }
        }
        __syncthreads();
        // one number per row and vector: item = [group of waves][half tile][vector][row]
        const int each = min(CHUNK, most - done) * 64;
        for (int item = tid; item < row_groups * each; item += (int)blockDim.x) {
            const int group = item / each, e = item - group * each;
            const int half = first_half(first_part + group) + done + (e >> 6);
            const int v = (e >> 4) & 3, row = 16 * half + (e & 15);
            if (v >= p.batch || half >= first_half(first_part + group + 1)) continue;
            const float *src = partial + ((e >> 6) * waves + group * p.slices) * 64 + (e & 63);
            float sum = 0.0f;
            for (int w = 0; w < s_end - s_begin; ++w) sum += src[w * 64];
            if (p.ranges == 1) {
                if (row < p.M) p.Y[(size_t)v * p.ldy + row] = float_to_half_bits(sum);
            } else {
                unsigned long long *const word = p.accum + (size_t)v * p.Mp + row;
                const unsigned long long add = encode_partial_f32(sum);
                const unsigned long long total = add + __hip_atomic_fetch_add(word, add, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (arrivals_of(total) == (unsigned)p.ranges) {
                    if (row < p.M) p.Y[(size_t)v * p.ldy + row] = float_to_half_bits(decode_total(total));
                    __hip_atomic_store(word, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        }
        if (done + CHUNK < most) __syncthreads();
    }
}

// ---------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------
bool few_applies(const Geom &g, int batch, const void *workspace)
{
    // One plane on one column slice: a wave has so few steps that what it does once, the digits above all, is the larger part, with two vectors as soon
    // as one wave per SIMD does not do with a half tile each.  us here / there (bcq_skinny.hip): two vectors 2885 x 512 3.6 / 4.0, 8483 x 512 3.6 / 4.3,
    // 14869 x 512 3.8 / 4.2, 19085 x 512 4.3 / 4.2, 40487 x 512 5.0 / 4.8; three and four 3733 x 512 4.1 / 3.9, 10967 x 384 4.1 / 3.9, 17301 x 512 4.7 / 4.3,
    // 52847 x 512 6.1 / 5.1.
    // With more slices this kernel is as fast or faster (60 layers of 20 to 72 slices and 4096 to 36864 rows: 0.77 to 1.03 of the time there).
    if (g.q == 1 && g.nslice == 1 && (batch > 2 || g.ntile > 2 * compute_units())) return false;
    // (split-K accumulators unless the layer is a single slice)
    return batch >= 2 && batch <= kFewBatch && g.sub == 1 && (workspace != nullptr || g.nslice == 1);
}

namespace {

// Time of a launch in us: what it takes with so many waves on the fullest SIMD before the first half tile is done, a step with three planes, a
// second workgroup on a row, a million additions to the accumulators, and waves that wait for eight or more others.  Only which plan is
// least matters.  Over all plans of 378 layers (one to four planes, 1 to 72 slices, 512 to 36864 rows, two and four vectors) the one chosen takes 1.00 to 1.02 of
// the best one's time in the middle, 1.06 to 1.11 in nine of ten, 1.24 at worst (1152 row tiles and 5 or 11 slices).  Without the term for four planes six of
// those layers change, five of them to plans 2 to 7 % slower; without the one for eight waves 28, most of them slower, by up to 10 %.
constexpr double kFewBase[4] = {0, 2.7, 3.5, 3.6}, kFewStep[4] = {0, 1.04, 1.48, 2.15}, kFewJoin = 0.8, kFewAdditions = 2.5, kFewCrowd = 0.5;

struct FewPlan {
    int ranges, slices, row_groups, parts;  // parts: groups of waves per range
};

FewPlan plan_few(const Geom &g, int batch, int forced)
{
    const unsigned cus = compute_units(), halves = (g.M + 15LL) / 16, nslice = g.nslice;
    FewPlan best = {g.nslice, 1, 1, 1};
    double least = 1e300;
    const double planes = (g.q + 0.2 * g.z + 0.5) / 3.5, half_tiles = halves;
    for (unsigned most = kFewWaves; most >= 1; --most) {
        const unsigned ranges = (nslice + most - 1) / most, slices = (nslice + ranges - 1) / ranges;
        if (slices < most) continue;
        unsigned room[3];  // workgroups per range
        for (unsigned per_cu = 1; per_cu <= 3; ++per_cu) {
            room[per_cu - 1] = (forced > 0 ? (unsigned)forced : cus * per_cu) / ranges;
            if (forced > 0 && room[per_cu - 1] < 1) room[per_cu - 1] = 1;
        }
        const double join = ranges > 1 ? kFewJoin + kFewAdditions * 1e-6 * ranges * g.M * batch : 0.0;
        for (unsigned row_groups = 1; row_groups * slices <= kFewWaves; ++row_groups) {
            const unsigned waves = row_groups * slices, enough = (halves + row_groups - 1) / row_groups;
            for (unsigned per_cu = 1; per_cu * ((waves + 3) / 4) <= 3; ++per_cu) {
                if (per_cu > 1 && room[per_cu - 2] >= enough) break;  // no more workgroups
                const unsigned groups = room[per_cu - 1] < enough ? room[per_cu - 1] : enough;
                if (groups < 1) continue;
                // steps: the mean counts too, only some of a compute unit's waves take one more
                const double mean = half_tiles / (groups * row_groups);
                const unsigned whole = (unsigned)mean;
                const double steps = 0.3 * mean + 0.7 * (whole + (mean > whole ? 1 : 0));
                const unsigned simd = per_cu * ((waves + 3) / 4);
                double cost = kFewBase[simd] + kFewStep[simd] * steps * planes + join;
                if (waves > 8) cost += kFewCrowd;
                if (g.q == 4 && simd == 3) cost += 0.3 * steps;  // (4096 x 28672: 8 steps of two 20.2, 5 of three 21.1)
                if (cost < least) {
                    least = cost;
                    best = {(int)ranges, (int)slices, (int)row_groups, (int)(groups * row_groups)};
                }
            }
        }
    }
    return best;
}

// The last plans of the calling thread: choosing one takes 0.13 to 0.3 us of the host, which a launch of a small layer waits for (512 x 512, four vectors,
// eager calls 5.65 us, 5.5 with the plan at hand).  `dev`: the current device, whose compute units count.
FewPlan kept_plan(const Geom &g, int batch, int forced, int dev)
{
    struct Entry {
        int M, nslice, planes, batch, forced, dev;
        FewPlan plan;
    };
    constexpr unsigned kEntries = 64;
    static thread_local Entry entries[kEntries];  // (zeros: no layer has no rows)
    const int planes = 2 * g.q + g.z;
    Entry &e = entries[((unsigned)g.M * 0x9e3779b1u + (unsigned)(g.nslice * 64 + planes * 4 + batch) * 0x85ebca6bu) >> 26];
    if (e.M != g.M || e.nslice != g.nslice || e.planes != planes || e.batch != batch || e.forced != forced || e.dev != dev)
        e = {g.M, g.nslice, planes, batch, forced, dev, plan_few(g, batch, forced)};
    return e.plan;
}

// `dev`: the current device, or -1 if it is not known or has a number from kFewDevices on.
constexpr int kFewDevices = 64;

template <int Q, int Z, int V, int CHUNK>
hipError_t launch_few_v(const FewParams &p, int waves, int groups, int dev, hipStream_t stream)
{
    const size_t lds = few_lds_bytes(waves, CHUNK);
    // more LDS than a launch gets by itself: asked for once per device
    static std::atomic<bool> asked[kFewDevices];
    if (dev < 0 || !asked[dev].load(std::memory_order_relaxed)) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(bcq_few_kernel<Q, Z, V, CHUNK>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)few_lds_bytes(kFewWaves, CHUNK));
        if (e != hipSuccess) return e;
        if (dev >= 0) asked[dev].store(true, std::memory_order_relaxed);
    }
    hipLaunchKernelGGL((bcq_few_kernel<Q, Z, V, CHUNK>), dim3((unsigned)groups), dim3(64 * waves), lds, stream, p);
    return hipGetLastError();
}

template <int Q, int Z>
hipError_t launch_few_qz(const FewParams &p, int waves, int groups, int dev, hipStream_t stream)
{
    const int chunk = few_chunk(waves, p.part_base + (p.part_rem > 0 ? 1 : 0));
    if (p.batch == 2)
        return chunk == 8 ? launch_few_v<Q, Z, 2, 8>(p, waves, groups, dev, stream) : launch_few_v<Q, Z, 2, 16>(p, waves, groups, dev, stream);
    return chunk == 8 ? launch_few_v<Q, Z, 4, 8>(p, waves, groups, dev, stream) : launch_few_v<Q, Z, 4, 16>(p, waves, groups, dev, stream);
}

}  // namespace

hipError_t launch_few(const Geom &g, const void *packed, const uint16_t *X, int ldx, uint16_t *Y, int ldy, int batch, void *workspace,
                      const GemvTuning &tuning, hipStream_t stream)
{
    if (!few_applies(g, batch, workspace)) return hipErrorInvalidValue;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kFewDevices) dev = -1;
    const FewPlan plan = dev < 0 ? plan_few(g, batch, tuning.workgroups) : kept_plan(g, batch, tuning.workgroups, dev);
    const int halves = (int)((g.M + 15LL) / 16), waves = plan.slices * plan.row_groups;
    FewParams p;
    p.blob = static_cast<const uint8_t *>(packed);
    p.X = X; p.Y = Y;
    p.accum = static_cast<unsigned long long *>(workspace);
    p.M = g.M; p.N = g.N; p.Mp = g.Mp; p.batch = batch; p.ldx = ldx; p.ldy = ldy;
    p.ntile = g.ntile; p.nslice = g.nslice;
    p.ranges = plan.ranges;
    p.slices = plan.slices;
    p.part_base = halves / plan.parts; p.part_rem = halves % plan.parts;
    p.tile_bytes = g.tile_bytes;
    p.scale_lane_mask = g.scale_lanes - 1;
    const int groups = plan.ranges * (plan.parts / plan.row_groups);
    switch (g.q * 2 + g.z) {
        case 2: return launch_few_qz<1, 0>(p, waves, groups, dev, stream);
        case 3: return launch_few_qz<1, 1>(p, waves, groups, dev, stream);
        case 4: return launch_few_qz<2, 0>(p, waves, groups, dev, stream);
        case 5: return launch_few_qz<2, 1>(p, waves, groups, dev, stream);
        case 6: return launch_few_qz<3, 0>(p, waves, groups, dev, stream);
        case 7: return launch_few_qz<3, 1>(p, waves, groups, dev, stream);
        case 8: return launch_few_qz<4, 0>(p, waves, groups, dev, stream);
        case 9: return launch_few_qz<4, 1>(p, waves, groups, dev, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace bcq
