// bcq_pack / bcq_unpack kernels: canonical operands of Eq. 11 (per-weight codes,
// alpha[M][G][q], offset[M][G]) <-> the tiled blob described in bcq_layout.h.
// Packing runs at the rate of memory (see pack_tile_kernel); unpacking is written for clarity.
#include "bcq_internal.h"

namespace bcq {

// A pack call covers the rows [row0, row0 + rows) of the layer; the call that reaches the last
// row also writes the padding rows.  `codes`, `alpha`, `offset` hold only the covered rows.
__device__ __forceinline__ bool row_is_mine(const Geom &g, int row, int row0, int rows)
{
    return row >= row0 && (row < row0 + rows || (row >= g.M && row0 + rows == g.M));
}

// Eight codes (a byte each) -> the eight bits of plane i, lowest column in bit 0: the bits as bytes, weighted and added.
__device__ __forceinline__ uint32_t plane_byte(uint2 v, int i)
{
    const uint32_t low = __builtin_amdgcn_udot4((v.x >> i) & 0x01010101u, 0x08040201u, 0u, false);
    return __builtin_amdgcn_udot4((v.y >> i) & 0x01010101u, 0x80402010u, low, false);
}

// One workgroup per tile of 32 rows x 512 columns: a thread owns one dword (four chunks of 8 columns) of a lane in every
// plane, so the codes are read once whatever the number of planes, in 8-byte loads that cover whole 512-byte row segments
// (ALIGNED: `codes` on 8 bytes; rows are multiples of 32 bytes), and then one scale entry at a time.  The loads of a thread
// are all under way together, not each behind the test whether its column exists.  Bound: memory.  28672
// x 7168, two planes with offset, one group per row: 117 us (a thread per dword and plane with byte loads, and a launch for
// the scales; 76 with loads behind branches) -> 56 us, 257 MB: 4.6 TB/s.  The row tiles come from the last to the first, all slices of
// one in turn: codes that have just been written are in the last-level cache from their end, and whole rows are read together:
// 56 -> 52 us behind the fusion (slice by slice over all rows before; the two together 135.5 -> 134.2, one tying for all rows 145.3 -> 136.5).
// Nontemporal loads, which share their lines with others: 75.
template <bool ALIGNED>
__global__ __launch_bounds__(256) void pack_tile_kernel(Geom g, int row0, int rows, const uint8_t *__restrict__ codes,
                                                        const uint16_t *__restrict__ alpha,
                                                        const uint16_t *__restrict__ offset, uint8_t *__restrict__ blob)
{
    const int from_end = blockIdx.x / (unsigned)g.nslice, slice = blockIdx.x - (unsigned)from_end * (unsigned)g.nslice;
    const int tile = g.ntile - 1 - from_end;
    uint8_t *const out = blob + tile_offset(g, slice, tile);
    uint2 v[2][4];  // all requested before the first is used; what does not exist is zero
    bool mine[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int idx = threadIdx.x + 256 * k, d = idx & 3, lane = (idx >> 2) & 63, t = idx >> 8;
        const int r = lane & 15, h = lane >> 4;
        const int row = kTileRows * tile + 16 * t + r, kb = 4 * slice + h;
        mine[k] = row_is_mine(g, row, row0, rows);
#pragma unroll
        for (int n = 0; n < 4; ++n) {
            const int col = kBlockCols * kb + kChunkCols * chunk_of_byte(4 * d + n, r, g.sub);
            const bool ok = mine[k] && row < g.M && col < g.N;
            const uint8_t *src = codes + (ok ? (size_t)(row - row0) * g.N + col : 0);
            uint2 c;
            if (ALIGNED) {
                c = *reinterpret_cast<const uint2 *>(src);
            } else {
                c.x = src[0] | src[1] << 8 | src[2] << 16 | (uint32_t)src[3] << 24;
                c.y = src[4] | src[5] << 8 | src[6] << 16 | (uint32_t)src[7] << 24;
            }
            v[k][n] = ok ? c : uint2{0u, 0u};
        }
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int idx = threadIdx.x + 256 * k, d = idx & 3, lane = (idx >> 2) & 63, t = idx >> 8;
        if (!mine[k]) continue;
#pragma unroll
        for (int i = 0; i < kMaxQ; ++i)
            if (i < g.q)
                *reinterpret_cast<uint32_t *>(out + ((size_t)((t * g.q + i) * 64 + lane) * 16 + 4 * d)) =
                    plane_byte(v[k][0], i) | plane_byte(v[k][1], i) << 8 | plane_byte(v[k][2], i) << 16 | plane_byte(v[k][3], i) << 24;
    }
    const unsigned per_tile = (unsigned)g.scale_lanes * 2u * g.nsc;  // with 16 records per half tile, `lane` below is the row
    const unsigned qz = g.q + g.z, G = g.N / g.group;
    for (unsigned e = threadIdx.x; e < per_tile; e += 256) {
        const unsigned lane = e / (2 * g.nsc), rr = e - lane * (2 * g.nsc);
        const unsigned t = rr / g.nsc, sc = rr - t * g.nsc;
        const unsigned range = sc / qz, c = sc - range * qz;
        const int r = lane & 15, h = lane >> 4;
        const int row = kTileRows * tile + 16 * t + r;
        if (!row_is_mine(g, row, row0, rows)) continue;
        const int col = kBlockCols * (4 * slice + h) + subgroup_of_range(range, r, g.sub) * (kBlockCols / g.sub);
        uint16_t val = 0;
        if (row < g.M && col < g.N) {
            const size_t at = (size_t)(row - row0) * G + (unsigned)col / (unsigned)g.group;
            val = c < (unsigned)g.q ? alpha[at * g.q + c] : offset[at];
        }
        *reinterpret_cast<uint16_t *>(out + g.tile_plane_bytes + (size_t)e * 2) = val;
    }
}

__global__ void unpack_codes_kernel(Geom g, const uint8_t *__restrict__ blob,
                                    uint8_t *__restrict__ codes)
{
    size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= (size_t)g.M * g.N) return;
    int row = (int)(gid / g.N), col = (int)(gid % g.N);
    int slice = col / kTileCols, h = (col % kTileCols) / kBlockCols;
    int c = (col % kBlockCols) / kChunkCols, bit = col % kChunkCols;
    int tile = row / kTileRows, t = (row % kTileRows) / 16, r = row % 16;
    int j = byte_of_chunk(c, r, g.sub);
    const uint8_t *base = blob + tile_offset(g, slice, tile);
    uint8_t code = 0;
    for (int i = 0; i < g.q; ++i) {
        uint8_t byte = base[(size_t)((t * g.q + i) * 64 + 16 * h + r) * 16 + j];
        code |= (uint8_t)(((byte >> bit) & 1) << i);
    }
    codes[gid] = code;
}

__global__ void unpack_scales_kernel(Geom g, const uint8_t *__restrict__ blob,
                                     uint16_t *__restrict__ alpha, uint16_t *__restrict__ offset)
{
    size_t G = g.N / g.group;
    size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= (size_t)g.M * G) return;
    int row = (int)(gid / G);
    int col = (int)(gid % G) * g.group;           // first column of the group
    int slice = col / kTileCols, h = (col % kTileCols) / kBlockCols;
    int tile = row / kTileRows, t = (row % kTileRows) / 16, r = row % 16;
    // subgroup_of_range is its own inverse in its first argument
    int range = subgroup_of_range((col % kBlockCols) / (kBlockCols / g.sub), r, g.sub);
    int lane = (16 * h + r) & (g.scale_lanes - 1), qz = g.q + g.z;
    const uint16_t *src = reinterpret_cast<const uint16_t *>(
        blob + tile_offset(g, slice, tile) + g.tile_plane_bytes) +
        (size_t)lane * 2 * g.nsc + (size_t)t * g.nsc + (size_t)range * qz;
    if (alpha)
        for (int c = 0; c < g.q; ++c) alpha[gid * g.q + c] = src[c];
    if (offset && g.z) offset[gid] = src[g.q];
}

__global__ void fill_zero_kernel(uint32_t *p, size_t n)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = 0u;
}

static unsigned blocks_for(size_t n, unsigned threads)
{
    return (unsigned)((n + threads - 1) / threads);
}

hipError_t launch_pack(const Geom &g, int row0, int rows, const uint8_t *codes, const uint16_t *alpha,
                       const uint16_t *offset, void *packed, hipStream_t stream)
{
    const size_t tiles = (size_t)g.nslice * g.ntile;
    const bool aligned = (reinterpret_cast<uintptr_t>(codes) & 7) == 0;
    hipLaunchKernelGGL((aligned ? pack_tile_kernel<true> : pack_tile_kernel<false>), dim3((unsigned)tiles), dim3(256), 0, stream, g,
                       row0, rows, codes, alpha, offset, static_cast<uint8_t *>(packed));
    return hipGetLastError();
}

hipError_t launch_unpack(const Geom &g, const void *packed, uint8_t *codes, uint16_t *alpha,
                         uint16_t *offset, hipStream_t stream)
{
    const uint8_t *blob = static_cast<const uint8_t *>(packed);
    if (codes) {
        size_t n = (size_t)g.M * g.N;
        hipLaunchKernelGGL(unpack_codes_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, stream, g,
                           blob, codes);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (alpha || offset) {
        size_t n = (size_t)g.M * (g.N / g.group);
        hipLaunchKernelGGL(unpack_scales_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, stream, g,
                           blob, alpha, offset);
    }
    return hipGetLastError();
}

hipError_t launch_fill_zero(void *ptr, size_t bytes, hipStream_t stream)
{
    size_t n = bytes / 4;
    if (n == 0) return hipSuccess;
    unsigned blocks = blocks_for(n, 256);
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(fill_zero_kernel, dim3(blocks), dim3(256), 0, stream,
                       static_cast<uint32_t *>(ptr), n);
    return hipGetLastError();
}

}  // namespace bcq
