// The GPTQT quantiser for one linear layer with row-wise parameters (paper Sec. II-A Eq. 1-2,
// Sec. II-B Eq. 5-6, Sec. II-C Eq. 7 and the algorithm that closes Sec. II-D), the step that
// produces what bcq_from_linear_rows / bcq_pack consume.  All reduction orders are fixed: the same inputs give the same bits.
//
//   search   per row m: qbias = min w, range = max w - min w; for S' on `grid` equidistant points
//            inside (range / (2^(n+1) - 1), range / (2^(n-1) - 1))  (Eq. 7), for every way of tying
//            the n linear bit-planes into q classes (Eq. 10): W_q = nearest member of that tying's
//            BCchoice to clamp(rne((w - qbias) / S'))  (Eq. 5 step 1, Eq. 6), output error
//            e = d (H / 2) d^T with d = S' W_q + qbias - w  (Eq. 5 step 2); the first candidate
//            with the smallest error is kept (scale-major order).
//   gptq     column by column, quant(w) = S W_q + qbias with the row's parameters; the error of
//            column j, divided by U[j][j], is spread over the later columns along row j of U, the
//            upper Cholesky factor of H^-1 (Eq. 2 in its usual one-factorisation form).
//
// The integer decisions (rounding to the linear grid, nearest BCchoice) are those of binary64 copies of the binary32
// inputs (the GPTQ pass takes them from binary32 where that cannot tell otherwise); the quadratic form and the GPTQ updates accumulate in binary32
// (the dense products with operands split into pairs of binary16 numbers, see bcq_product.h).
#include <algorithm>
#include <vector>

#include "bcq_internal.h"
#include "bcq_device.h"
#include "bcq_product.h"
#include "bcq_screen.h"
#include "bcq_tying.h"

namespace bcq {

// One way of tying the planes: class of every bit, and the integers it can represent (ascending).
struct Tying {
    int8_t label[kMaxBits];
    int nchoice;
    int choice[16];
    unsigned long long nibbles;  // up to four bits: nearest choice of every integer
};

// All partitions of the planes 1..n into q non-empty classes; classes ordered by their smallest
// plane, partitions ordered lexicographically by their classes (shorter class first on a tie of
// the common prefix).
static std::vector<Tying> all_tyings(int n, int q)
{
    std::vector<std::vector<std::vector<int>>> parts;
    std::vector<int> lab(n, 0);
    // restricted growth strings: lab[0] = 0, lab[i] <= 1 + max(lab[0..i-1])
    std::vector<int> stack;
    struct Rec {
        static void go(int i, int n, int q, int used, std::vector<int> &lab,
                       std::vector<std::vector<std::vector<int>>> &out)
        {
            if (i == n) {
                if (used != q) return;
                std::vector<std::vector<int>> p(q);
                for (int k = 0; k < n; ++k) p[lab[k]].push_back(k + 1);
                out.push_back(p);
                return;
            }
            for (int c = 0; c <= used && c < q; ++c) {
                lab[i] = c;
                go(i + 1, n, q, c == used ? used + 1 : used, lab, out);
            }
        }
    };
    Rec::go(0, n, q, 0, lab, parts);
    std::sort(parts.begin(), parts.end());
    std::vector<Tying> out;
    for (const auto &p : parts) {
        Tying t{};
        for (int c = 0; c < q; ++c)
            for (int plane : p[c]) t.label[plane - 1] = (int8_t)c;
        TyingPlan plan;
        make_tying_plan(n, q, t.label, false, &plan);
        t.nchoice = plan.nchoice;
        std::copy(plan.choice, plan.choice + plan.nchoice, t.choice);
        for (int w = 0; n <= 4 && w < 1 << n; ++w) t.nibbles |= (unsigned long long)nearest_choice(w, t.choice, t.nchoice) << (4 * w);
        out.push_back(t);
    }
    return out;
}

// Eq. 5 step 1 for one weight, in binary64: clamp(rne(x / S)), x = w - qbias.  The product with inv_s = 1 / S is off by less
// than 2^-44 for the up to 2^8 steps of the grid, so it rounds to the same integer as the quotient unless it lies within
// 2^-30 of a half; then the division is carried out.
__device__ __forceinline__ int linear_int(double x, double S, double inv_s, double top)
{
    const double t = x * inv_s;
    double v = rint(t);  // round half to even
    if (__builtin_expect(!(fabs(t - v) < 0.5 - 0x1p-30), 0)) v = rint(x / S);
    v = v < 0.0 ? 0.0 : (v > top ? top : v);
    return (int)v;
}

// ---------------------------------------------------------------------------------
// working layout
// ---------------------------------------------------------------------------------
// Both steps work on transposed binary32 copies, [column k][row m] with the row index fastest and a
// pitch Mp = M rounded up to 4: one thread per row then reads and writes coalesced, and both dense
// products (bcq_product.h) take their operands "k-major" (the summation index is the slow one).  Workspace, in floats:
//   Wt [N][Mp] | Dt [N][Mp] | part [ceil(N/128)][Mp] | wmin, wmax, best [3][Mp] | small [128][Mp]
// (search: Wt becomes the halves of d, Dt holds d, small the exponents of its scales; the screened search: see
// search_screened; GPTQ pass: Dt holds the errors of two panels, part or small the tables, small the smallest diagonals of two panels)
struct QuantWorkspace {
    int Mp, ntile;
    float *Wt, *Dt, *part, *wmin, *wmax, *best, *small;
};

static int pitch_of(int M) { return (M + 3) / 4 * 4; }

static QuantWorkspace carve(void *workspace, int M, int N)
{
    QuantWorkspace w;
    w.Mp = pitch_of(M);
    w.ntile = (N + 127) / 128;
    w.Wt = static_cast<float *>(workspace);
    w.Dt = w.Wt + (size_t)N * w.Mp;
    w.part = w.Dt + (size_t)N * w.Mp;
    w.wmin = w.part + (size_t)w.ntile * w.Mp;
    w.wmax = w.wmin + w.Mp;
    w.best = w.wmax + w.Mp;
    w.small = w.best + w.Mp;
    return w;
}

size_t quant_workspace_bytes(int M, int N)
{
    const size_t Mp = pitch_of(M), ntile = (size_t)(N + 127) / 128;
    const size_t floats = 2 * (size_t)N * Mp + ntile * Mp + 3 * Mp + 128 * Mp;
    return (floats * 4 + 255) / 256 * 256;
}

// Wt[k][m] = W[m][k]; the pad rows m in [M, Mp) are written as zeros.
__global__ void transpose_kernel(int M, int Mp, int N, const float *__restrict__ W, float *__restrict__ Wt)
{
    __shared__ float tile[32][33];
    const int m0 = blockIdx.y * 32, k0 = blockIdx.x * 32;
    for (int i = threadIdx.y; i < 32; i += blockDim.y) {
        const int m = m0 + i, k = k0 + threadIdx.x;
        tile[i][threadIdx.x] = (m < M && k < N) ? W[(size_t)m * N + k] : 0.0f;
    }
    __syncthreads();
    for (int i = threadIdx.y; i < 32; i += blockDim.y) {
        const int k = k0 + i, m = m0 + threadIdx.x;
        if (m < Mp && k < N) Wt[(size_t)k * Mp + m] = tile[threadIdx.x][i];
    }
}

// ---------------------------------------------------------------------------------
// Hessian of the layer-wise objective (Sec. II-A): H += 2 X^T X for T more calibration inputs
// ---------------------------------------------------------------------------------
hipError_t launch_quant_hessian(int N, int T, const float *X, float *H, hipStream_t stream)
{
    // X is [T][N]: k-major for both operands, C[r][c] = sum_t X[t][r] X[t][c]
    launch_product<kAddTwiceSymmetric>(stream, X, N, N, X, N, N, T, H, N);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------
// U with (H + lambda I)^-1 = U^T U, U upper triangular: what the GPTQ pass reads (Eq. 2)
// ---------------------------------------------------------------------------------
// With H_d = H + lambda I = R R^T, R UPPER triangular (a Cholesky factorisation taken from the last
// row upwards), H_d^-1 = R^-T R^-1, so U = R^-1.  Both steps are blocked by 128 columns; the diagonal
// blocks are inverted by one workgroup, everything else is the k-major product of bcq_product.h (K = 128
// panels, trailing updates of K = 128 and 512 for R; growing K for the off-diagonal blocks of U).
// Working matrices (binary32, pitch N): Hw = H_d (consumed), Rt = R^T, Ut = U^T, T = one panel.
constexpr int kFactorBlock = 128, kFactorPanel = 512;
// Tiles of a trailing update from which its far part runs beside the next panel: 128 are done in 24 us by themselves, with the rows of the next
// panel, which alone take as long.
constexpr int kFactorBeside = 128;

// H_d is factored as D^-1 H_d D^-1, D = diag(2^e) with 2^2e <= H_d[j][j] < 2^(2e + 2): powers of two, so every rounding is that of
// the unscaled factorisation, but all rows and columns of what the products multiply are of one size.  (They hold an operand
// to a step that its row's or column's largest value sets: with loud channels the ordinary entries of a column would lose bits
// that count once a block's inverse has scaled the large ones down again.)  The columns of U are scaled back where they are
// first written; Ut stays as it is.
__device__ __forceinline__ int channel_shift(float h, float lambda)
{
    const unsigned bits = __float_as_uint(h + lambda);
    return bits - 0x00800000u < 0x7f000000u ? (((int)(bits >> 23) - 127) >> 1) : 0;  // (not a positive normal number: no scale)
}

// lambda and the scale of every channel
__global__ void diag_mean_kernel(int N, const float *__restrict__ H, float damp, float *__restrict__ lambda, float *__restrict__ scale)
{
    __shared__ float part[256];
    float s = 0.0f;
    for (int i = threadIdx.x; i < N; i += 256) s += H[(size_t)i * N + i];
    part[threadIdx.x] = s;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if ((int)threadIdx.x < k) part[threadIdx.x] += part[threadIdx.x + k];
        __syncthreads();
    }
    const float l = damp * part[0] / (float)N;
    if (threadIdx.x == 0) *lambda = l;
    for (int i = threadIdx.x; i < N; i += 256) scale[i] = ldexpf(1.0f, -channel_shift(H[(size_t)i * N + i], l));
}

__global__ void damped_copy_kernel(int N, const float *__restrict__ H, const float *__restrict__ lambda, const float *__restrict__ scale,
                                   float *__restrict__ Hw)
{
    const int i = blockIdx.y, j = 4 * (blockIdx.x * blockDim.x + threadIdx.x);  // N is a multiple of 4
    if (j >= N) return;
    prod_f32x4 v = *reinterpret_cast<const prod_f32x4 *>(H + (size_t)i * N + j);
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (i == j + k) v[k] += *lambda;
    const prod_f32x4 s = *reinterpret_cast<const prod_f32x4 *>(scale + j);
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] *= scale[i] * s[k];
    *reinterpret_cast<prod_f32x4 *>(Hw + (size_t)i * N + j) = v;
}

// Diagonal block [r0, r0 + b): writes the blocks V = R^-1 of U and V^T of Ut, with D = R R^T, R upper triangular.  V is all
// that is needed of it (the panel is V times the rows of the block), and it comes straight out of an elimination in
// place, from the last row j upwards: with the pivot d = x[j][j] and f_i = x[i][j] / d,
//     x[i][l] -= f_i x[j][l]   for i < j and every l but j,      x[i][j] = -f_i.
// To the left of the pivot that is the Schur complement of D; the columns from j on are done with as parts of D and hold M,
// unit upper triangular, the product of the row operations, for which M D M^T = diag(d): V = diag(d)^-1/2 M.
// The rows are taken 16 at a time, J = j0 .. j0 + 15, in the block's place in LDS:
//   A   the elimination of D's 16 x 16 block by itself, which gives M_J and its pivots d: one wave, a row per lane, row j handed
//       round by DPP operands;
//   B   the 16 rows: X[J][:] becomes Y = M_J X[J][:], with M_J itself at J; and G = X[I][J] M_J^T diag(1 / d) for the rows I above
//       (X[J][I]^T: of the symmetric Schur complement only the tiles on and below the diagonal are kept);
//   C   the rows above: X[I][:] -= G Y, and X[I][J] = -G M_J.
// B and C are 16 x 16 tiles of binary32 matrix instructions.  What bounds it is that chain of one workgroup, so the tile that A needs next
// is C's first, and its wave goes on to A while the other three do the rest.  A block takes 24 us (A eight times
// 1.0, B 0.6, reading and writing 5); with two rows handed round per barrier and the block in registers 39 to 40, with one row 50.
constexpr int kDiagPitch = 148, kDiagG = 20;  // floats per row in LDS: a tile's elements in 16 x 4 lanes fall into different banks

// Elimination of a symmetric 16 x 16 block from the last row upwards: lane i of each 16 holds row i.  On return x[l] with l > i
// holds M[i][l] (unit upper triangular); this lane's pivot and its reciprocal.
__device__ __forceinline__ void eliminate_16(float (&x)[16], int i, float *pivot, float *inverse)
{
    auto step = [&](auto row) PROD_INLINE {
        constexpr int j = decltype(row)::value;
        float d;
        asm volatile("s_nop 1\n\tv_mov_b32_dpp %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf" : "=v"(d) : "v"(x[j]), "n"(j));
        float inv = __builtin_amdgcn_rcpf(d);
        inv = fmaf(fmaf(-d, inv, 1.0f), inv, inv);
        inv = d > 0.0f ? inv : __builtin_nanf("");  // not positive definite: no numbers from here on
        const float nf = i < j ? -(x[j] * inv) : 0.0f;
        if (i == j) { *pivot = d; *inverse = inv; }
        asm volatile("" ::"v"(nf));
#pragma unroll
        for (int l = 15; l >= 0; --l)
            if (l != j)
                asm volatile("v_fmac_f32_dpp %0, %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf" : "+v"(x[l]) : "v"(nf), "n"(j));
        x[j] = nf;  // (0 in the rows from j on)
    };
    step(std::integral_constant<int, 15>{}); step(std::integral_constant<int, 14>{}); step(std::integral_constant<int, 13>{});
    step(std::integral_constant<int, 12>{}); step(std::integral_constant<int, 11>{}); step(std::integral_constant<int, 10>{});
    step(std::integral_constant<int, 9>{}); step(std::integral_constant<int, 8>{}); step(std::integral_constant<int, 7>{});
    step(std::integral_constant<int, 6>{}); step(std::integral_constant<int, 5>{}); step(std::integral_constant<int, 4>{});
    step(std::integral_constant<int, 3>{}); step(std::integral_constant<int, 2>{}); step(std::integral_constant<int, 1>{});
    step(std::integral_constant<int, 0>{});
}

__device__ __forceinline__ void factor_diag(int N, int r0, int b, const float *__restrict__ Hw, const float *__restrict__ H,
                                            const float *__restrict__ lambda, float *__restrict__ U, float *__restrict__ Ut)
{
    __shared__ __attribute__((aligned(16))) float X[kFactorBlock][kDiagPitch];
    __shared__ float G[kFactorBlock][kDiagG];  // negated
    __shared__ __attribute__((aligned(16))) float pivot[kFactorBlock], inverse[kFactorBlock];
    const int tid = threadIdx.x, lane = tid & 63, lo = lane & 15, hi = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // this thread's four columns l .. l + 3 (b and N are multiples of 4) and rows first + 8 k, in and out
    const int l = 4 * (tid & 31), first = tid >> 5, l_in = l < b ? l : 0;
    prod_f32x4 v[16], scale;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const int i = first + 8 * k < b ? first + 8 * k : 0;
        v[k] = *reinterpret_cast<const prod_f32x4 *>(Hw + (size_t)(r0 + i) * N + r0 + l_in);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) scale[e] = H[(size_t)(r0 + l_in + e) * (N + 1)];
    const float damping = *lambda;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const int i = first + 8 * k;
        if (i >= b || l >= b)  // beyond b: the identity, which changes nothing
            v[k] = prod_f32x4{i == l ? 1.0f : 0.0f, i == l + 1 ? 1.0f : 0.0f, i == l + 2 ? 1.0f : 0.0f, i == l + 3 ? 1.0f : 0.0f};
        *reinterpret_cast<prod_f32x4 *>(&X[i][l]) = v[k];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) scale[e] = ldexpf(1.0f, -channel_shift(scale[e], damping));
    __syncthreads();
    auto inner = [&](int J) PROD_INLINE {  // A: M_J in the place of the block, with its zeros and ones
        float x[16], d = 1.0f, inv = 1.0f;
#pragma unroll
        for (int l = 0; l < 16; l += 4) {
            const prod_f32x4 v = *reinterpret_cast<const prod_f32x4 *>(&X[16 * J + lo][16 * J + l]);
#pragma unroll
            for (int e = 0; e < 4; ++e) x[l + e] = v[e];
        }
        eliminate_16(x, lo, &d, &inv);
        if (hi == 0) {
            pivot[16 * J + lo] = d;
            inverse[16 * J + lo] = inv;
#pragma unroll
            for (int l = 0; l < 16; ++l) X[16 * J + lo][16 * J + l] = l > lo ? x[l] : (l == lo ? 1.0f : 0.0f);
        }
    };
    // C for one tile
    auto update = [&](int J, int I, int L) PROD_INLINE {
        prod_f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        if (L != J) {
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i] = X[16 * I + 4 * hi + i][16 * L + lo];
        }
        float g[4], y[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            g[k] = G[16 * I + lo][4 * k + hi];
            y[k] = X[16 * J + 4 * k + hi][16 * L + lo];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(g[k], y[k], acc, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) X[16 * I + 4 * hi + i][16 * L + lo] = acc[i];
    };
    if (wave == 0) inner(7);
    __syncthreads();
    for (int J = 7; J >= 0; --J) {
        // B, a tile of columns L at a time: the elements of X[J][L] are the operand of both products
        {
            float m[4], w[4];
            const float inv = inverse[16 * J + lo];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                m[k] = X[16 * J + lo][16 * J + 4 * k + hi];
                w[k] = -(m[k] * inv);
            }
            float x[2][4];  // (of the wave's two tiles; M_J itself is left alone)
            prod_f32x4 y[2], g[2];
#pragma unroll
            for (int n = 0; n < 2; ++n) {
                y[n] = g[n] = prod_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int k = 0; k < 4; ++k) x[n][k] = X[16 * J + 4 * k + hi][16 * (wave + 4 * n) + lo];
            }
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int n = 0; n < 2; ++n) {
                    y[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(m[k], x[n][k], y[n], 0, 0, 0);
                    g[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[n][k], w[k], g[n], 0, 0, 0);
                }
#pragma unroll
            for (int n = 0; n < 2; ++n) {
                const int L = wave + 4 * n;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (L != J) X[16 * J + 4 * hi + i][16 * L + lo] = y[n][i];
                    if (L < J) G[16 * L + 4 * hi + i][lo] = g[n][i];
                }
            }
        }
        __syncthreads();
        if (J == 0) break;
        // C, and A of the next 16 rows: the tiles (I, L), I < J, with L <= I (the Schur complement) or L >= J (M); tile (J - 1, J - 1)
        // is the first wave's
        if (wave == 0) {
            update(J, J - 1, J - 1);
            inner(J - 1);
        } else {
            int skip = wave - 1;
            for (int I = J - 1; I >= 0; --I) {
                const int below = I == J - 1 ? I : I + 1, count = below + 8 - J;
                for (; skip < count; skip += 3) update(J, I, skip < below ? skip : J + skip - below);
                skip -= count;
            }
        }
        __syncthreads();
    }
    if (tid < kFactorBlock) inverse[tid] = 1.0f / sqrtf(pivot[tid]);
    __syncthreads();
#pragma unroll 4
    for (int k = 0; k < 16; ++k) {
        const int i = first + 8 * k;
        const float root = inverse[i];
        prod_f32x4 u = *reinterpret_cast<const prod_f32x4 *>(&X[i][l]);
#pragma unroll
        for (int e = 0; e < 4; ++e) u[e] = l + e >= i ? u[e] * root * scale[e] : 0.0f;
        if (i < b && l < b) *reinterpret_cast<prod_f32x4 *>(U + (size_t)(r0 + i) * N + r0 + l) = u;
    }
    // Ut's rows i .. i + 3 from row c of X
    const int c = tid & (kFactorBlock - 1), half = 64 * (tid >> 7);
    const float root = inverse[c];
    if (c < b) {
#pragma unroll 4
        for (int i = half; i < half + 64; i += 4) {
            const prod_f32x4 x = *reinterpret_cast<const prod_f32x4 *>(&X[c][i]);
            if (i < b) {
#pragma unroll
                for (int e = 0; e < 4; ++e) Ut[(size_t)(r0 + i + e) * N + r0 + c] = i + e >= c ? x[e] * root : 0.0f;
            }
        }
    }
}

__global__ __launch_bounds__(256) void factor_diag_kernel(int N, int r0, int b, const float *__restrict__ Hw, const float *__restrict__ H,
                                                          const float *__restrict__ lambda, float *__restrict__ U, float *__restrict__ Ut)
{
    factor_diag(N, r0, b, Hw, H, lambda, U, Ut);
}

// The same in the first workgroup, and in those from the eighth on (workgroup numbers go round the XCDs) the tiles
// `first_tile`, .. of `far`, the update of the rows above this panel's by the panel before: a diagonal block is one workgroup's chain, and
// the chip is free beside it.  The LDS makes that one tile per compute unit; with 248 tiles a launch takes 30 to 35 us, 25 without any.
// 7168 channels, with the order of the products of the inverse (bcq_product.h): 4.36 -> 4.00 ms, of which this is half (in launches of
// their own the 13 trailing updates are 0.73 ms).
__global__ __launch_bounds__(256) void factor_diag_far_kernel(int N, int r0, int b, float *Hw, const float *__restrict__ H,
                                                              const float *__restrict__ lambda, float *__restrict__ U,
                                                              float *__restrict__ Ut, ProductArgs far, int first_tile, int tiles)
{
    __shared__ ProductShared s;
    if (blockIdx.x == 0) {
        __builtin_amdgcn_s_setprio(3);
        factor_diag(N, r0, b, Hw, H, lambda, U, Ut);
    } else if (blockIdx.x >= 8) {
        product_tile_of<kSubtractLower>(far, first_tile + (int)blockIdx.x - 8, tiles, s.stage_a0, s.stage_a1, s.stage_b, s.largest,
                                        s.largest_of_tile, s.shift);
    }
}

// dst[c][r] = src[r][c], without the scale of channel c, for size x size blocks of a matrix of pitch N, block z of them z * stride
// floats on, the last one with columns_end - 2 size z columns; the columns of the first one are the channels from `size` on.
__global__ void transpose_blocks_kernel(int size, int N, size_t stride, int columns_end, const float *__restrict__ src,
                                        const float *__restrict__ H, const float *__restrict__ lambda, float *__restrict__ dst)
{
    __shared__ float tile[32][33];
    src += blockIdx.z * stride;
    dst += blockIdx.z * stride;
    const int left = columns_end - 2 * size * (int)blockIdx.z, cols = left < size ? left : size;
    const int r0 = blockIdx.y * 32, c0 = blockIdx.x * 32;
    for (int i = threadIdx.y; i < 32; i += blockDim.y) {
        const int r = r0 + i, c = c0 + threadIdx.x;
        tile[i][threadIdx.x] = c < cols ? src[(size_t)r * N + c] : 0.0f;  // size is a multiple of 32
    }
    __syncthreads();
    for (int i = threadIdx.y; i < 32; i += blockDim.y) {
        const int c = c0 + i, r = r0 + threadIdx.x;
        if (c >= cols) continue;
        const size_t channel = (size_t)size + 2 * (size_t)size * blockIdx.z + c;
        dst[(size_t)c * N + r] = tile[threadIdx.x][i] * ldexpf(1.0f, channel_shift(H[channel * N + channel], *lambda));
    }
}

size_t quant_factor_workspace_bytes(int N)
{
    const size_t floats = 3 * (size_t)N * N + 64;
    return (floats * 4 + 255) / 256 * 256;
}

// Off-diagonal blocks of U = R^-1 (the diagonal blocks are in place), in neighbouring pairs of 1, 2, 4, ... blocks: with
// the rows / columns [lo, mid) and [mid, hi) of a pair done, U12 = -U11 (R12 U22).  All pairs of one size are one launch
// per product (28 of the 128-column ones at 7168, at 11 us each they were most of the inverse: 2.4 -> 1.1 ms).  T = R12 U22
// takes the place of the same block of a matrix that is free.
static void invert_blocks(hipStream_t stream, int N, const float *Rt, const float *H, const float *lambda, float *U, float *Ut, float *T)
{
    for (int size = kFactorBlock; size < N; size *= 2) {
        const int count = (N - size + 2 * size - 1) / (2 * size);  // pairs whose second half is not empty
        const size_t stride = (size_t)2 * size * ((size_t)N + 1);
        const size_t above = size, below = (size_t)size * N;  // block (lo, mid), block (mid, lo) of the first pair
        // T[i][c] = sum_m R[lo + i][mid + m] U[mid + m][mid + c]
        launch_products<kStore>(stream, count, stride, N - size, Rt + below, U + below + above, T + above, N, size);
        // U[lo + r][mid + c] = -sum_j U[lo + r][lo + j] T[j][c]
        launch_products<kStoreNegated>(stream, count, stride, N - size, Ut, T + above, U + above, N, size);
        hipLaunchKernelGGL(transpose_blocks_kernel, dim3(size / 32, size / 32, count), dim3(32, 8), 0, stream, size, N, stride,
                           N - size, U + above, H, lambda, Ut + below);
    }
}

hipError_t launch_quant_factor(int N, float damp, const float *H, float *U, void *workspace, hipStream_t stream)
{
    float *Hw = static_cast<float *>(workspace);
    float *Rt = Hw + (size_t)N * N, *Ut = Rt + (size_t)N * N;
    float *lambda = Ut + (size_t)N * N;
    float *const scale = Rt;  // (written over by the first panel)
    hipLaunchKernelGGL(diag_mean_kernel, dim3(1), dim3(256), 0, stream, N, H, damp, lambda, scale);
    hipLaunchKernelGGL(damped_copy_kernel, dim3((N / 4 + 255) / 256, N), dim3(256), 0, stream, N, H, lambda, scale, Hw);
    hipError_t e = launch_fill_zero(U, (size_t)N * N * 4, stream);
    if (e != hipSuccess) return e;
    e = launch_fill_zero(Ut, (size_t)N * N * 4, stream);
    if (e != hipSuccess) return e;
    // R, from the last block column to the first.  Only the part of Hw on and below its diagonal blocks is kept up to date:
    // after a block the rows of its panel (four blocks), which the next blocks need, after a panel all rows above it, with
    // the panel's 512 columns at once (a pass over what remains costs its reading and writing however few columns it adds): first
    // the rows of the next panel, then, beside that panel's diagonal blocks, those above them.
    ProductArgs far = {};
    int tiles = 0, done = 0;  // of `far`, in multiples of 8
    const int beside = (compute_units() - 1) / 8 * 8;
    auto diag = [&](int r0, int b, int count) {
        if (count > 0)
            hipLaunchKernelGGL(factor_diag_far_kernel, dim3((unsigned)(8 + count)), dim3(256), 0, stream, N, r0, b, Hw, H, lambda, U, Ut, far, done,
                               tiles);
        else
            hipLaunchKernelGGL(factor_diag_kernel, dim3(1), dim3(256), 0, stream, N, r0, b, Hw, H, lambda, U, Ut);
        done += count;
    };
    for (int p1 = N; p1 > 0;) {
        const int p0 = (p1 - 1) / kFactorPanel * kFactorPanel;
        // What does not fit beside the panel's blocks goes before them, two workgroups to a compute unit: 3 % of the tiles at 7168 channels,
        // 62 % at 14336, 89 % at 28672.  ms, all trailing updates in launches of their own / this / with the rest in the kernel that
        // has a diagonal block beside, one workgroup to a compute unit: 10240 channels 8.0 / 7.2 / 7.5, 14336 15.3 / 14.1 / 15.3, 28672 88.0 / 80.3 / 93.7,
        // 32768 138 / 125 / 145.
        const int blocks = (p1 - p0 + kFactorBlock - 1) / kFactorBlock;
        if (const int rest = tiles - blocks * beside; rest > 0) {
            hipLaunchKernelGGL(product_part_kernel<kSubtractLower>, dim3((unsigned)rest), dim3(256), 0, stream, far, 0, tiles);
            done = rest;
        }
        for (int r1 = p1; r1 > p0;) {
            const int r0 = (r1 - 1) / kFactorBlock * kFactorBlock, b = r1 - r0;
            diag(r0, b, tiles - done < beside ? tiles - done : beside);
            if (r0 > 0) {
                // panel, transposed: Rt[r0 + c][i] = R[i][r0 + c] = sum_m V[c][m] Hw[r0 + m][i]   (Hw symmetric, V = R_kk^-1)
                launch_product<kStore>(stream, Ut + (size_t)r0 * N + r0, N, b, Hw + (size_t)r0 * N, N, r0, b, Rt + (size_t)r0 * N, N);
                // Hw[i][j] -= sum_c R[i][r0 + c] R[j][r0 + c] for p0 <= i < r0, j < r0
                if (r0 > p0)
                    launch_product<kSubtract>(stream, Rt + (size_t)r0 * N + p0, N, r0 - p0, Rt + (size_t)r0 * N, N, r0, b,
                                              Hw + (size_t)p0 * N, N);
            }
            r1 = r0;
        }
        // Hw[i][j] -= sum_c R[i][p0 + c] R[j][p0 + c] for j <= i < p0 (by tiles); where there is much of it, only q0 <= i now
        const int q0 = p0 > 0 ? (p0 - 1) / kFactorPanel * kFactorPanel : 0;
        tiles = done = 0;
        if (p0 > 0 && product_groups<kSubtractLower>(q0, q0) >= kFactorBeside) {
            launch_product<kSubtract>(stream, Rt + (size_t)p0 * N + q0, N, p0 - q0, Rt + (size_t)p0 * N, N, p0, p1 - p0, Hw + (size_t)q0 * N, N);
            far = product_args(Rt + (size_t)p0 * N, N, q0, Rt + (size_t)p0 * N, N, q0, p1 - p0, Hw, N);
            tiles = product_groups<kSubtractLower>(q0, q0);
        } else if (p0 > 0) {
            launch_product<kSubtractLower>(stream, Rt + (size_t)p0 * N, N, p0, Rt + (size_t)p0 * N, N, p0, p1 - p0, Hw, N);
        }
        p1 = p0;
    }
    // U = R^-1: Hw is free now and holds the intermediate products
    invert_blocks(stream, N, Rt, H, lambda, U, Ut, Hw);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------
// search
// ---------------------------------------------------------------------------------
// Row minimum and maximum in two steps: `chunks` slabs of columns each leave a partial pair in
// scratch ([chunks][Mp] minima, then [chunks][Mp] maxima), a second launch combines them.
__global__ void row_range_partial_kernel(int M, int Mp, int N, int chunks, const float *__restrict__ Wt,
                                         float *__restrict__ scratch)
{
    const int m = blockIdx.x * blockDim.x + threadIdx.x, chunk = blockIdx.y;
    if (m >= M) return;
    const int per = (N + chunks - 1) / chunks;
    const int k_end = (chunk + 1) * per < N ? (chunk + 1) * per : N;
    float lo = INFINITY, hi = -INFINITY;
    for (int k = chunk * per; k < k_end; ++k) {
        const float v = Wt[(size_t)k * Mp + m];
        lo = fminf(lo, v);
        hi = fmaxf(hi, v);
    }
    scratch[(size_t)chunk * Mp + m] = lo;
    scratch[(size_t)(chunks + chunk) * Mp + m] = hi;
}

__global__ void row_range_final_kernel(int M, int Mp, int chunks, const float *__restrict__ scratch,
                                       float *__restrict__ wmin, float *__restrict__ wmax)
{
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= M) return;
    float lo = INFINITY, hi = -INFINITY;
    for (int c = 0; c < chunks; ++c) {
        lo = fminf(lo, scratch[(size_t)c * Mp + m]);
        hi = fmaxf(hi, scratch[(size_t)(chunks + c) * Mp + m]);
    }
    wmin[m] = lo;
    wmax[m] = hi;
}

// The same from W itself, a wave per row, where its rows can be read four weights at a time.
__global__ __launch_bounds__(256) void row_range_kernel(int M, int N, const float *__restrict__ W, float *__restrict__ wmin,
                                                        float *__restrict__ wmax)
{
    const int m = 4 * blockIdx.x + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (m >= M) return;
    const prod_f32x4 *const row = reinterpret_cast<const prod_f32x4 *>(W + (size_t)m * N);
    float lo = INFINITY, hi = -INFINITY;
    for (int k = lane; k < N / 4; k += 64) {
        const prod_f32x4 v = row[k];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            lo = fminf(lo, v[j]);
            hi = fmaxf(hi, v[j]);
        }
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
        lo = fminf(lo, __shfl_xor(lo, d));
        hi = fmaxf(hi, __shfl_xor(hi, d));
    }
    if (lane == 0) {
        wmin[m] = lo;
        wmax[m] = hi;
    }
}

// Scale of grid point g (0-based) of a row, Eq. 7, in binary64.
__device__ __forceinline__ double grid_scale(double wmin, double wmax, int n_bits, int g, int grid)
{
    if (wmax == wmin) return 1.0;  // a constant row: Eq. 7's interval is empty, any scale reproduces it
    const double lo = (wmax - wmin) / (double)((1 << (n_bits + 1)) - 1);
    const double hi = (wmax - wmin) / (double)((1 << (n_bits - 1)) - 1);
    return lo + (hi - lo) * ((double)(g + 1) / ((double)grid + 1.0));
}

// What the quadratic forms take their scales from.  Exponent of the power of two by which a row's d are scaled before they are
// split: |d| stays below twice the row's range, which goes to at most 2^15.  The last block: the largest finite value on the
// diagonal of H (a launch of its own for it was 3 us of a small search).
__global__ __launch_bounds__(256) void split_shift_kernel(int M, int Mp, const float *__restrict__ wmin, const float *__restrict__ wmax,
                                                          int *__restrict__ shift, int N, const float *__restrict__ H,
                                                          float *__restrict__ diag_max)
{
    if (blockIdx.x < gridDim.x - 1) {
        const int m = blockIdx.x * blockDim.x + threadIdx.x;
        if (m < Mp) shift[m] = m < M ? product_shift(__float_as_uint(wmax[m] - wmin[m]), 13) : 0;
        return;
    }
    __shared__ float part[4];
    float most = 0.0f;
    for (int i = threadIdx.x; i < N; i += 256) {
        const float d = H[(size_t)i * N + i];
        if (d < INFINITY) most = fmaxf(most, d);
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) most = fmaxf(most, __shfl_xor(most, d));
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = most;
    __syncthreads();
    if (threadIdx.x == 0) *diag_max = fmaxf(fmaxf(part[0], part[1]), fmaxf(part[2], part[3]));
}

// What the search keeps of a candidate of a chunk: the nearest representable integer of every integer, as nibbles (up to four
// bits) and bytes, and the class of every plane.
struct CandidateTable {
    unsigned long long nibbles;
    int8_t label[kMaxBits];
    uint8_t nearest[1 << kMaxBits];
};

// Rows to evaluate and with which candidate of the chunk each.
struct SearchList {
    const int *count, *row, *candidate;
    const CandidateTable *tables;
    int first_candidate, tyings;
};

// d = S' W_q + qbias - w of one candidate (grid point g, tying t), in three forms:
//   kPlain    Dt[k][m] from Wt; zeros in the pad rows
//   kSplit    Dt[k][m] from W, and the same values as two binary16 halves in the operand layout of the matrix instructions, [hi,
//             lo][k / 8][m][k % 8], so that the product does not have to convert them once per column tile
//   kListed   kSplit of the rows and candidates of a list
// A workgroup takes 64 rows by 32 columns, a thread eight columns of a row.  Bound: memory.  7168 x 7168: 218 us per candidate (a
// division and a scan of the representable set per weight, nothing split) -> 111 us with the split, 617 MB.
enum DeltaForm { kPlain = 0, kSplit = 1, kListed = 2 };
template <int FORM>
__global__ __launch_bounds__(256) void delta_kernel(int M, int Mp, int N, int n_bits, int g, int grid, Tying t,
                                                    const float *__restrict__ W, const float *__restrict__ wmin,
                                                    const float *__restrict__ wmax, float *__restrict__ Dt,
                                                    const int *__restrict__ shift, uint16_t *__restrict__ split, size_t plane,
                                                    SearchList list, int *__restrict__ slot_shift)
{
    const int slot = blockIdx.x * 64 + (threadIdx.x & 63);
    if (FORM == kListed && blockIdx.x * 64 >= (unsigned)*list.count) return;
    if (slot >= Mp) return;
    int k0 = 8 * (blockIdx.y * 4 + (threadIdx.x >> 6));
    bool live = slot < M;
    int m = live ? slot : 0;
    const CandidateTable *of = nullptr;
    unsigned long long nibbles = t.nibbles;
    if (FORM == kListed) {
        live = slot < *list.count;
        m = live ? list.row[slot] : 0;
        const int c = live ? list.candidate[slot] : 0;
        of = list.tables + c;
        nibbles = of->nibbles;
        g = (list.first_candidate + c) / list.tyings;
        if (k0 == 0) slot_shift[slot] = live ? shift[m] : 0;
    }
    for (; k0 < N; k0 += FORM == kListed ? 32 * (int)gridDim.y : N) {
        float w[8], d[8];
        if (FORM != kPlain) {  // N is a multiple of 8, W on 16 bytes
            const prod_f32x4 *src = reinterpret_cast<const prod_f32x4 *>(W + (size_t)m * N + k0);
#pragma unroll
            for (int j = 0; j < 8; ++j) w[j] = src[j >> 2][j & 3];
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) w[j] = k0 + j < N ? W[(size_t)(k0 + j) * Mp + slot] : 0.0f;
        }
        if (live) {
            const double lo = wmin[m], S = grid_scale(lo, wmax[m], n_bits, g, grid), inv_s = 1.0 / S, top = (double)((1 << n_bits) - 1);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int lin = linear_int((double)w[j] - lo, S, inv_s, top);
                const int wq = n_bits <= 4 ? (int)(nibbles >> (4 * lin)) & 15
                               : FORM == kListed ? of->nearest[lin] : nearest_choice(lin, t.choice, t.nchoice);
                d[j] = (float)(S * wq + lo - (double)w[j]);
            }
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) d[j] = 0.0f;
        }
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (k0 + j < N) Dt[(size_t)(k0 + j) * Mp + slot] = d[j];
        if (FORM != kPlain) {
            const float s = ldexpf(1.0f, live ? shift[m] : 0);
            prod_f16x8 hi, lo;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                hi[j] = (_Float16)(d[j] * s);
                lo[j] = (_Float16)fmaf(d[j], s, -(float)hi[j]);
            }
            uint16_t *const at = split + ((size_t)(k0 >> 3) * Mp + slot) * 8;
            *reinterpret_cast<prod_f16x8 *>(at) = hi;
            *reinterpret_cast<prod_f16x8 *>(at + plane) = lo;
        }
    }
}

// The same d for the screened search: of up to kPlanes tyings of one grid point, each a binary16 number rounded at random (see
// bcq_screen.h), in planes of the operand layout; also fills the candidates' tables.  Bound: memory.  7168 x 7168, three tyings: 68 us each one by one, W
// being read each time, 32 together, and 35 with the random roundings.
constexpr int kPlanes = 3;  // (the workspace holds 4 - N / M planes, for N <= M three)
struct TyingSet { Tying t[kPlanes]; };
template <int PLANES>
__global__ __launch_bounds__(256) void delta_single_kernel(int M, int Mp, int N, int n_bits, int g, int grid, TyingSet set,
                                                           const float *__restrict__ W, const float *__restrict__ wmin,
                                                           const float *__restrict__ wmax, const int *__restrict__ shift,
                                                           uint16_t *__restrict__ out, CandidateTable *__restrict__ tables)
{
    const int m = blockIdx.x * 64 + (threadIdx.x & 63), k0 = 8 * (blockIdx.y * 4 + (threadIdx.x >> 6));
    if (blockIdx.x == 0 && blockIdx.y == 0) {
        const int w = threadIdx.x;
#pragma unroll
        for (int p = 0; p < PLANES; ++p) {
            const Tying &t = set.t[p];
            if (w == 0) tables[p].nibbles = t.nibbles;
            if (w < kMaxBits) tables[p].label[w] = t.label[w];
            if (w < 1 << n_bits) tables[p].nearest[w] = (uint8_t)nearest_choice(w, t.choice, t.nchoice);
        }
    }
    if (m >= Mp || k0 >= N) return;
    prod_f16x8 d[PLANES];
#pragma unroll
    for (int p = 0; p < PLANES; ++p) d[p] = prod_f16x8{0, 0, 0, 0, 0, 0, 0, 0};
    if (m < M) {
        const prod_f32x4 *src = reinterpret_cast<const prod_f32x4 *>(W + (size_t)m * N + k0);
        const prod_f32x4 w0 = src[0], w1 = src[1];
        const double lo = wmin[m], S = grid_scale(lo, wmax[m], n_bits, g, grid), inv_s = 1.0 / S, top = (double)((1 << n_bits) - 1);
        const float s = ldexpf(1.0f, shift[m]);
        unsigned random[4];  // for two values each, the same for all candidates (each has a bound of its own)
#pragma unroll
        for (int j = 0; j < 4; ++j) random[j] = screen_hash((unsigned)m, (unsigned)(k0 / 2 + j), 2u);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const double w = j < 4 ? w0[j & 3] : w1[j & 3];
            const int lin = linear_int(w - lo, S, inv_s, top);
#pragma unroll
            for (int p = 0; p < PLANES; ++p) {
                const int wq = n_bits <= 4 ? (int)(set.t[p].nibbles >> (4 * lin)) & 15 : nearest_choice(lin, set.t[p].choice, set.t[p].nchoice);
                d[p][j] = (_Float16)screen_round((float)(S * wq + lo - w) * s, random[j >> 1] >> (16 * (j & 1)));
            }
        }
    }
    const size_t at = ((size_t)(k0 >> 3) * Mp + m) * 8, plane = (size_t)N * Mp;
#pragma unroll
    for (int p = 0; p < PLANES; ++p) *reinterpret_cast<prod_f16x8 *>(out + p * plane + at) = d[p];
}

// err = sum of the row's tile partials, in tile order (each is half of its part of d H d^T: H = 2 X X^T); keep the
// candidate if it is strictly better.
__global__ void keep_best_kernel(int M, int Mp, int n_bits, int ntile, int g, int grid, int first, Tying t,
                                 const float *__restrict__ part, const float *__restrict__ wmin,
                                 const float *__restrict__ wmax, float *__restrict__ best, float *__restrict__ S,
                                 float *__restrict__ qbias, int8_t *__restrict__ labels)
{
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= M) return;
    float e = 0.0f;
    for (int k = 0; k < ntile; ++k) e += part[(size_t)k * Mp + m];
    if (first || e < best[m]) {
        best[m] = e;
        S[m] = (float)grid_scale(wmin[m], wmax[m], n_bits, g, grid);
        qbias[m] = wmin[m];
        for (int i = 0; i < n_bits; ++i) labels[(size_t)m * n_bits + i] = t.label[i];
    }
}

// A round of the screened search, per row: takes the errors of the round before (entries of the row's range in the list), and lists
// what is to be evaluated next: in the first round the candidate with the lowest bound, then all whose bound does not exclude
// that they are better than the best so far, or as good and earlier.  As much as fits; the rest comes in the next round.
struct SearchRound {
    float *bound;             // [candidate of the chunk][Mp]; infinite: done with
    int candidates, first_candidate, tyings;
    int *total;               // entries of this round, zero before
    const int *last_total;    // and of the one before: none means that nothing is left
    int *row, *candidate;     // its list, up to Mp entries
    const int *last_candidate; // the list of the round before
    int *begin, *count;       // [Mp] range of a row's entries
    int *index;               // [Mp] candidate that is best (-1: decided, first candidate without a number)
    const CandidateTable *tables;
    int fresh, start, end;    // nothing evaluated yet; first round of a chunk; no further round
};
__global__ __launch_bounds__(256) void search_round_kernel(int M, int Mp, int n_bits, int grid, int ntile, SearchRound r,
                                                           const float *__restrict__ part, const float *__restrict__ wmin,
                                                           const float *__restrict__ wmax, float *__restrict__ best_out,
                                                           float *__restrict__ S, float *__restrict__ qbias, int8_t *__restrict__ labels)
{
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= M || (!r.start && *r.last_total == 0)) return;
    float best = r.fresh ? INFINITY : best_out[m];
    int index = r.fresh ? 0x7fffffff : r.index[m];
    if (!r.start) {
        const int before = index, begin = r.begin[m], count = r.count[m];
        int won = 0;
        for (int e = begin; e < begin + count; ++e) {
            const int c = r.last_candidate[e], j = r.first_candidate + c;
            float err = 0.0f;
            for (int k = 0; k < ntile; ++k) err += part[(size_t)k * Mp + e];
            if (j == 0 && err != err) {
                best = err;
                index = -1;
                won = c;
            } else if (index >= 0 && (err < best || (err == best && j < index))) {
                best = err;
                index = j;
                won = c;
            }
        }
        if (index != before) {
            S[m] = (float)grid_scale(wmin[m], wmax[m], n_bits, (r.first_candidate + won) / r.tyings, grid);
            qbias[m] = wmin[m];
            for (int i = 0; i < n_bits; ++i) labels[(size_t)m * n_bits + i] = r.tables[won].label[i];
        }
    }
    best_out[m] = best;
    r.index[m] = index;
    if (r.end) return;
    int n = 0, lowest = 0;
    float low = INFINITY;
    if (index >= 0)
        for (int c = 0; c < r.candidates; ++c) {
            const float b = r.bound[(size_t)c * Mp + m];
            if (!(b < INFINITY) || b > best || (b == best && r.first_candidate + c > index)) continue;
            ++n;
            if (b < low) {
                low = b;
                lowest = c;
            }
        }
    const bool one = r.fresh && n > 1;
    if (one) n = 1;
    int at = n ? atomicAdd(r.total, n) : 0;
    if (at >= Mp) n = 0;  // (the total may run beyond the list; who reads it takes no more than fits)
    else if (at + n > Mp) n = Mp - at;
    r.begin[m] = at;
    r.count[m] = n;
    for (int c = one ? lowest : 0; n > 0 && c < r.candidates; ++c) {
        float &b = r.bound[(size_t)c * Mp + m];
        if (!(b < INFINITY) || b > best || (b == best && r.first_candidate + c > index)) continue;
        r.row[at] = m;
        r.candidate[at++] = c;
        b = INFINITY;
        --n;
    }
}

// The screened search (bcq_screen.h) keeps its matrices in the place of Wt and Dt, where the listed rows' d come afterwards:
//   Dh binary16 [planes][N / 8][Mp][8] (before that z) | Hh binary16 [N / 8][N][8] | R binary16 [N / 8][projection][8]
// and in `small`: shift [Mp] | diag_max, frobenius | bound [chunk][Mp] | sums [planes][kScreenSums][Mp] | slot_shift, row and candidate of two
// lists, begin, count, index [8][Mp] | unscale, norms [2][N] | totals [chunk] | tables [chunk] | R where there was no room for it.
constexpr int kChunk = 48;
struct ScreenPlan { int planes, projections, chunk, r_in_small; };  // candidates at a time and per chunk; no planes: there is no room
static ScreenPlan screen_plan(int M, int N, int tyings, int candidates)
{
    const long long Mp = pitch_of(M);
    for (int planes = tyings < kPlanes ? tyings : kPlanes; planes > 0; --planes)
        for (int projections = kProjections; projections >= kFewProjections; projections /= 2) {
            const long long left = 2 * N * Mp - (long long)N * N / 2 - (long long)planes * N * Mp / 2;  // floats
            const long long r = (long long)N * projections / 2;
            if (left < 0) continue;
            const int r_in_small = left < r;
            const long long fixed = (9 + kScreenSums * planes) * Mp + 16 + 2LL * N + 64 + (r_in_small ? r : 0);
            long long chunk = (128 * Mp - fixed) / (Mp + 1 + (long long)sizeof(CandidateTable) / 4);
            chunk = chunk < kChunk ? chunk : kChunk;
            chunk = chunk < candidates ? chunk : candidates;
            if (chunk >= (candidates < 8 ? candidates : 8)) return {planes, projections, (int)chunk, r_in_small};
        }
    return {0, 0, 0, 0};
}

// Screening is two rounds of three products each and a product per candidate instead of three per candidate.  us, all candidates /
// screened, three bits, two planes, eight scales: 7168 x 7168 31450 / 11230 (before it took any H: 10300), 2500 x 7168 11690 / 5700, 2048 x 2048
// 2100 / 858, 512 x 512 768 / 380.  Candidates evaluated of 24, 7168 x 7168: 1.15 per row with samples like the tests', 1.3 with channel means of 2
// sigma, 2.7 of 5, 7.9 of 30 (23.4 ms), 2.2 with two channels 1000 times as loud; 4096 x 4096 with means of 30 sigma 11.1 (6.6 / 6.9 ms).
// A screened search has about as many launches per candidate for rounds that find nothing (22 here), and H to prepare.  The line
// lies where that is made up for: from four candidates on for large layers (4096 x 4096 1164 / 1104, 3000 x 3000 653 / 662), from six
// where three tyings share a launch or from 1024 channels on (256 x 256 158 / 152, 344 x 1024 305 / 307), from eight where two do or from
// 2^20 weights on (256 x 512 293 / 255 at nine; 7168 x 512 353 / 342, six 274 / 288), below that from 6144 / N (256 x 256 552 / 529,
// 16 candidates 376 / 382; 512 x 512 392 / 363, eight 270 / 280).
static bool screen_pays(int M, int N, int planes, int candidates)
{
    const long long weights = (long long)M * N;
    if (candidates >= 8 && (planes > 1 || weights >= 1 << 20 || candidates * N >= 6144)) return true;
    return candidates >= 6 ? planes == 3 || N >= 1024 || weights >= 1 << 24 : candidates >= 4 && weights >= 1 << 24;
}

static hipError_t search_screened(int M, int N, int n_bits, int grid, const std::vector<Tying> &tyings, ScreenPlan plan, const float *W,
                                  const float *H, float *S, float *qbias, int8_t *labels, const QuantWorkspace &w, hipStream_t stream)
{
    const int Mp = w.Mp, T = (int)tyings.size(), all = grid * T;
    auto *Dh = reinterpret_cast<uint16_t *>(w.Wt);
    uint16_t *const Hh = Dh + (size_t)plan.planes * N * Mp;
    auto *shift = reinterpret_cast<int *>(w.small);
    float *diag_max = w.small + Mp, *frobenius = diag_max + 4, *bound = diag_max + 16, *sums = bound + (size_t)plan.chunk * Mp;
    const size_t sums_floats = (size_t)kScreenSums * plan.planes * Mp;
    auto *slot_shift = reinterpret_cast<int *>(sums + sums_floats);
    int *list[2] = {slot_shift + Mp, slot_shift + 3 * (size_t)Mp};
    int *begin = slot_shift + 5 * (size_t)Mp, *count = begin + Mp, *index = count + Mp;
    float *unscale = reinterpret_cast<float *>(index + Mp), *norms = unscale + N;
    int *totals = reinterpret_cast<int *>(norms + N);
    auto *tables = reinterpret_cast<CandidateTable *>((reinterpret_cast<uintptr_t>(totals + plan.chunk) + 15) & ~(uintptr_t)15);
    auto *const R = plan.r_in_small ? reinterpret_cast<uint16_t *>(tables + plan.chunk) : Hh + (size_t)N * N;
    float *const z = w.Wt;
    const dim3 delta_grid((Mp + 63) / 64, (N + 31) / 32), rows((M + 63) / 64);
    const size_t plane = (size_t)N * Mp;
    SearchRound round = {};
    round.bound = bound;
    round.tyings = T;
    round.begin = begin;
    round.count = count;
    round.index = index;
    round.tables = tables;
    SearchList listed = {nullptr, nullptr, nullptr, tables, 0, T};
    hipError_t e = launch_fill_zero(sums, 4 * sums_floats, stream);
    if (e != hipSuccess) return e;
    for (int first = 0; first < all; first += plan.chunk) {
        const int candidates = all - first < plan.chunk ? all - first : plan.chunk;
        e = launch_fill_zero(norms, (size_t)(N + plan.chunk) * 4, stream);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(screen_h_kernel, dim3((N + 63) / 64, (N + 255) / 256), dim3(256), 0, stream, N, H, diag_max, Hh, unscale, norms);
        hipLaunchKernelGGL(screen_frobenius_kernel, dim3(1 + (N * (plan.projections / 2) + 1023) / 1024), dim3(1024), 0, stream, N, norms, frobenius, z,
                           plan.projections);
        hipLaunchKernelGGL(screen_project_kernel, dim3((N + 31) / 32), dim3(512), 0, stream, N, H, diag_max, frobenius, z, R, plan.projections);
        for (int c = 0; c < candidates;) {
            // tyings of one grid point, as many as there are planes
            const int g = (first + c) / T, t0 = (first + c) % T;
            int planes = plan.planes < T - t0 ? plan.planes : T - t0;
            planes = planes < candidates - c ? planes : candidates - c;
            TyingSet set = {};
            for (int p = 0; p < planes; ++p) set.t[p] = tyings[t0 + p];
            const auto delta = planes == 1 ? delta_single_kernel<1> : planes == 2 ? delta_single_kernel<2> : delta_single_kernel<3>;
            hipLaunchKernelGGL(delta, delta_grid, dim3(256), 0, stream, M, Mp, N, n_bits, g, grid, set, W, w.wmin, w.wmax, shift, Dh, tables + c);
            launch_screen(stream, ScreenArgs{Hh, Dh, unscale, norms, sums, N, M, Mp, planes, R, plan.projections});
            hipLaunchKernelGGL(screen_bound_kernel, dim3(rows.x, planes), dim3(64), 0, stream, M, Mp, N, sums, shift, w.wmin, w.wmax, diag_max, frobenius, plan.projections,
                               bound + (size_t)c * Mp);
            c += planes;
        }
        // As many rounds as there can be: one candidate per row, then all that are left, Mp at a time.  Nearly always the first two
        // have work, and a launch that finds an empty list ends at once.
        round.candidates = candidates;
        round.first_candidate = listed.first_candidate = first;
        for (int p = 0; p <= candidates; ++p) {
            int *const mine = list[p & 1];
            round.fresh = first == 0 && p == 0;
            round.start = p == 0;
            round.end = p == candidates;
            round.total = totals + p;
            round.last_total = totals + p - 1;
            round.row = mine;
            round.candidate = mine + Mp;
            round.last_candidate = list[(p & 1) ^ 1] + Mp;
            hipLaunchKernelGGL(search_round_kernel, rows, dim3(64), 0, stream, M, Mp, n_bits, grid, w.ntile, round, w.part, w.wmin, w.wmax,
                               w.best, S, qbias, labels);
            if (round.end) break;
            listed.count = totals + p;
            listed.row = mine;
            listed.candidate = mine + Mp;
            // (from the third round on the list is nearly always empty: fewer workgroups find that out)
            hipLaunchKernelGGL(delta_kernel<kListed>, dim3(delta_grid.x, p < 2 ? delta_grid.y : (delta_grid.y + 15) / 16), dim3(256), 0, stream, M, Mp, N, n_bits, 0, grid, Tying{}, W, w.wmin,
                               w.wmax, w.Dt, shift, Dh, plane, listed, slot_shift);
            launch_quad_form<kQuadFormSplit>(stream, Dh, plane, slot_shift, w.Dt, Mp, H, N, diag_max, N, w.part, Mp, totals + p);
        }
    }
    return hipSuccess;
}

static hipError_t search_rows(int M, int N, int n_bits, int q, int grid, const float *W, const float *H, float *S, float *qbias,
                              int8_t *labels, float *err_out, void *workspace, hipStream_t stream)
{
    const QuantWorkspace w = carve(workspace, M, N);
    // From W itself, and with d split beforehand (in place of Wt), where rows can be read eight weights at a time; else from the
    // transposed copy, and the product splits what it reads.
    const bool split = N % 8 == 0 && (reinterpret_cast<uintptr_t>(W) & 15) == 0;
    if (split) {
        hipLaunchKernelGGL(row_range_kernel, dim3((M + 3) / 4), dim3(256), 0, stream, M, N, W, w.wmin, w.wmax);
    } else {
        hipLaunchKernelGGL(transpose_kernel, dim3((N + 31) / 32, (w.Mp + 31) / 32), dim3(32, 8), 0, stream, M, w.Mp, N, W, w.Wt);
        const int chunks = N / 2 < 64 ? N / 2 : 64;  // Dt (N rows, not yet in use) holds the 2 * chunks partial rows
        hipLaunchKernelGGL(row_range_partial_kernel, dim3((M + 63) / 64, chunks), dim3(64), 0, stream, M, w.Mp, N, chunks,
                           w.Wt, w.Dt);
        hipLaunchKernelGGL(row_range_final_kernel, dim3((M + 63) / 64), dim3(64), 0, stream, M, w.Mp, chunks, w.Dt, w.wmin,
                           w.wmax);
    }
    auto *halves = reinterpret_cast<uint16_t *>(w.Wt);
    auto *shift = reinterpret_cast<int *>(w.small);
    const size_t plane = (size_t)N * w.Mp;
    auto *diag_max = reinterpret_cast<float *>(shift + w.Mp);
    hipLaunchKernelGGL(split_shift_kernel, dim3((w.Mp + 255) / 256 + 1), dim3(256), 0, stream, M, w.Mp, w.wmin, w.wmax, shift, N, H,
                       diag_max);
    const std::vector<Tying> tyings = all_tyings(n_bits, q);
    const int candidates = grid * (int)tyings.size();
    const ScreenPlan plan = split && M >= 256 && N >= 256 ? screen_plan(M, N, (int)tyings.size(), candidates) : ScreenPlan{};
    if (plan.planes > 0 && screen_pays(M, N, plan.planes, candidates)) {
        const hipError_t e = search_screened(M, N, n_bits, grid, tyings, plan, W, H, S, qbias, labels, w, stream);
        if (e != hipSuccess) return e;
    } else {
        bool first = true;
        for (int g = 0; g < grid; ++g)
            for (const Tying &t : tyings) {
                hipLaunchKernelGGL((split ? delta_kernel<kSplit> : delta_kernel<kPlain>), dim3((w.Mp + 63) / 64, (N + 31) / 32), dim3(256),
                                   0, stream, M, w.Mp, N, n_bits, g, grid, t, split ? W : w.Wt, w.wmin, w.wmax, w.Dt, shift, halves, plane,
                                   SearchList{}, nullptr);
                // d H d^T / 2 row by row: sum_l Dt[l][m] sum_{k <= l} w_kl H[k][l] Dt[k][m], w = 1/2 on the diagonal
                // (only the upper triangle of H is read), one partial per tile of 128 values of l
                (split ? launch_quad_form<kQuadFormSplit> : launch_quad_form<kQuadForm>)(stream, halves, plane, shift, w.Dt, w.Mp, H, N,
                                                                                         diag_max, N, w.part, w.Mp, nullptr);
                hipLaunchKernelGGL(keep_best_kernel, dim3((M + 255) / 256), dim3(256), 0, stream, M, w.Mp, n_bits, w.ntile, g,
                                   grid, first ? 1 : 0, t, w.part, w.wmin, w.wmax, w.best, S, qbias, labels);
                first = false;
            }
    }
    if (err_out) {
        hipError_t e = hipMemcpyAsync(err_out, w.best, (size_t)M * 4, hipMemcpyDeviceToDevice, stream);
        if (e != hipSuccess) return e;
    }
    return hipGetLastError();
}

// Rows are independent in the search and in the GPTQ pass, and both take at most this many at a time (in the same workspace): the
// products address a tile of [column][row] matrices by 32-bit byte offsets, which reach 2^23 rows, and the grids of the
// row-wise kernels have 2^16 blocks of 32 rows in their second dimension.
constexpr int kMaxRows = 1 << 20;

hipError_t launch_quant_search(int M, int N, int n_bits, int q, int grid, const float *W, const float *H, float *S,
                               float *qbias, int8_t *labels, float *err_out, void *workspace, hipStream_t stream)
{
    hipError_t e = hipSuccess;
    for (int rows; M > 0 && e == hipSuccess; M -= rows) {
        rows = M < kMaxRows ? M : kMaxRows;
        e = search_rows(rows, N, n_bits, q, grid, W, H, S, qbias, labels, err_out, workspace, stream);
        W += (size_t)rows * N;
        S += rows;
        qbias += rows;
        labels += (size_t)rows * n_bits;
        if (err_out) err_out += rows;
    }
    return e;
}

// ---------------------------------------------------------------------------------
// GPTQ pass
// ---------------------------------------------------------------------------------
// What Eq. 6 makes of every integer of a row, as a table: 16 nibbles for up to four bits, else a byte per integer.
__global__ void gptq_tables_kernel(int M, int n_bits, int q, const int8_t *__restrict__ labels,
                                   unsigned long long *__restrict__ nibbles, uint8_t *__restrict__ bytes)
{
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= M) return;
    TyingPlan plan;  // labels come from device memory the host cannot inspect: out-of-range ones are folded
    make_tying_plan(n_bits, q, labels + (size_t)m * n_bits, true, &plan);
    int choice[16];
    for (int k = 0; k < 16; ++k) choice[k] = plan.choice[k];
    unsigned long long packed = 0;
    for (int w = 0; w < 1 << n_bits; ++w) {
        const int c = nearest_choice(w, choice, 1 << q);
        if (n_bits <= 4) packed |= (unsigned long long)c << (4 * w);
        else bytes[(size_t)m * 256 + w] = (uint8_t)c;
    }
    if (n_bits <= 4) nibbles[m] = packed;
}

// A panel of up to four blocks of up to 128 columns, [p0, p1).  The columns of a row are decided one after the other, each from
// a weight that carries the compensation of all before it, so the time of a panel is the length of that chain.  Rows do not
// depend on each other: a workgroup takes 32 rows through all blocks of the panel.
// Within a block a row is spread over eight lanes (lane l holds the columns 8 i + l in registers), every lane works out the
// decision for its own column at hand, the one whose turn it is hands its deviation a = w - quant(w) to the others and all of them
// add its share -U[c][k] / U[c][c] a to their columns.  A wave takes eight rows; at 7168 rows that is one wave on nearly every
// SIMD.  Measured on such a wave: an instruction that needs the one before takes 8.5 clocks, one that does not 5.4, a DPP move
// with its wait states 17, a read of LDS 68.  So what counts is the number of dependent instructions from one decision to the
// next, nine here (eleven at four bits), and the rest goes between them:
//   * the integer, clamp(rint((w - qbias) / S)), is rounded from w / S - qbias / S with both terms off by few 2^-24: the quotient
//     lies less than 2^-22 (2^n + |qbias / S|) from the exact one, so the integer is the same unless that is so close to a half;
//   * Eq. 6 is a look-up in a table that the lane holds (a byte permutation), for more than four bits in LDS;
//   * S W_q + qbias is one multiply-add;
//   * U's rows are divided by their diagonal when they are staged: a division less on the way, and as many roundings as with
//     err = a / U[c][c] rounded.  The errors themselves, for the columns beyond the block, are divisions afterwards;
//   * the share of the column that is decided next is added straight from the lanes (a DPP operand per half of a row of 16
//     lanes), those of the others by the multiply-adds that fill the next step;
//   * a step's factors are requested from LDS a step ahead.
// The factors are zero up to the diagonal, so a weight stays as it was when its column was decided, and after the eighth step of a
// group of eight columns every lane holds the decision of its own: a group with one that is too close to a half is gone through
// again with decisions from binary64, and one with a diagonal beyond 2^-40 .. 2^40 with errors by division, too.  The
// sums are those of the first time, so that a wave's other rows come out the same.  (With U's rows read from memory again a single row
// of constant weights or with an offset of 2^20 steps took the pass of 7168 x 7168 from 2.7 to
// 8.7 and 7.9 ms, now 2.8 and 3.2.)  A wave with a row whose quotients the first way hardly ever tells goes the second way at once.
// Before a block the errors of the panel's earlier ones are applied to its columns by binary32 matrix instructions.
// The factors are staged in LDS such that the 16 of a lane for column c, those of the columns 8 (c / 8 + k) + l, come in
// up to four 16-byte reads: [c][k / 4][l][k % 4], of which columns from 32 g on need 4 - g.
constexpr int kGptqBlock = 128, kGptqRows = 32;  // columns per block, rows per workgroup
constexpr int kGptqPanel = 4 * kGptqBlock;

// Single instructions, in this order (the compiler leaves the order of volatile ones alone): d = a b + c; w += x u with x
// from lane LANE of each group of eight; x from that lane.  A DPP operand must have been written kGptqDppWait instructions before (or
// WAIT), and the compiler keeps no such distance across inline assembly.
constexpr int kGptqDppWait = 2;
#define GPTQ_FMA(d, a, b, c) asm volatile("v_fma_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c))
template <int LANE, bool WAIT>
__device__ __forceinline__ void gptq_add_from(float &w, float x, float u)
{
    if (WAIT) asm volatile("s_nop 1");
    asm volatile("v_fmac_f32_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0x3" : "+v"(w) : "v"(x), "v"(u), "n"(LANE));
    asm volatile("v_fmac_f32_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xc" : "+v"(w) : "v"(x), "v"(u), "n"(LANE + 8));
}
template <int LANE>
__device__ __forceinline__ float gptq_from(float x)
{
    float y;
    asm volatile("v_mov_b32_dpp %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0x3\n\t"
                 "v_mov_b32_dpp %0, %1 row_newbcast:%3 row_mask:0xf bank_mask:0xc" : "=&v"(y) : "v"(x), "n"(LANE), "n"(LANE + 8));
    return y;
}

constexpr int kGptqUs = 32 * 32 * (4 + 3 + 2 + 1);  // staged factors of a block

__device__ __forceinline__ bool ordinary(float d) { return fabsf(d) >= 0x1p-40f && fabsf(d) <= 0x1p40f; }

enum GptqTable { kEight = 0, kSixteen = 1, kBytes = 2 };  // integers a row can hold: up to 8, up to 16, a byte each in LDS

template <int TABLE>
struct GptqShared {
    float Us[kGptqUs + 32];
    float Ws[kGptqRows][kGptqBlock + 4];
    float diag[kGptqBlock];
    uint8_t Qs[kGptqRows][kGptqBlock + 4];
    uint8_t table[TABLE == kBytes ? kGptqRows : 1][256];
};

template <int TABLE>
__device__ __forceinline__ void gptq_panel(GptqShared<TABLE> &shared, int M, int Mp, int N, int n_bits, int p0, int p1,
                                           const float *__restrict__ Wt, const float *__restrict__ U,
                                           const float *__restrict__ S, const float *__restrict__ qbias,
                                           const unsigned long long *__restrict__ nibbles,
                                           const uint8_t *__restrict__ bytes, uint8_t *__restrict__ w_int,
                                           float *Err, float *__restrict__ least)
{
    auto &Us = shared.Us;
    auto &Ws = shared.Ws;
    auto &diag = shared.diag;
    auto &Qs = shared.Qs;
    auto &table = shared.table;
    const int tid = threadIdx.x, l = tid & 7, row = tid >> 3, m0 = blockIdx.x * kGptqRows, m = m0 + row;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool live = m < M, aligned = (reinterpret_cast<uintptr_t>(w_int) & 3) == 0;

    // U's block at c0, requested before the block before it is decided: a thread brings ten of the 16-byte pieces of Us, pieces tid +
    // 256 n (n = 0..3: columns from 0, 4..6 from 32, 7 and 8 from 64, 9 from 96), and each piece's diagonal.  Columns that do not exist
    // read others.
    float next_u[10][4], next_d[10];
    auto piece = [&](int n, int t, int *c, int *x) PROD_INLINE {  // of column c, the columns 8 (c / 8) + x + 8 j
        const int g = n < 4 ? 0 : n < 7 ? 1 : n < 9 ? 2 : 3, from = g == 0 ? 0 : g == 1 ? 4 : g == 2 ? 7 : 9;
        const int chunk = (t >> 3) + 32 * (n - from);
        *c = 32 * g + chunk / (4 - g);
        *x = 32 * (chunk % (4 - g)) + (t & 7);
    };
    auto request_u = [&](int c0, int cols) PROD_INLINE {
        int t = tid;
        asm volatile("" : "+v"(t));  // (no addresses kept in registers from block to block)
        const float *const from = U + (size_t)c0 * (N + 1);
#pragma unroll
        for (int n = 0; n < 10; ++n) {
            int c, x;
            piece(n, t, &c, &x);
            const unsigned row = c < cols ? (unsigned)c * (unsigned)N : 0u;  // (N is at most 2^15)
            next_d[n] = from[row + (c < cols ? c : 0)];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int col = (c & ~7) + x + 8 * j;
                next_u[n][j] = from[row + (col < cols ? col : 0)];
            }
        }
    };
    auto stage_u = [&](int cols) PROD_INLINE {
        int t = tid;
        asm volatile("" : "+v"(t));
#pragma unroll
        for (int n = 0; n < 10; ++n) {
            int c, x;
            piece(n, t, &c, &x);
            const float d = c < cols ? next_d[n] : 1.0f;
            if (x == 0) diag[c] = d;
            prod_f32x4 f;
            const float inv = -1.0f / d;  // quotient, remainder and correction: correctly rounded where nothing underflows
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float q = next_u[n][j] * inv;
                f[j] = fmaf(fmaf(q, d, next_u[n][j]), inv, q);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (!(x + 8 * j > (c & 7) && (c & ~7) + x + 8 * j < cols) || !ordinary(d)) f[j] = 0.0f;
            *reinterpret_cast<prod_f32x4 *>(&Us[4 * (t + 256 * n)]) = f;
        }
    };
    request_u(p0, min(kGptqBlock, p1 - p0));

    float sf = 1.0f, bf = 0.0f;
    uint32_t tab0 = 0, tab1 = 0, tab2 = 0, tab3 = 0;  // a byte per integer
    if (live) {
        sf = S[m];
        bf = qbias[m];
        if (TABLE != kBytes) {
            const unsigned long long nib = nibbles[m];
            auto spread = [&](int k) {
                const uint32_t four = (uint32_t)(nib >> (16 * k)) & 0xffffu, two = (four | (four << 8)) & 0x00ff00ffu;
                return (two | (two << 4)) & 0x0f0f0f0fu;
            };
            tab0 = spread(0); tab1 = spread(1); tab2 = spread(2); tab3 = spread(3);
        }
    }
    if (TABLE == kBytes) {
        for (int e = tid; e < kGptqRows * 256; e += 256) {
            const int r = e >> 8, mr = m0 + r;
            table[r][e & 255] = mr < M && (e & 255) < 1 << n_bits ? bytes[(size_t)mr * 256 + (e & 255)] : 0;
        }
    }
    const float topf = (float)((1 << n_bits) - 1), inv_f = sf == 0.0f ? 0.0f : 1.0f / sf, shift_f = -bf * inv_f;
    // how far a quotient may be from its integer without doubt; scales out of the ordinary leave none
    const float steps = ldexpf(1.0f, n_bits) + fabsf(shift_f);
    const float sure = sf == 0.0f ? 0.5f : fabsf(sf) >= 0x1p-60f && fabsf(sf) <= 0x1p60f ? fmaf(steps, -0x1p-22f, 0.5f) : -1.0f;
    const bool far = __any(sure < 0.46875f);  // a group of the wave would nearly always be gone through again
    constexpr float kRound = 0x1.8p23f;

    for (int c0 = p0; c0 < p1; c0 += kGptqBlock) {
        const int cols = min(kGptqBlock, p1 - c0);
        // Ws[row][column] = Wt - what the errors of the panel's earlier columns leave: wave w the columns 32 w .. 32 w + 31, 2 x 2
        // tiles of 16; element i of a tile: column 4 hi + i, row lo
        {
            prod_f32x4 acc[2][2];
#pragma unroll
            for (int a = 0; a < 4; ++a) acc[a >> 1][a & 1] = prod_f32x4{0.f, 0.f, 0.f, 0.f};
            // (rows and columns that do not exist read others, and nobody reads what they give)
            int col[2], mm[2], at = lane;
            asm volatile("" : "+v"(at));
            const int lo = at & 15, hi = at >> 4;
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                col[t] = 32 * wave + 16 * t + lo;
                col[t] = c0 + (col[t] < cols ? col[t] : 0);
                mm[t] = m0 + 16 * t + lo;
                mm[t] = mm[t] < Mp ? mm[t] : 0;
            }
            // 32 of them at a time (there are whole blocks of 128), the next ones requested before these are multiplied
            float u[2][8][2], e[2][8][2];
            auto request = [&](int k, float (&uu)[8][2], float (&ee)[8][2]) PROD_INLINE {
                const float *const from_u = U + (size_t)k * N, *const from_e = Err + (size_t)(k - p0) * Mp;
#pragma unroll
                for (int x = 0; x < 8; ++x)
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        uu[x][t] = from_u[(unsigned)(4 * x + hi) * (unsigned)N + col[t]];
                        ee[x][t] = from_e[(unsigned)(4 * x + hi) * (unsigned)Mp + mm[t]];
                    }
                __builtin_amdgcn_sched_barrier(0);
            };
            auto multiply = [&](const float (&uu)[8][2], const float (&ee)[8][2]) PROD_INLINE {
#pragma unroll
                for (int x = 0; x < 8; ++x)
#pragma unroll
                    for (int a = 0; a < 4; ++a)
                        acc[a >> 1][a & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(uu[x][a >> 1], ee[x][a & 1], acc[a >> 1][a & 1], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            };
            if (c0 > p0) request(p0, u[0], e[0]);
            for (int k = p0; k < c0; k += 64) {
                request(k + 32, u[1], e[1]);
                multiply(u[0], e[0]);
                request(k + 64 < c0 ? k + 64 : p0, u[0], e[0]);  // (behind the last ones, others that nobody uses)
                multiply(u[1], e[1]);
            }
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const int first = 32 * wave + 16 * (a >> 1) + 4 * hi;  // (a multiple of 4, as cols is)
                prod_f32x4 v = {0.f, 0.f, 0.f, 0.f};
                if (first < cols) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[i] = Wt[(size_t)(c0 + first + i) * Mp + mm[a & 1]] - acc[a >> 1][a & 1][i];
                }
                *reinterpret_cast<prod_f32x4 *>(&Ws[16 * (a & 1) + lo][first]) = v;
            }
        }
        stage_u(cols);
        __syncthreads();
        if (c0 + kGptqBlock < p1) request_u(c0 + kGptqBlock, min(kGptqBlock, p1 - c0 - kGptqBlock));
        if (blockIdx.x == 0 && tid < 64) {  // for the products with these errors: smallest diagonal of the block and of its first 32 columns
            auto size_of = [&](int c) {
                const float d = fabsf(diag[c]);
                return c < cols && d > 0.0f ? d : INFINITY;
            };
            float first = tid < 32 ? size_of(tid) : INFINITY, all = fminf(size_of(tid), size_of(tid + 64));
#pragma unroll
            for (int d = 32; d > 0; d >>= 1) {
                first = fminf(first, __shfl_xor(first, d));
                all = fminf(all, __shfl_xor(all, d));
            }
            if (tid == 0) {
                least[2 * ((c0 - p0) / kGptqBlock)] = all;
                least[2 * ((c0 - p0) / kGptqBlock) + 1] = first;
            }
        }
        float w[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) w[i] = live ? Ws[row][8 * i + l] : 0.0f;
        int odd = 0;  // groups with a diagonal out of the ordinary: by the definition, step by step
        for (int i = 0; i < 16; ++i) odd |= (int)!ordinary(diag[8 * i + l]) << i;
        odd |= __shfl_xor(odd, 1); odd |= __shfl_xor(odd, 2); odd |= __shfl_xor(odd, 4);

        // groups of eight columns, with the 4 kChunks columns of a lane that are still to come
        auto groups = [&](auto chunks_of, int i_begin) PROD_INLINE {
            constexpr int kChunks = decltype(chunks_of)::value, g = 4 - kChunks, kSlots = 4 * kChunks;
            constexpr int kAfter = kGptqDppWait;
            static_assert(kSlots - 1 >= kAfter, "a step's shares behind the deviation are the wait states of gptq_add_from");
            // factors of the step before, this step and the next (behind the last one, others that nobody uses)
            prod_f32x4 u[4][kChunks];
            auto fetch = [&](int c, prod_f32x4 (&to)[kChunks]) PROD_INLINE {
                const float *const from = Us + 32 * (32 * (4 * g - g * (g - 1) / 2) + (c - 32 * g) * kChunks) + 4 * l;
#pragma unroll
                for (int k = 0; k < kChunks; ++k) to[k] = *reinterpret_cast<const prod_f32x4 *>(from + 32 * k);
            };
            fetch(32 * g, u[0]);
#pragma unroll 1
            for (int i = i_begin; i < i_begin + 4 && 8 * i < cols; ++i) {  // (columns beyond `cols` are decided too, and dropped)
                float v[kSlots];  // the weights on the way; `w` keeps what they were before the group
                float a = 0.0f, e = 0.0f, t = 0.0f, r = 0.0f, wqf = 0.0f;
                v[0] = w[0];
                auto decide = [&](auto lane_of) PROD_INLINE {
                    constexpr int kLane = decltype(lane_of)::value;
                    __builtin_amdgcn_sched_barrier(0);
                    fetch(8 * i + kLane + 1, u[(kLane + 1) & 3]);
                    __builtin_amdgcn_sched_barrier(0);
                    // the shares of the step before, between the instructions that wait for each other; kAfter of them are
                    // kept for behind the last one, whose result DPP operands read
                    int slot = 1, end = kSlots - kAfter;
                    auto fill = [&](int count) PROD_INLINE {
#pragma unroll
                        for (int n = 0; n < count; ++n)
                            if (kLane > 0 && slot < end) {
                                GPTQ_FMA(v[slot], e, u[(kLane + 3) & 3][slot >> 2][slot & 3], kLane == 1 ? w[slot] : v[slot]);
                                ++slot;
                            }
                    };
                    constexpr int kEach = kSlots >= 16 ? 2 : kSlots >= 8 ? 1 : 0;
                    GPTQ_FMA(t, v[0], inv_f, shift_f);
                    fill(kEach);
                    asm volatile("v_med3_f32 %0, %1, 0, %2" : "=v"(t) : "v"(t), "v"(topf));
                    fill(kEach);
                    asm volatile("v_add_f32 %0, 0x4b400000, %1" : "=v"(r) : "v"(t));  // the integer in the low byte
                    if (TABLE == kBytes) {
                        wqf = (float)table[row][__float_as_uint(r) & 0xffu];
                        fill(2 * kEach);
                    } else {
                        uint32_t q;
                        if (TABLE == kSixteen) {
                            float r8;  // the integer less 8
                            uint32_t q8;
                            unsigned long long upper;
                            asm volatile("v_add_f32 %0, 0x4b3ffff8, %1" : "=v"(r8) : "v"(t));
                            asm volatile("v_cmp_lt_f32 %0, %1, %2" : "=s"(upper) : "v"(7.5f), "v"(t));
                            fill(1);
                            asm volatile("v_perm_b32 %0, %1, %2, %3" : "=v"(q) : "v"(tab1), "v"(tab0), "v"(r));
                            asm volatile("v_perm_b32 %0, %1, %2, %3" : "=v"(q8) : "v"(tab3), "v"(tab2), "v"(r8));
                            fill(1);
                            asm volatile("v_cndmask_b32 %0, %1, %2, %3" : "=v"(q) : "v"(q), "v"(q8), "s"(upper));
                        } else {
                            fill(kEach);
                            asm volatile("v_perm_b32 %0, %1, %2, %3" : "=v"(q) : "v"(tab1), "v"(tab0), "v"(r));
                        }
                        fill(kEach);
                        asm volatile("v_cvt_f32_ubyte0 %0, %1" : "=v"(wqf) : "v"(q));
                    }
                    fill(kEach);
                    float qv;
                    GPTQ_FMA(qv, sf, wqf, bf);
                    fill(end - 1 - slot);
                    asm volatile("v_sub_f32 %0, %1, %2" : "=v"(a) : "v"(v[0]), "v"(qv));
                    end = kSlots;
                    fill(kSlots);
                };
                auto step = [&](auto lane_of) PROD_INLINE {
                    constexpr int kLane = decltype(lane_of)::value;
                    decide(lane_of);
                    gptq_add_from<kLane, kLane == 0>(v[0], a, u[kLane & 3][0][0]);  // (lane 0's step has no shares)
                    e = gptq_from<kLane>(a);
                };
                bool again = far;
                if (far) {
                    fetch(8 * i + 7, u[3]);
                    fetch(8 * i + 8, u[0]);
                } else {
                    step(std::integral_constant<int, 0>{}); step(std::integral_constant<int, 1>{});
                    step(std::integral_constant<int, 2>{}); step(std::integral_constant<int, 3>{});
                    step(std::integral_constant<int, 4>{}); step(std::integral_constant<int, 5>{});
                    step(std::integral_constant<int, 6>{});
                    decide(std::integral_constant<int, 7>{});
                    // (a deviation without end has made the weights decided before it no numbers; a row of one weight, S = 0,
                    // stays what it is: any integer will do unless something was added to it)
                    const bool doubt = !(fabsf(t - (r - kRound)) < sure) || !(fabsf(a) < INFINITY) || (sf == 0.0f && a != 0.0f);
                    again = __any(doubt || ((odd >> i) & 1));
                }
                int my_q = (int)wqf;
                float last = a;
                if (__builtin_expect(again, 0)) {
                    const bool by_u = (odd >> i) & 1;  // (of all rows)
#pragma unroll
                    for (int k = 0; k < kSlots; ++k) v[k] = w[k];
                    const float near = fabsf(sf) >= 0x1p-60f && fabsf(sf) <= 0x1p60f ? 0.5f - ldexpf(1.0f, n_bits - 21) : -1.0f;
                    float from_prev = 0.0f;
#pragma unroll 1
                    for (int turn = 0; turn < 8; ++turn) {
                        prod_f32x4 f[kChunks];
                        fetch(8 * i + turn, f);
                        __builtin_amdgcn_sched_barrier(0);
                        // the difference is off by 2^-24 of itself, so this quotient by less than 2^(n - 21), whatever qbias is
                        const float tq = fminf(fmaxf((v[0] - bf) * inv_f, 0.0f), topf), rq = rintf(tq);
                        int lin = (int)rq;
                        if (__any(!(fabsf(tq - rq) < near))) lin = linear_int((double)v[0] - (double)bf, sf, 1.0 / (double)sf, topf);
                        int wq;
                        if (TABLE == kBytes) wq = table[row][lin];
                        else wq = (int)((lin & 8 ? (lin & 4 ? tab3 : tab2) : (lin & 4 ? tab1 : tab0)) >> (8 * (lin & 3))) & 0xff;
                        const float now = v[0] - fmaf(sf, (float)wq, bf);
                        my_q = l == turn ? wq : my_q;
                        a = l == turn ? now : a;
                        from_prev = __shfl(now, turn, 8);
                        if (turn == 7) break;
                        const int c = 8 * i + turn;
                        if (by_u) {
                            const float err = from_prev / diag[c];
                            const float *const of_u = U + (size_t)(c0 + c) * N + c0 + 8 * i + l;
#pragma unroll
                            for (int k = 0; k < kSlots; ++k)
                                if (8 * k + l > turn && 8 * (i + k) + l < cols) v[k] = fmaf(-err, of_u[8 * k], v[k]);
                        } else {
                            if (l > turn) v[0] = fmaf(from_prev, f[0][0], v[0]);
#pragma unroll
                            for (int k = 1; k < kSlots; ++k) v[k] = fmaf(from_prev, f[k >> 2][k & 3], v[k]);
                        }
                    }
                    last = a;
                    if (by_u) {  // the last column's share too
                        last = 0.0f;
                        const float err = from_prev / diag[8 * i + 7];
                        const float *const of_u = U + (size_t)(c0 + 8 * i + 7) * N + c0 + 8 * i + l;
#pragma unroll
                        for (int k = 1; k < kSlots; ++k)
                            if (8 * (i + k) + l < cols) v[k] = fmaf(-err, of_u[8 * k], v[k]);
                    }
                }
                // the last column's share, and every lane goes on to its next column
                gptq_add_from<7, true>(v[1], last, u[3][0][1]);
                e = gptq_from<7>(last);
                w[0] = v[1];
#pragma unroll
                for (int k = 2; k < kSlots; ++k) GPTQ_FMA(w[k - 1], e, u[3][k >> 2][k & 3], v[k]);
                Ws[row][8 * i + l] = a;
                Qs[row][8 * i + l] = (uint8_t)my_q;
            }
        };
        groups(std::integral_constant<int, 4>{}, 0);
        groups(std::integral_constant<int, 3>{}, 4);
        groups(std::integral_constant<int, 2>{}, 8);
        groups(std::integral_constant<int, 1>{}, 12);
        __syncthreads();
        // the block's errors and integers, each division beside others
        {
            int t = tid;
            asm volatile("" : "+v"(t));
            const int r = t & 31, first = t >> 5, mr = m0 + r;
#pragma unroll
            for (int k = 0; k < kGptqBlock / 8; ++k) {
                const int c = first + 8 * k;
                const float err = Ws[r][c] / diag[c];
                if (c < cols && mr < Mp) Err[(size_t)(c0 - p0 + c) * Mp + mr] = mr < M ? err : 0.0f;  // zeros in the pad rows
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int c = 4 * (8 * k + l);  // (cols, N and c0 are multiples of 4)
                const uint32_t four = *reinterpret_cast<const uint32_t *>(&Qs[row][c]);
                if (live && c < cols) {
                    uint8_t *const to = w_int + (size_t)m * N + c0 + c;
                    if (aligned) *reinterpret_cast<uint32_t *>(to) = four;
                    else for (int j = 0; j < 4; ++j) to[j] = (uint8_t)(four >> (8 * j));
                }
            }
        }
        __syncthreads();  // the errors are in memory, and everyone is done with U's block and Ws
    }
}

// The first `rows_groups` workgroups (a multiple of 8: workgroup numbers go round the XCDs) take the panel [p0, p1), 32 rows each; the
// others the tiles of `rest`, the update of the columns beyond the panel by the errors of the panel before.  A panel is a chain that
// leaves most of the chip's instruction slots and power unused, the update is what uses them.  The panel's waves go
// first where both want to issue.
template <int TABLE>
__global__ __launch_bounds__(256, 2) void gptq_panel_kernel(int M, int Mp, int N, int n_bits, int p0, int p1, int row_groups,
                                                            const float *__restrict__ Wt, const float *__restrict__ U,
                                                            const float *__restrict__ S, const float *__restrict__ qbias,
                                                            const unsigned long long *__restrict__ nibbles,
                                                            const uint8_t *__restrict__ bytes, uint8_t *__restrict__ w_int,
                                                            float *Err, float *__restrict__ least, ProductArgs rest)
{
    constexpr size_t kPanel = sizeof(GptqShared<TABLE>), kProduct = sizeof(ProductShared);
    __shared__ __attribute__((aligned(16))) uint8_t shared[kPanel > kProduct ? kPanel : kProduct];
    if ((int)blockIdx.x < row_groups) {
        if ((int)blockIdx.x * kGptqRows >= Mp) return;
        __builtin_amdgcn_s_setprio(3);
        gptq_panel<TABLE>(*reinterpret_cast<GptqShared<TABLE> *>(shared), M, Mp, N, n_bits, p0, p1, Wt, U, S, qbias, nibbles, bytes, w_int,
                          Err, least);
    } else {
        ProductShared &s = *reinterpret_cast<ProductShared *>(shared);
        product_tile_of<kSubtract>(rest, blockIdx.x - row_groups, gridDim.x - row_groups, s.stage_a0, s.stage_a1, s.stage_b, s.largest,
                                   s.largest_of_tile, s.shift);
    }
}

// Columns beyond a panel of four blocks are brought up to date once per panel (K = 512): every pass over the remaining weights
// reads and writes them all, which at one pass per block was most of its time (5.7 ms of a 7168 x 7168 layer, now 1.7).  The panel's own
// columns are its kernel's: with a launch per block and a product for the rest of the panel after each, 38 us a block, now 22 (a panel of
// 7168 rows, four bits: updates 25 us, chains 42, staging, errors and integers 20).  Only the next panel's columns are updated before it
// starts (33 us); the update of those beyond runs beside it, in the same launch: 3.05 -> 2.67 ms, 3.78 with none of this.  So the errors
// of two panels are kept, by turns, in Dt, which the pass does not use otherwise.
//
// Few far columns are updated before the panel with the next ones instead: the extra launch is not made up for (us, all before / from
// this many tiles on beside: 4096 x 4096 1312 / 1280, 7168 x 4096 1398 / 1286, 7168 x 7168 2814 / 2680; from 1200 on 1317, 1362, 2710).
constexpr int kBesideTiles = 600;

static hipError_t gptq_rows(int M, int N, int n_bits, int q, const float *W, const float *U, const float *S, const float *qbias,
                            const int8_t *labels, uint8_t *w_int, void *workspace, hipStream_t stream)
{
    const QuantWorkspace w = carve(workspace, M, N);
    auto *nibbles = reinterpret_cast<unsigned long long *>(w.part);  // two of the (ceil(N / 128) + 3) Mp floats from here
    auto *bytes = reinterpret_cast<uint8_t *>(w.small);              // 256 of the 512 bytes per row
    float *const leasts = w.small + 64 * (size_t)w.Mp;               // 2 x 8 floats: smallest diagonals of the blocks of two panels
    hipLaunchKernelGGL(transpose_kernel, dim3((N + 31) / 32, (w.Mp + 31) / 32), dim3(32, 8), 0, stream, M, w.Mp, N, W,
                       w.Wt);
    hipLaunchKernelGGL(gptq_tables_kernel, dim3((M + 63) / 64), dim3(64), 0, stream, M, n_bits, q, labels, nibbles, bytes);
    const auto panel = n_bits <= 3 ? gptq_panel_kernel<kEight> : n_bits == 4 ? gptq_panel_kernel<kSixteen> : gptq_panel_kernel<kBytes>;
    const int row_groups = ((w.Mp + kGptqRows - 1) / kGptqRows + 7) / 8 * 8;
    for (int p0 = 0, turn = 0; p0 < N; p0 += kGptqPanel, turn ^= 1) {
        const int p1 = p0 + kGptqPanel < N ? p0 + kGptqPanel : N;
        float *const err = w.Dt + (size_t)(turn * kGptqPanel) * w.Mp, *const last = w.Dt + (size_t)((turn ^ 1) * kGptqPanel) * w.Mp;
        float *const least = leasts + 8 * turn, *const last_least = leasts + 8 * (turn ^ 1);
        // Wt[k][m] -= sum_j U[j][k] Err[j][m] for the errors j of the panel before and the columns k of [from, to)
        auto update = [&](int from, int to) {
            return product_args(U + (size_t)(p0 - kGptqPanel) * N + from, N, to - from, last, w.Mp, w.Mp, kGptqPanel,
                                w.Wt + (size_t)from * w.Mp, w.Mp, last_least);
        };
        ProductArgs rest = {};
        int tiles = 0;
        if (p0 > 0) {
            const bool beside = product_groups<kSubtract>(N - p1, w.Mp) >= kBesideTiles;
            const int to = beside ? p1 : N;
            hipLaunchKernelGGL(product_kernel<kSubtract>, dim3((unsigned)product_groups<kSubtract>(to - p0, w.Mp)), dim3(256), 0, stream,
                               update(p0, to));
            if (beside) {
                rest = update(p1, N);
                tiles = product_groups<kSubtract>(N - p1, w.Mp);
            }
        }
        hipLaunchKernelGGL(panel, dim3((unsigned)(row_groups + tiles)), dim3(256), 0, stream, M, w.Mp, N, n_bits, p0, p1, row_groups, w.Wt, U,
                           S, qbias, nibbles, bytes, w_int, err, least, rest);
    }
    return hipGetLastError();
}

hipError_t launch_quant_gptq(int M, int N, int n_bits, int q, const float *W, const float *U, const float *S,
                             const float *qbias, const int8_t *labels, uint8_t *w_int, void *workspace,
                             hipStream_t stream)
{
    hipError_t e = hipSuccess;
    for (int rows; M > 0 && e == hipSuccess; M -= rows) {
        rows = M < kMaxRows ? M : kMaxRows;
        e = gptq_rows(rows, N, n_bits, q, W, U, S, qbias, labels, w_int, workspace, stream);
        W += (size_t)rows * N;
        S += rows;
        qbias += rows;
        labels += (size_t)rows * n_bits;
        w_int += (size_t)rows * N;
    }
    return e;
}

// ---------------------------------------------------------------------------------
// fusion with one tying per row (row-wise parameters: one scaling group per row)
// ---------------------------------------------------------------------------------
// A workgroup takes up to 16 rows (fewer where that would leave the chip idle): one thread per row works out its tying, all
// at the same time (a sort each), all threads fill one table of codes per row, and the rows are then mapped WIDTH weights
// (1, 4 or 16, by the alignment) at a time.  Bound: memory.  28672 x 7168: 441 us (a workgroup per row whose first thread worked out the tying, a scan of the representable
// set per weight) -> 78 us with the plan worked out in LDS, 74 in registers, 411 MB: 5.5 TB/s; 512 x 64: 8.3 -> 10.8 -> 7.0 us.
// Many integers are read past the caches (PAST, nontemporal): nobody reads them again, and what the packing reads next, the codes, stays in
// the 256 MB last-level cache instead.  Both calls together, plain / nontemporal: 16 Mi integers 18.9 / 21.0 us, 32 Mi 26.2 / 28.5, 59 Mi
// 46.9 / 46.4, 78 Mi 59.4 / 58.2, 98 Mi 77.4 / 69.7, 117 Mi 93.8 / 82.9, 196 Mi 134.2 / 130.2 (one tying for all rows 17.1 / 18.4, 25.2 / 27.2,
// 43.4 / 43.4, 55.8 / 53.9, 72.2 / 66.8, 82.6 / 81.2, 136.5 / 130.5): the line is 2^26, where they are equal.
constexpr int kFuseRows = 16;
template <int WIDTH, bool PAST>
__global__ __launch_bounds__(256) void from_linear_rows_kernel(int M, int N, int per_group, int n_bits, int q,
                                                               const int8_t *__restrict__ labels,
                                                               const uint8_t *__restrict__ w_int, const float *__restrict__ S,
                                                               const float *__restrict__ qbias, uint8_t *__restrict__ codes,
                                                               uint16_t *__restrict__ alpha, uint16_t *__restrict__ offset)
{
    const int m0 = blockIdx.x * per_group, rows = M - m0 < per_group ? M - m0 : per_group, tid = threadIdx.x;
    __shared__ TyingPlan plan[kFuseRows];
    __shared__ __attribute__((aligned(4))) uint8_t table[kFuseRows][1 << kMaxBits];
    if (tid < rows) {
        const int m = m0 + tid;
        TyingPlan mine;
        make_tying_plan(n_bits, q, labels + (size_t)m * n_bits, true, &mine);
        plan[tid] = mine;
        const double s = S[m];
#pragma unroll
        for (int o = 0; o < kMaxQ; ++o)
            if (o < q) alpha[(size_t)m * q + o] = double_to_half_bits(s * mine.alpha_hat[o]);
        offset[m] = double_to_half_bits(((1 << n_bits) - 1) / 2.0 * s + (double)qbias[m]);
    }
    __syncthreads();
    for (int e = tid; e < rows << n_bits; e += 256) {
        const TyingPlan &p = plan[e >> n_bits];
        const int w = e & ((1 << n_bits) - 1);
        table[e >> n_bits][w] = code_of(nearest_choice(w, p.choice, p.nchoice), p, q);  // Eq. 6 (members pass unchanged)
    }
    __syncthreads();
    const uint32_t mask = ((1u << n_bits) - 1u) * 0x01010101u;
    const unsigned per_row = (unsigned)N / WIDTH;  // N is a multiple of WIDTH
    for (int r = 0; r < rows; ++r) {
        const size_t row = (size_t)(m0 + r) * N;
        const uint8_t *const lut = table[r];
        for (unsigned k = tid; k < per_row; k += 256) {
            const size_t at = row + (size_t)k * WIDTH;
            if constexpr (WIDTH == 16) {
                const auto *const src = reinterpret_cast<const prod_u32x4 *>(w_int + at);
                const prod_u32x4 w = PAST ? __builtin_nontemporal_load(src) : *src;
                uint4 c;
                c.x = map_codes(lut, w.x, mask); c.y = map_codes(lut, w.y, mask);
                c.z = map_codes(lut, w.z, mask); c.w = map_codes(lut, w.w, mask);
                *reinterpret_cast<uint4 *>(codes + at) = c;
            } else if constexpr (WIDTH == 4) {
                *reinterpret_cast<uint32_t *>(codes + at) = map_codes(lut, *reinterpret_cast<const uint32_t *>(w_int + at), mask);
            } else {
                codes[at] = lut[w_int[at] & (mask & 0xffu)];
            }
        }
    }
}

hipError_t launch_from_linear_rows(int M, int N, int n_bits, int q, const int8_t *labels, const uint8_t *w_int,
                                   const float *S, const float *qbias, uint8_t *codes, uint16_t *alpha,
                                   uint16_t *offset, hipStream_t stream)
{
    const uintptr_t both = reinterpret_cast<uintptr_t>(w_int) | reinterpret_cast<uintptr_t>(codes);
    const bool past = (size_t)M * N > kReadPastCaches;
    const auto kernel = N % 16 == 0 && both % 16 == 0 ? (past ? from_linear_rows_kernel<16, true> : from_linear_rows_kernel<16, false>)
                        : both % 4 == 0               ? from_linear_rows_kernel<4, false> : from_linear_rows_kernel<1, false>;  // N % 4 == 0
    int per_group = M / 2048;  // at least about 2048 workgroups, eight per compute unit
    per_group = per_group < 1 ? 1 : (per_group > kFuseRows ? kFuseRows : per_group);
    hipLaunchKernelGGL(kernel, dim3((M + per_group - 1) / per_group), dim3(256), 0, stream, M, N, per_group, n_bits, q, labels,
                       w_int, S, qbias, codes, alpha, offset);
    return hipGetLastError();
}

}  // namespace bcq
