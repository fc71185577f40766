// Tiles of the fp32 path on the fp64 matrix instruction (see f32_kernels.hip), and its low-rank products, which the preparation
// kernel runs beside its own work.
#pragma once
#include "plora_internal.h"

namespace plora {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));   // rows of any length: 4-byte aligned

constexpr int F32_CK = 32;                 // contraction elements per chunk

// Operand fragment of one chunk for 16 rows (or columns): lane (i = lane % 16, q = lane / 16) holds, of row i, the
// elements k0 + 16 s + 4 q + j in v[4 s + j].  MFMA step (s, j) then contracts the four k of its four lane groups; both
// operands number k the same way, so which k a step takes does not matter.
// An operand is addressed by a uniform pointer, which the chunk moves, and a byte offset of the lane, which stays: registers
// decide how many workgroups share a compute unit, and with them how much of the latency is hidden.
// k contiguous in memory: base = row 0 of the tile; off: the lane's row, in bytes, plus 16 q
__device__ inline void frag_k_contiguous(const float *base, uint32_t off, int64_t k0, int64_t n_k, int q, float *v)
{
    const char *p = reinterpret_cast<const char *>(base + k0);
    if (k0 + F32_CK <= n_k) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const f32x4_a4 t = *reinterpret_cast<const f32x4_a4 *>(p + 64 * s + off);
#pragma unroll
            for (int j = 0; j < 4; ++j) v[4 * s + j] = t[j];
        }
        return;
    }
    const int left = (int)(n_k - k0) - 4 * q;                         // elements of the lane's row from its first on
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int e = 16 * s + j;
            const float t = *reinterpret_cast<const float *>(p + (int64_t)off + 4 * (e < left ? e : -4 * q));   // past the end: the row's first, not used
            v[4 * s + j] = e < left ? t : 0.f;
        }
}

// k is the row index of a [n_k][ld] matrix: base = row 0; off: the lane's column, in bytes, plus 4 q rows
__device__ inline void frag_k_rows(const float *base, uint32_t off, int64_t ld, int64_t k0, int64_t n_k, int q, float *v)
{
    const char *p = reinterpret_cast<const char *>(base + k0 * ld);
    if (k0 + F32_CK <= n_k) {
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int j = 0; j < 4; ++j) v[4 * s + j] = *reinterpret_cast<const float *>(p + (16 * s + j) * ld * 4 + off);
        return;
    }
    const int left = (int)(n_k - k0) - 4 * q;
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int e = 16 * s + j;
            const float t = *reinterpret_cast<const float *>(p + (int64_t)off + (e < left ? e : -4 * q) * ld * 4);
            v[4 * s + j] = e < left ? t : 0.f;
        }
}

template <int RB, int CB>
__device__ inline void multiply_chunk(const float (*a)[8], const float (*b)[8], f64x4 (*acc)[CB])
{
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        double bd[CB];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) bd[cb] = (double)b[cb][e];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const double ad = (double)a[rb][e];
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) acc[rb][cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(ad, bd[cb], acc[rb][cb], 0, 0, 0);
        }
    }
}

// In front of the first vector-ALU read of a matrix instruction's sums.  The compiler pads that distance itself, but not where
// the two meet at a join of branches: a loop that kept its sums in accumulation registers read the last of them one instruction
// behind the product (seen in its assembly; rows 12 to 15 of a tile were wrong).  The kernels below are therefore bounded to two
// waves per SIMD, at which the compiler leaves the sums in vector registers (build.py refuses anything else), and wait here.
template <int RB, int CB> __device__ inline void settle(f64x4 (*acc)[CB])
{
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) asm volatile("s_nop 15\n\ts_nop 7" : "+v"(acc[rb][cb]));
}

// Chunks first, first + step, ... of a contraction with n_k elements; load_a(k0, a) and load_b(k0, b) fetch the operands
// of a chunk.  The next chunk is requested before the current one is multiplied.
template <int RB, int CB, class LA, class LB>
__device__ inline void contract(int first, int step, int64_t n_k, const LA &load_a, const LB &load_b, f64x4 (*acc)[CB])
{
    const int n_chunks = (int)((n_k + F32_CK - 1) / F32_CK);
    if (first >= n_chunks) return;
    float a[RB][8], b[CB][8], an[RB][8], bn[CB][8];
    load_a((int64_t)first * F32_CK, a);
    load_b((int64_t)first * F32_CK, b);
    for (int c = first; c < n_chunks; c += step) {
        const bool more = c + step < n_chunks;
        if (more) {
            load_a((int64_t)(c + step) * F32_CK, an);
            load_b((int64_t)(c + step) * F32_CK, bn);
        }
        multiply_chunk<RB, CB>(a, b, acc);
        if (more) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) a[rb][e] = an[rb][e];
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) b[cb][e] = bn[cb][e];
            }
        }
    }
}

template <int RB, int CB> __device__ inline void clear(f64x4 (*acc)[CB])
{
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) acc[rb][cb] = f64x4{0.0, 0.0, 0.0, 0.0};
}

// Sum of the waves' tiles, in wave order, handed to store(row, column, value) by element (columns fastest over threads).
// The matrix instruction leaves row q + 4 i, column lane % 16 of a 16 x 16 block in element i of lane (q, lane % 16).
template <int RB, int CB, int NW, class ST>
__device__ inline void sum_waves(f64x4 (*acc)[CB], double *lds, const ST &store)
{
    settle<RB, CB>(acc);
    constexpr int ROWS = 16 * RB, COLS = 16 * CB;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i16 = lane & 15, q = lane >> 4;
    double *mine = lds + wave * (ROWS * COLS);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int i = 0; i < 4; ++i) mine[(rb * 16 + q + 4 * i) * COLS + cb * 16 + i16] = acc[rb][cb][i];
    __syncthreads();
    for (int e = threadIdx.x; e < ROWS * COLS; e += 64 * NW) {
        double v = lds[e];
#pragma unroll
        for (int w = 1; w < NW; ++w) v += lds[w * (ROWS * COLS) + e];
        store(e / COLS, e % COLS, v);
    }
    __syncthreads();
}

__device__ inline int64_t readlane64(int64_t v, int l)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), l);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// ---- low-rank products: 16 tokens x 16 ranks per workgroup, four waves ---------------------------------------------------
// mode 0: out[t][j] = sum_c x[t][c] A_k[c][j]              (low-rank activation h, unscaled)
// mode 1: out[t][j] = scale_k sum_c dy[t][c] B_k[j][c]     (gradient case 2)
// out is the ragged [len][r] fp32 layout; t0: first token inside the segment, j0: first rank, M: A_k or B_k.
constexpr int F32_NW = 4;
__device__ inline void f32_lowrank_tile(const F32LowRank &job, const SegInfo &g, float scale, const float *M, int t0, int j0, double *lds)
{
    const int len = g.row1 - g.row0, r = g.r, mode = job.mode;
    if (t0 >= len || j0 >= r) return;
    const int64_t C = job.C;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), i16 = lane & 15, q = lane >> 4;
    const int t = t0 + i16 < len ? t0 + i16 : len - 1;              // clamped rows and columns are not stored
    const int j = j0 + i16 < r ? j0 + i16 : r - 1;
    const float *rows = job.S + (int64_t)(g.row0 + t0) * C;
    const uint32_t off_x = ((uint32_t)(t - t0) * (uint32_t)C + 4 * q) * 4u;       // 15 rows of at most 2^22 elements
    const uint32_t off_m = mode == 0 ? ((uint32_t)(4 * q * r) + (uint32_t)j) * 4u : ((uint32_t)(j - j0) * (uint32_t)C + 4 * q) * 4u;
    f64x4 acc[1][1];
    clear<1, 1>(acc);
    auto load_a = [&](int64_t k0, float (*v)[8]) { frag_k_contiguous(rows, off_x, k0, C, q, v[0]); };
    auto load_b = [&](int64_t k0, float (*v)[8]) {
        if (mode == 0) frag_k_rows(M, off_m, r, k0, C, q, v[0]);
        else frag_k_contiguous(M + (int64_t)j0 * C, off_m, k0, C, q, v[0]);
    };
    contract<1, 1>(wave, F32_NW, C, load_a, load_b, acc);
    const double mult = mode == 0 ? 1.0 : (double)scale;
    sum_waves<1, 1, F32_NW>(acc, lds, [&](int rr, int cc, double v) {
        if (t0 + rr < len && j0 + cc < r) job.out[g.h_off + (int64_t)(t0 + rr) * r + j0 + cc] = (float)(v * mult);
    });
}

}  // namespace plora
