// Tiles of the fp32 path on the fp64 matrix instruction (see f32_kernels.hip), and its low-rank products, which the preparation
// kernel runs beside its own work.
#pragma once
#include "plora_internal.h"

namespace plora {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));   // rows of any length: 4-byte aligned

constexpr int F32_CK = 16;                 // contraction elements per chunk

// NB blocks of 16 rows (or columns) of an operand.  Fragment of one chunk: lane (i = lane % 16, q = lane / 16) holds, of row i,
// the elements k0 + 4 q + j in v[block][j].  MFMA step j then contracts the four k of its four lane groups; both operands
// number k the same way, so which k a step takes does not matter.
// An operand is addressed by a uniform pointer, which the chunk moves, and a byte offset of the lane, which stays: registers
// decide how many workgroups share a compute unit, and with them how much of the latency is hidden.
// ROWS true: k is the row index of a [n_k][ld] matrix, 16 lanes read 64 bytes of a row.  false: k contiguous in memory, base =
// row 0 of the tile, rows ld apart; there the four lanes that read the 64 bytes of a row are neighbours (one access to the
// L1 instead of four) and the elements go to their lanes afterwards.
template <bool ROWS, int NB> struct F32Operand {
    const float *base;
    int64_t ld;
    uint32_t off[NB];                      // bytes; of 31 rows of at most 2^22 elements, or 15 rows and a column
    // row (or column) of the tile whose offset the lane keeps, and its place in the chunk, in elements
    __device__ static inline int own_row() { const int lane = threadIdx.x & 63; return ROWS ? lane & 15 : lane >> 2; }
    __device__ static inline int own_k() { const int lane = threadIdx.x & 63; return 4 * (ROWS ? lane >> 4 : lane & 3); }
    // i: own_row() of block b, clamped to the rows that there are
    __device__ inline void row(int b, int i) { off[b] = ROWS ? ((uint32_t)own_k() * (uint32_t)ld + (uint32_t)i) * 4u : ((uint32_t)i * (uint32_t)ld + (uint32_t)own_k()) * 4u; }
    // the chunk k0 .. k0 + F32_CK - 1, all of it there
    __device__ inline void load(int64_t k0, float (*v)[4]) const
    {
        const char *p = reinterpret_cast<const char *>(ROWS ? base + k0 * ld : base + k0);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            if (ROWS) {
#pragma unroll
                for (int j = 0; j < 4; ++j) v[b][j] = *reinterpret_cast<const float *>(p + j * ld * 4 + off[b]);
            } else {
                const f32x4_a4 t = *reinterpret_cast<const f32x4_a4 *>(p + off[b]);
#pragma unroll
                for (int j = 0; j < 4; ++j) v[b][j] = t[j];
            }
        }
    }
    // the elements of a chunk that are among the contraction's n_k, zeros for the others
    __device__ inline void load_part(int64_t k0, int64_t n_k, float (*v)[4]) const
    {
        const char *p = reinterpret_cast<const char *>(ROWS ? base + k0 * ld : base + k0);
        const int left = (int)(n_k - k0);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool in = own_k() + j < left;
            const int step = (in ? j : -own_k()) * (ROWS ? (int)ld : 1);      // past the end: the row's first, not used
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const float t = *reinterpret_cast<const float *>(p + (off[b] + (uint32_t)step * 4u));
                v[b][j] = in ? t : 0.f;
            }
        }
    }
    // from the lanes that loaded the elements to those that multiply them
    __device__ static inline void arrange(float (*v)[4])
    {
        if (ROWS) return;
        const int lane = threadIdx.x & 63, from = 4 * (4 * (lane & 15) + (lane >> 4));
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int j = 0; j < 4; ++j) v[b][j] = __int_as_float(__builtin_amdgcn_ds_bpermute(from, __float_as_int(v[b][j])));
    }
};

template <int RB, int CB>
__device__ inline void multiply_chunk(const float (*a)[4], const float (*b)[4], f64x4 (*acc)[CB])
{
#pragma unroll
    for (int e = 0; e < 4; ++e) {
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
// behind the product (seen in its assembly; rows 12 to 15 of a tile were wrong).  The kernels of this path are therefore bounded
// to four waves per SIMD (k_f32_lowrank: two), at which the compiler leaves the sums in vector registers (build.py refuses anything else), and wait here.
template <int RB, int CB> __device__ inline void settle(f64x4 (*acc)[CB])
{
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) asm volatile("s_nop 15\n\ts_nop 7" : "+v"(acc[rb][cb]));
}

// The pairs of chunks first, first + step, ... (a pair is a line of 128 bytes where k is contiguous) of a contraction with n_k
// elements.  DEPTH chunks are held, so DEPTH - 1 are in flight while one is multiplied; behind the last one the last is
// requested again: a request under a condition would make every wait one for all that is in flight.  A last chunk that is not
// whole starts earlier and leaves out what the chunk before it held.
template <int RB, int CB, int DEPTH, class OA, class OB>
__device__ inline void contract(int first, int step, int64_t n_k, const OA &oa, const OB &ob, f64x4 (*acc)[CB])
{
    const int q = (threadIdx.x & 63) >> 4;
    float a[DEPTH][RB][4], b[DEPTH][CB][4];
    if (n_k < F32_CK) {
        if (first != 0 || n_k <= 0) return;
        oa.load_part(0, n_k, a[0]);
        ob.load_part(0, n_k, b[0]);
        oa.arrange(a[0]);
        ob.arrange(b[0]);
        multiply_chunk<RB, CB>(a[0], b[0], acc);
        return;
    }
    const int n_chunks = (int)((n_k + F32_CK - 1) / F32_CK), n_pairs = (n_chunks + 1) / 2;
    if (first >= n_pairs) return;
    const int own = (n_pairs - 1 - first) / step;                     // pairs of this wave behind its first
    const int n = 2 * own + (2 * (first + own * step) + 1 < n_chunks ? 2 : 1);
    auto start = [&](int i) {                                          // of the wave's chunk i
        const int c = 2 * (first + (i >> 1) * step) + (i & 1);
        const int64_t k0 = (int64_t)c * F32_CK, k_last = n_k - F32_CK;
        return k0 < k_last ? k0 : k_last;
    };
#pragma unroll
    for (int u = 0; u < DEPTH - 1; ++u) {
        const int64_t k0 = start(u < n ? u : n - 1);
        oa.load(k0, a[u]);
        ob.load(k0, b[u]);
    }
    for (int i0 = 0; i0 < n; i0 += DEPTH) {
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) {
            const int i = i0 + u, ahead = i + DEPTH - 1 < n ? i + DEPTH - 1 : n - 1;
            const int64_t k0 = start(ahead);
            oa.load(k0, a[(u + DEPTH - 1) % DEPTH]);
            ob.load(k0, b[(u + DEPTH - 1) % DEPTH]);
            if (i < n) {
                const int c = 2 * (first + (i >> 1) * step) + (i & 1);
                const int skip = (int)((int64_t)(c + 1) * F32_CK - n_k) - 4 * q;
                oa.arrange(a[u]);
                ob.arrange(b[u]);
                if (c == n_chunks - 1) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
#pragma unroll
                        for (int rb = 0; rb < RB; ++rb) a[u][rb][j] = j < skip ? 0.f : a[u][rb][j];
#pragma unroll
                        for (int cb = 0; cb < CB; ++cb) b[u][cb][j] = j < skip ? 0.f : b[u][cb][j];
                    }
                }
                multiply_chunk<RB, CB>(a[u], b[u], acc);
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
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    f64x4 acc[1][1];
    clear<1, 1>(acc);
    auto clamped = [](int i, int n) { return i < n ? i : n - 1; };   // rows and columns past the end are not stored
    F32Operand<false, 1> rows{job.S + (int64_t)(g.row0 + t0) * C, C, {}};
    rows.row(0, clamped(rows.own_row(), len - t0));
    if (mode == 0) {
        F32Operand<true, 1> m{M + j0, r, {}};
        m.row(0, clamped(m.own_row(), r - j0));
        contract<1, 1, 6>(wave, F32_NW, C, rows, m, acc);
    } else {
        F32Operand<false, 1> m{M + (int64_t)j0 * C, C, {}};
        m.row(0, clamped(m.own_row(), r - j0));
        contract<1, 1, 6>(wave, F32_NW, C, rows, m, acc);
    }
    const double mult = mode == 0 ? 1.0 : (double)scale;
    sum_waves<1, 1, F32_NW>(acc, lds, [&](int rr, int cc, double v) {
        if (t0 + rr < len && j0 + cc < r) job.out[g.h_off + (int64_t)(t0 + rr) * r + j0 + cc] = (float)(v * mult);
    });
}

}  // namespace plora
