// fp32 I/O path of the packed multi-LoRA layer.  Inputs and outputs are fp32; every sum is accumulated in fp64 and rounded
// once, so the result is within an ulp or two of the exact value for any problem size.
//
// Every product runs on the fp64 matrix instruction (16x16x4): its rate is that of the vector ALU's fp64 FMA, but one
// instruction replaces sixteen per lane and an operand element is converted once per 16 outputs.  The problems of this path
// are small (the fp32 configuration: 256 tokens, 256 x 256, 72 MFLOP in six launches), so latency bounds it and the shape of
// the kernels follows from that: small output tiles for many workgroups, the contraction of a tile dealt to its waves in
// chunks of 32, operands straight from memory into registers (no staging, no barrier until the waves' sums meet in LDS), the
// next chunk in flight while one is multiplied.  Measured (256-token configuration, then 777 tokens, 500 -> 750, in us):
// low-rank products 69 and 498 with one dot product per thread, now 5.6 and 8.2; base products 49 and 145 with 64 x 64 tiles
// on the vector ALU, now 10.7 and 27; the two weight gradients 63 and 216 with one dot product per thread in two launches,
// now 5.4 and 9.0 in one.  The whole step: 322 -> 45 and 1948 -> 95.  Larger ones, 4 adapters of rank 16, both weight orders
// alike: 1024 tokens, 1024 -> 1024 2.46 -> 0.16 ms; 4096 tokens, 4096 -> 4096 18.3 -> 5.8 ms (base products 4.5 -> 2.6 - 3.0 each, 46 -
// 53 TFLOP/s of the nominal 78.6); 8192 tokens, 2048 -> 2048, 8 adapters of rank 64 33 -> 3.2 ms.
#include "plora_internal.h"

namespace plora {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));   // rows of any length: 4-byte aligned

constexpr int F32_CK = 32;                 // contraction elements per chunk

// Operand fragment of one chunk for 16 rows (or columns): lane (i = lane % 16, q = lane / 16) holds, of row i, the
// elements k0 + 16 s + 4 q + j in v[4 s + j].  MFMA step (s, j) then contracts the four k of its four lane groups; both
// operands number k the same way, so which k a step takes does not matter.
// k contiguous in memory: `row` is the lane's row
__device__ inline void frag_k_contiguous(const float *row, int64_t k0, int64_t n_k, int q, float *v)
{
    if (k0 + F32_CK <= n_k) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const f32x4_a4 t = *reinterpret_cast<const f32x4_a4 *>(row + k0 + 16 * s + 4 * q);
#pragma unroll
            for (int j = 0; j < 4; ++j) v[4 * s + j] = t[j];
        }
        return;
    }
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t k = k0 + 16 * s + 4 * q + j;
            v[4 * s + j] = k < n_k ? row[k] : 0.f;
        }
}

// k is the row index of a [n_k][ld] matrix: `col` points at the lane's column in row 0
__device__ inline void frag_k_rows(const float *col, int64_t ld, int64_t k0, int64_t n_k, int q, float *v)
{
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t k = k0 + 16 * s + 4 * q + j;
            v[4 * s + j] = k < n_k ? col[k * ld] : 0.f;
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
__device__ inline void sum_waves(const f64x4 (*acc)[CB], double *lds, const ST &store)
{
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

// Segment that holds row t (segments are few; a scan is cheaper than a table lookup).
__device__ inline int seg_of_row(const MetaView &mv, int t)
{
    const int n = mv.hdr->n_seg;
    for (int s = 0; s < n; ++s)
        if (t >= mv.seg[s].row0 && t < mv.seg[s].row1) return s;
    return -1;
}

// ---- low-rank products: 16 tokens x 32 ranks per workgroup, eight waves ------------------------------------------------
// mode 0: out[t][j] = sum_c x[t][c] A_k[c][j]              (low-rank activation h, unscaled)
// mode 1: out[t][j] = scale_k sum_c dy[t][c] B_k[j][c]     (gradient case 2)
// grid (slices of 16 rows of the token blocks, 32 ranks each); out is the ragged [len][r] fp32 layout.
constexpr int F32_LR_NW = 8;
__global__ void __launch_bounds__(64 * F32_LR_NW) k_f32_lowrank(MetaView mv, int mode, const float *__restrict__ S, int64_t C,
                                                               float *__restrict__ out)
{
    __shared__ double lds[F32_LR_NW * 16 * 32];
    const int blk = blockIdx.x / (kSkinnyRows / 16);
    const SegInfo g = mv.seg[mv.blk_seg[blk]];
    const int t0 = (blk - g.blk0) * kSkinnyRows + (blockIdx.x % (kSkinnyRows / 16)) * 16;
    const int len = g.row1 - g.row0, r = g.r, j0 = blockIdx.y * 32;
    if (t0 >= len || j0 >= r) return;
    const AdapterInfo a = mv.ad[g.adapter];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i16 = lane & 15, q = lane >> 4;
    const int t = t0 + i16 < len ? t0 + i16 : len - 1;              // clamped rows and columns are not stored
    const float *row = S + (int64_t)(g.row0 + t) * C;
    const float *M = static_cast<const float *>(mode == 0 ? a.A : a.B);
    int j[2];
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) j[cb] = j0 + cb * 16 + i16 < r ? j0 + cb * 16 + i16 : r - 1;
    f64x4 acc[1][2];
    clear<1, 2>(acc);
    auto load_a = [&](int64_t k0, float (*v)[8]) { frag_k_contiguous(row, k0, C, q, v[0]); };
    auto load_b = [&](int64_t k0, float (*v)[8]) {
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
            if (mode == 0) frag_k_rows(M + j[cb], r, k0, C, q, v[cb]);
            else frag_k_contiguous(M + (int64_t)j[cb] * C, k0, C, q, v[cb]);
        }
    };
    contract<1, 2>(wave, F32_LR_NW, C, load_a, load_b, acc);
    const double mult = mode == 0 ? 1.0 : (double)a.scale;
    sum_waves<1, 2, F32_LR_NW>(acc, lds, [&](int rr, int cc, double v) {
        if (t0 + rr < len && j0 + cc < r) out[g.h_off + (int64_t)(t0 + rr) * r + j0 + cc] = (float)(v * mult);
    });
}

hipError_t launch_f32_lowrank(const MetaView &mv, const MetaHeader &h, int mode, const float *S, int64_t C,
                              float *out, hipStream_t st)
{
    if (h.n_blocks == 0) return hipSuccess;
    const dim3 grid((unsigned)h.n_blocks * (kSkinnyRows / 16), (unsigned)((h.max_r16 + 31) / 32));
    hipLaunchKernelGGL(k_f32_lowrank, grid, dim3(64 * F32_LR_NW), 0, st, mv, mode, S, C, out);
    return hipGetLastError();
}

// ---- base products with the low-rank term, and the weight gradients: 32 x 32 outputs per workgroup, four waves ------------
constexpr int F32_NW = 4;

// forward : C[t][n] = sum_i x[t][i]  W[i][n] + scale_k sum_j h[t][j] B_k[j][n]
// backward: C[t][i] = sum_n dy[t][n] W[i][n] +         sum_j g[t][j] A_k[i][j]     (g carries scale_k)
// WK: the contraction index is W's row index (forward with W [d_in][d_out], backward with W [d_out][d_in]).  The low-rank
// terms of the segments in a tile are further chunks of its contraction, added to the rows of that segment alone.
template <bool FWD, bool WK>
__device__ inline void f32_gemm_tile(const MetaView &mv, int n_seg, int64_t T, int64_t Kd, int64_t N, const float *__restrict__ S,
                                     const float *__restrict__ W, const float *__restrict__ side, float *Cout, int accumulate,
                                     int64_t m0, int64_t n0, double *lds)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i16 = lane & 15, q = lane >> 4;
    int64_t m[2], n[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        m[b] = m0 + b * 16 + i16 < T ? m0 + b * 16 + i16 : T - 1;     // clamped rows and columns are not stored
        n[b] = n0 + b * 16 + i16 < N ? n0 + b * 16 + i16 : N - 1;
    }
    f64x4 acc[2][2];
    clear<2, 2>(acc);
    auto load_a = [&](int64_t k0, float (*v)[8]) {
#pragma unroll
        for (int b = 0; b < 2; ++b) frag_k_contiguous(S + m[b] * Kd, k0, Kd, q, v[b]);
    };
    auto load_b = [&](int64_t k0, float (*v)[8]) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            if (WK) frag_k_rows(W + n[b], N, k0, Kd, q, v[b]);
            else frag_k_contiguous(W + n[b] * Kd, k0, Kd, q, v[b]);
        }
    };
    contract<2, 2>(wave, F32_NW, Kd, load_a, load_b, acc);
    const int64_t m1 = m0 + 32 < T ? m0 + 32 : T;
    int turn = (int)((Kd + F32_CK - 1) / F32_CK);                      // chunks handed out so far, to keep the waves level
    for (int s = mv.tile[m0 / kGemmTileRows].first_seg; s < n_seg; ++s) {
        const SegInfo g = mv.seg[s];
        if (g.row0 >= m1) break;
        if (g.adapter < 0 || g.row1 <= g.row0 || g.row1 <= m0) continue;
        const AdapterInfo ad = mv.ad[g.adapter];
        const int r = g.r;
        const float mult = FWD ? ad.scale : 1.f;
        const float *op = static_cast<const float *>(FWD ? ad.B : ad.A);
        for (int k0 = 0; k0 < r; k0 += F32_CK, ++turn) {
            if (turn % F32_NW != wave) continue;
            float a[2][8], b[2][8];
#pragma unroll
            for (int rb = 0; rb < 2; ++rb) {
                const int64_t t = m[rb] - g.row0;
                const bool in = m[rb] >= g.row0 && m[rb] < g.row1;
                frag_k_contiguous(side + g.h_off + (in ? t : 0) * r, k0, r, q, a[rb]);
                if (FWD) frag_k_rows(op + n[rb], N, k0, r, q, b[rb]);
                else frag_k_contiguous(op + n[rb] * r, k0, r, q, b[rb]);
            }
            f64x4 low[2][2];
            clear<2, 2>(low);
            multiply_chunk<2, 2>(a, b, low);
#pragma unroll
            for (int rb = 0; rb < 2; ++rb)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int64_t row = m0 + rb * 16 + q + 4 * i;
                    if (row < g.row0 || row >= g.row1) continue;      // rows of other segments: untouched, also by NaN and infinities
#pragma unroll
                    for (int cb = 0; cb < 2; ++cb) acc[rb][cb][i] += (double)mult * low[rb][cb][i];
                }
        }
    }
    sum_waves<2, 2, F32_NW>(acc, lds, [&](int rr, int cc, double v) {
        if (m0 + rr >= T || n0 + cc >= N) return;
        float *dst = Cout + (m0 + rr) * N + n0 + cc;
        *dst = (float)(accumulate ? v + (double)*dst : v);
    });
}

// want_dA: dA_k[c][j] = sum_t x[t][c]  g[t][j]                (case 3; g carries scale_k)
// else   : dB_k[j][c] = scale_k sum_t h[t][j] dy[t][c]        (case 1)
// summed over every segment of adapter k; 32 hidden columns c0 .. and 32 ranks j0 .. of adapter k.
template <bool WANT_DA>
__device__ inline void f32_wgrad_tile(const MetaView &mv, const float *__restrict__ S, int64_t C, const float *__restrict__ side,
                                      int k, int64_t c0, int j0, double *lds)
{
    const AdapterInfo ad = mv.ad[k];
    const int r = ad.r;
    if (j0 >= r) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i16 = lane & 15, q = lane >> 4;
    int64_t c[2];
    int j[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        c[b] = c0 + b * 16 + i16 < C ? c0 + b * 16 + i16 : C - 1;
        j[b] = j0 + b * 16 + i16 < r ? j0 + b * 16 + i16 : r - 1;
    }
    f64x4 acc[2][2];
    clear<2, 2>(acc);
    int turn = 0;
    for (int li = 0; li < ad.n_own; ++li) {
        const SegInfo g = mv.seg[mv.seg_list[ad.seg_list0 + li]];
        const int len = g.row1 - g.row0;
        const float *s0 = S + (int64_t)g.row0 * C, *z0 = side + g.h_off;
        auto load_s = [&](int64_t k0, float (*v)[8]) {
#pragma unroll
            for (int b = 0; b < 2; ++b) frag_k_rows(s0 + c[b], C, k0, len, q, v[b]);
        };
        auto load_z = [&](int64_t k0, float (*v)[8]) {
#pragma unroll
            for (int b = 0; b < 2; ++b) frag_k_rows(z0 + j[b], r, k0, len, q, v[b]);
        };
        const int first = (wave + F32_NW - turn % F32_NW) % F32_NW;
        if (WANT_DA) contract<2, 2>(first, F32_NW, len, load_s, load_z, acc);     // rows c, columns j
        else contract<2, 2>(first, F32_NW, len, load_z, load_s, acc);             // rows j, columns c
        turn += (len + F32_CK - 1) / F32_CK;
    }
    const double mult = WANT_DA ? 1.0 : (double)ad.scale;
    sum_waves<2, 2, F32_NW>(acc, lds, [&](int rr, int cc, double v) {
        if (WANT_DA) {
            if (c0 + rr < C && j0 + cc < r) ad.dA[(c0 + rr) * r + j0 + cc] = (float)v;
        } else {
            if (j0 + rr < r && c0 + cc < C) ad.dB[(int64_t)(j0 + rr) * C + c0 + cc] = (float)(v * mult);
        }
    });
}

template <bool FWD, bool WK>
__global__ void __launch_bounds__(64 * F32_NW, 2) k_f32_gemm(MetaView mv, int n_seg, int64_t T, int64_t Kd, int64_t N, const float *S,
                                                         const float *W, const float *side, float *Cout, int accumulate,
                                                         int64_t tiles_n, int64_t n_tiles)
{
    __shared__ double lds[F32_NW * 32 * 32];
    for (int64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x)
        f32_gemm_tile<FWD, WK>(mv, n_seg, T, Kd, N, S, W, side, Cout, accumulate, tile / tiles_n * 32, tile % tiles_n * 32, lds);
}

// Both weight gradients in one launch, one output tile per workgroup.  grid (tiles of hidden columns, rank tiles of every
// adapter, 0: dB from dy and h / 1: dA from x and g).
__global__ void __launch_bounds__(64 * F32_NW) k_f32_wgrad(MetaView mv, const float *x, int64_t D, const float *gf, const float *dy,
                                                          int64_t K, const float *hf, int tiles_j)
{
    __shared__ double lds[F32_NW * 32 * 32];
    const int64_t c0 = (int64_t)blockIdx.x * 32;
    const int j0 = (int)(blockIdx.y % tiles_j) * 32, k = (int)(blockIdx.y / tiles_j);
    if (c0 >= (blockIdx.z == 0 ? K : D)) return;
    if (blockIdx.z == 0) f32_wgrad_tile<false>(mv, dy, K, hf, k, c0, j0, lds);
    else f32_wgrad_tile<true>(mv, x, D, gf, k, c0, j0, lds);
}

hipError_t launch_f32_gemm(const MetaView &mv, const MetaHeader &h, bool forward, const float *S, const float *W,
                           const float *side, float *C, bool accumulate, hipStream_t st)
{
    if (h.T == 0) return hipSuccess;
    const int acc = accumulate ? 1 : 0;
    const int64_t Kd = forward ? h.D : h.K, N = forward ? h.K : h.D;
    const int64_t tiles_n = (N + 31) / 32, n_tiles = tiles_n * ((h.T + 31) / 32);
    const dim3 grid((unsigned)(n_tiles < (1 << 22) ? n_tiles : (1 << 22)));      // beyond that a workgroup walks several tiles
    const bool wk = forward != (h.w_out_in != 0);
#define PL_F32G(F_, W_) hipLaunchKernelGGL((k_f32_gemm<F_, W_>), grid, dim3(64 * F32_NW), 0, st, mv, (int)h.n_seg, h.T, Kd, N, S, W, side, C, acc, tiles_n, n_tiles)
    if (forward && wk) PL_F32G(true, true);
    else if (forward) PL_F32G(true, false);
    else if (wk) PL_F32G(false, true);
    else PL_F32G(false, false);
#undef PL_F32G
    return hipGetLastError();
}

hipError_t launch_f32_wgrad(const MetaView &mv, const MetaHeader &h, int max_rank, const float *x, const float *gf, const float *dy,
                            const float *hf, hipStream_t st)
{
    if (h.n_adapters == 0) return hipSuccess;
    const int tiles_j = (max_rank + 31) / 32;
    const int64_t widest = h.K > h.D ? h.K : h.D;
    const dim3 grid((unsigned)((widest + 31) / 32), (unsigned)(tiles_j * h.n_adapters), 2);
    hipLaunchKernelGGL(k_f32_wgrad, grid, dim3(64 * F32_NW), 0, st, mv, x, h.D, gf, dy, h.K, hf, tiles_j);
    return hipGetLastError();
}

// Stand-alone low-rank update: C[t][n] += mult * sum_j side[t][j] * op_k(j, n)   (fp64 accumulation)
//   to_y : side = h (unscaled), op_k = B_k [r][N], mult = scale_k;   else side = g (carries scale_k), op_k = A_k^T, A_k [N][r]
template <bool TO_Y>
__global__ void __launch_bounds__(256) k_f32_expand(MetaView mv, float *C, int64_t N, const float *side)
{
    const int64_t t = (int64_t)blockIdx.x * 2 + threadIdx.x / 128;
    const int64_t n = (int64_t)blockIdx.y * 128 + threadIdx.x % 128;
    if (t >= mv.hdr->T || n >= N) return;
    const int s = seg_of_row(mv, (int)t);
    const SegInfo g = mv.seg[s];
    if (g.adapter < 0) return;
    const AdapterInfo a = mv.ad[g.adapter];
    const float *row = side + g.h_off + (int64_t)(t - g.row0) * g.r;
    double l = 0.0;
    if (TO_Y) {
        const float *Bk = static_cast<const float *>(a.B);
        for (int q = 0; q < g.r; ++q) l += (double)row[q] * (double)Bk[(int64_t)q * N + n];
        l *= (double)a.scale;
    } else {
        const float *Ak = static_cast<const float *>(a.A);
        for (int q = 0; q < g.r; ++q) l += (double)row[q] * (double)Ak[n * g.r + q];
    }
    C[t * N + n] = (float)((double)C[t * N + n] + l);
}

hipError_t launch_f32_expand(const MetaView &mv, const MetaHeader &h, bool to_y, float *C, const float *side, hipStream_t st)
{
    if (h.T == 0 || h.n_blocks == 0) return hipSuccess;
    const int64_t N = to_y ? h.K : h.D;
    dim3 grid((unsigned)((h.T + 1) / 2), (unsigned)((N + 127) / 128));     // N <= 2^22: at most 32768 in y
    if (to_y) hipLaunchKernelGGL(k_f32_expand<true>, grid, dim3(256), 0, st, mv, C, N, side);
    else hipLaunchKernelGGL(k_f32_expand<false>, grid, dim3(256), 0, st, mv, C, N, side);
    return hipGetLastError();
}

}  // namespace plora
