// fp32 I/O path of the packed multi-LoRA layer.  Inputs and outputs are fp32; every sum is accumulated in fp64 and rounded
// once, so the result is within an ulp or two of the exact value for any problem size.
//
// Every product runs on the fp64 matrix instruction (16x16x4): its rate is that of the vector ALU's fp64 FMA, but one
// instruction replaces sixteen per lane and an operand element is converted once per 16 outputs.  The problems of this path
// are small (the fp32 configuration: 256 tokens, 256 x 256, 72 MFLOP), so latency bounds it and the shape of
// the kernels follows from that: small output tiles for many workgroups, the contraction of a tile dealt to its waves in
// chunks of 32, operands straight from memory into registers (no staging, no barrier until the waves' sums meet in LDS), the
// next chunk in flight while one is multiplied.  Measured (256-token configuration, then 777 tokens, 500 -> 750, in us):
// low-rank products 69 and 498 with one dot product per thread, 5.6 and 8.2 in launches of their own, now beside the preparation
// (together 5.6 and 8.4); base products 49 and 145 with 64 x 64 tiles on the vector ALU, now 11 and 29; the two weight gradients 63
// and 216 with one dot product per thread in two launches, 5.4 and 9.0 in one, now in the launch of the gradient of x (together 11
// and 29.5, before 15.3 and 36.6).  The whole step: 322 -> 45 -> 33 and 1948 -> 94 -> 73.  Larger ones, 4 adapters of rank 16: 1024 tokens,
// 1024 -> 1024 2.46 ms -> 0.157 -> 0.138; 4096 tokens, 1024 -> 1024 0.478 -> 0.446; 4096 tokens, 4096 -> 4096 18.3 -> 5.8 ms (base products
// 4.5 -> 2.6 - 3.0 each, 46 - 53 TFLOP/s of the nominal 78.6).  Three waves per SIMD instead of two spill: 4096 tokens 0.403,
// 512 tokens, 300 -> 900 54 -> 59 us.
#include "f32_tiles.h"

namespace plora {

// Segment that holds row t (segments are few; a scan is cheaper than a table lookup).
__device__ inline int seg_of_row(const MetaView &mv, int t)
{
    const int n = mv.hdr->n_seg;
    for (int s = 0; s < n; ++s)
        if (t >= mv.seg[s].row0 && t < mv.seg[s].row1) return s;
    return -1;
}

// ---- low-rank products (f32_tiles.h) with the tables in place: grouped calls, long descriptions ------------------------
__global__ void __launch_bounds__(64 * F32_NW, 2) k_f32_lowrank(MetaView mv, F32LowRank job)
{
    __shared__ double lds[F32_NW * 16 * 16];
    const int blk = blockIdx.x / (kSkinnyRows / 16);
    const SegInfo g = mv.seg[mv.blk_seg[blk]];
    const AdapterInfo a = mv.ad[g.adapter];
    f32_lowrank_tile(job, g, a.scale, static_cast<const float *>(job.mode == 0 ? a.A : a.B),
                     (blk - g.blk0) * kSkinnyRows + (blockIdx.x % (kSkinnyRows / 16)) * 16, blockIdx.y * 16, lds);
}

hipError_t launch_f32_lowrank(const MetaView &mv, const MetaHeader &h, int mode, const float *S, int64_t C,
                              float *out, hipStream_t st)
{
    if (h.n_blocks == 0) return hipSuccess;
    const dim3 grid((unsigned)h.n_blocks * (kSkinnyRows / 16), (unsigned)(h.max_r16 / 16));
    hipLaunchKernelGGL(k_f32_lowrank, grid, dim3(64 * F32_NW), 0, st, mv, F32LowRank{S, out, C, mode});
    return hipGetLastError();
}

// ---- base products with the low-rank term, and the weight gradients: 32 x 32 outputs per workgroup, four waves ------------
// forward : C[t][n] = sum_i x[t][i]  W[i][n] + scale_k sum_j h[t][j] B_k[j][n]
// backward: C[t][i] = sum_n dy[t][n] W[i][n] +         sum_j g[t][j] A_k[i][j]     (g carries scale_k)
// WK: the contraction index is W's row index (forward with W [d_in][d_out], backward with W [d_out][d_in]).  The low-rank
// terms of the segments in a tile are further chunks of its contraction, added to the rows of that segment alone.
template <bool FWD, bool WK>
__device__ inline void f32_gemm_tile(const MetaView &mv, int n_seg, int64_t T, int64_t Kd, int64_t N, const float *__restrict__ S,
                                     const float *__restrict__ W, const float *__restrict__ side, float *Cout, int accumulate,
                                     int64_t m0, int64_t n0, double *lds)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), i16 = lane & 15, q = lane >> 4;
    int m[2], n[2];                                                   // of the tile; clamped rows and columns are not stored
    uint32_t off_s[2], off_w[2];                                      // 31 rows of at most 2^22 elements
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        m[b] = m0 + b * 16 + i16 < T ? b * 16 + i16 : (int)(T - 1 - m0);
        n[b] = n0 + b * 16 + i16 < N ? b * 16 + i16 : (int)(N - 1 - n0);
        off_s[b] = ((uint32_t)m[b] * (uint32_t)Kd + 4 * q) * 4u;
        off_w[b] = WK ? (4u * q * (uint32_t)N + (uint32_t)n[b]) * 4u : ((uint32_t)n[b] * (uint32_t)Kd + 4 * q) * 4u;
    }
    // the segments from the row tile's first one on, one per lane, with what the low-rank terms need of them: requested ahead of
    // the contraction (one after the other behind it, segment and adapter, they were 3 us for each segment of a tile)
    const int64_t m1 = m0 + 32 < T ? m0 + 32 : T;
    const int first_seg = mv.tile[m0 / kGemmTileRows].first_seg;
    int s_row0 = 0, s_row1 = 0, s_r = 0;
    int64_t s_h = 0, s_op = 0;
    float s_mult = 0.f;
    bool s_in = false, s_past = true;
    auto load_window = [&](int s) {
        s_in = false; s_past = true;
        if (s < n_seg) {
            const SegInfo g = mv.seg[s];
            s_row0 = g.row0; s_row1 = g.row1; s_r = g.r; s_h = g.h_off;
            s_past = g.row0 >= m1;
            s_in = !s_past && g.adapter >= 0 && g.row1 > g.row0 && g.row1 > m0;
            if (s_in) {
                const AdapterInfo *ad = mv.ad + g.adapter;
                s_op = (int64_t)(uintptr_t)(FWD ? ad->B : ad->A);
                s_mult = FWD ? ad->scale : 1.f;
            }
        }
    };
    load_window(first_seg + lane);
    f64x4 acc[2][2];
    clear<2, 2>(acc);
    auto load_a = [&](int64_t k0, float (*v)[8]) {
#pragma unroll
        for (int b = 0; b < 2; ++b) frag_k_contiguous(S + m0 * Kd, off_s[b], k0, Kd, q, v[b]);
    };
    auto load_b = [&](int64_t k0, float (*v)[8]) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            if (WK) frag_k_rows(W + n0, off_w[b], N, k0, Kd, q, v[b]);
            else frag_k_contiguous(W + n0 * Kd, off_w[b], k0, Kd, q, v[b]);
        }
    };
    contract<2, 2>(wave, F32_NW, Kd, load_a, load_b, acc);
    int turn = (int)((Kd + F32_CK - 1) / F32_CK);                      // chunks handed out so far, to keep the waves level
    for (int win = first_seg; win < n_seg; win += 64) {
        if (win > first_seg) load_window(win + lane);
        const bool last = __ballot(s_past) != 0;
        for (uint64_t todo = __ballot(s_in); todo; todo &= todo - 1) {
            const int l = __builtin_ctzll(todo);
            const int row0 = __builtin_amdgcn_readlane(s_row0, l), row1 = __builtin_amdgcn_readlane(s_row1, l), r = __builtin_amdgcn_readlane(s_r, l);
            const float mult = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(s_mult), l));
            const float *op = reinterpret_cast<const float *>((uintptr_t)readlane64(s_op, l));
            const int64_t h_off = readlane64(s_h, l);
            for (int k0 = 0; k0 < r; k0 += F32_CK, ++turn) {
                if (turn % F32_NW != wave) continue;
                float a[2][8], b[2][8];
#pragma unroll
                for (int rb = 0; rb < 2; ++rb) {
                    const int row = (int)m0 + m[rb], t = row >= row0 && row < row1 ? row - row0 : 0;
                    frag_k_contiguous(side + h_off + (int64_t)t * r, 16u * q, k0, r, q, a[rb]);
                    if (FWD) frag_k_rows(op + n0, (4u * q * (uint32_t)N + (uint32_t)n[rb]) * 4u, N, k0, r, q, b[rb]);
                    else frag_k_contiguous(op + n0 * r, ((uint32_t)(n[rb] * r) + 4 * q) * 4u, k0, r, q, b[rb]);
                }
                f64x4 low[2][2];
                clear<2, 2>(low);
                multiply_chunk<2, 2>(a, b, low);
                settle<2, 2>(low);
                settle<2, 2>(acc);
#pragma unroll
                for (int rb = 0; rb < 2; ++rb)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int64_t row = m0 + rb * 16 + q + 4 * i;
                        if (row < row0 || row >= row1) continue;          // rows of other segments: untouched, also by NaN and infinities
#pragma unroll
                        for (int cb = 0; cb < 2; ++cb) acc[rb][cb][i] += (double)mult * low[rb][cb][i];
                    }
            }
        }
        if (last) break;
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
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), i16 = lane & 15, q = lane >> 4;
    uint32_t off_s[2], off_z[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const uint32_t c = (uint32_t)(c0 + b * 16 + i16 < C ? b * 16 + i16 : C - 1 - c0);
        const uint32_t j = (uint32_t)(j0 + b * 16 + i16 < r ? j0 + b * 16 + i16 : r - 1);
        off_s[b] = (4u * q * (uint32_t)C + c) * 4u;
        off_z[b] = (4u * q * (uint32_t)r + j) * 4u;
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
            for (int b = 0; b < 2; ++b) frag_k_rows(s0 + c0, off_s[b], C, k0, len, q, v[b]);
        };
        auto load_z = [&](int64_t k0, float (*v)[8]) {
#pragma unroll
            for (int b = 0; b < 2; ++b) frag_k_rows(z0, off_z[b], r, k0, len, q, v[b]);
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

// Both weight gradients in one launch, one output tile per workgroup: tiles of hidden columns (of dB, then of dA) fastest, then
// rank tiles, then adapters.
struct F32Wgrad {
    const float *x, *gf, *dy, *hf;
    int64_t D, K;
    int32_t tiles_j, tiles_b, tiles_a, reserved;
};
__device__ inline void f32_wgrad_unit(const MetaView &mv, const F32Wgrad &w, int64_t unit, double *lds)
{
    const int64_t across = w.tiles_b + w.tiles_a;
    const int c = (int)(unit % across), jk = (int)(unit / across), j0 = jk % w.tiles_j * 32, k = jk / w.tiles_j;
    if (c < w.tiles_b) f32_wgrad_tile<false>(mv, w.dy, w.K, w.hf, k, (int64_t)c * 32, j0, lds);
    else f32_wgrad_tile<true>(mv, w.x, w.D, w.gf, k, (int64_t)(c - w.tiles_b) * 32, j0, lds);
}
__global__ void __launch_bounds__(64 * F32_NW, 2) k_f32_wgrad(MetaView mv, F32Wgrad w)
{
    __shared__ double lds[F32_NW * 32 * 32];
    f32_wgrad_unit(mv, w, (int64_t)blockIdx.y * gridDim.x + blockIdx.x, lds);
}

// The weight gradients and the gradient of x in one launch (they need g and nothing of each other): the units of the gradients
// first, each walks all tokens of an adapter.
template <bool WK>
__global__ void __launch_bounds__(64 * F32_NW, 2) k_f32_bwd(MetaView mv, F32Wgrad w, int64_t n_units, int n_seg, int64_t T, const float *W,
                                                        float *dx, int64_t tiles_n, int64_t n_tiles)
{
    __shared__ double lds[F32_NW * 32 * 32];
    if ((int64_t)blockIdx.x < n_units) { f32_wgrad_unit(mv, w, blockIdx.x, lds); return; }
    for (int64_t tile = blockIdx.x - n_units; tile < n_tiles; tile += gridDim.x - n_units)
        f32_gemm_tile<false, WK>(mv, n_seg, T, w.K, w.D, w.dy, W, w.gf, dx, 0, tile / tiles_n * 32, tile % tiles_n * 32, lds);
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

static F32Wgrad wgrad_of(const MetaHeader &h, int max_rank, const float *x, const float *gf, const float *dy, const float *hf)
{
    return F32Wgrad{x, gf, dy, hf, h.D, h.K, (max_rank + 31) / 32, (int32_t)((h.K + 31) / 32), (int32_t)((h.D + 31) / 32), 0};
}

hipError_t launch_f32_wgrad(const MetaView &mv, const MetaHeader &h, int max_rank, const float *x, const float *gf, const float *dy,
                            const float *hf, hipStream_t st)
{
    if (h.n_adapters == 0) return hipSuccess;
    const F32Wgrad w = wgrad_of(h, max_rank, x, gf, dy, hf);
    hipLaunchKernelGGL(k_f32_wgrad, dim3((unsigned)(w.tiles_b + w.tiles_a), (unsigned)(w.tiles_j * h.n_adapters)), dim3(64 * F32_NW), 0, st, mv, w);
    return hipGetLastError();
}

bool f32_bwd_fits(const MetaHeader &h, int max_rank)
{
    const F32Wgrad w = wgrad_of(h, max_rank, nullptr, nullptr, nullptr, nullptr);
    return (int64_t)(w.tiles_b + w.tiles_a) * w.tiles_j * h.n_adapters <= (1 << 22);
}

hipError_t launch_f32_bwd(const MetaView &mv, const MetaHeader &h, int max_rank, const float *x, const float *gf, const float *dy,
                          const float *hf, const float *W, float *dx, hipStream_t st)
{
    const F32Wgrad w = wgrad_of(h, max_rank, x, gf, dy, hf);
    const int64_t units = (int64_t)(w.tiles_b + w.tiles_a) * w.tiles_j * h.n_adapters;
    const int64_t tiles_n = (h.D + 31) / 32, n_tiles = tiles_n * ((h.T + 31) / 32);
    const dim3 grid((unsigned)(units + (n_tiles < (1 << 22) ? n_tiles : (1 << 22))));
    if (h.w_out_in) hipLaunchKernelGGL(k_f32_bwd<true>, grid, dim3(64 * F32_NW), 0, st, mv, w, units, (int)h.n_seg, h.T, W, dx, tiles_n, n_tiles);
    else hipLaunchKernelGGL(k_f32_bwd<false>, grid, dim3(64 * F32_NW), 0, st, mv, w, units, (int)h.n_seg, h.T, W, dx, tiles_n, n_tiles);
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
