// fp32 I/O path of the packed multi-LoRA layer.  Inputs and outputs are fp32; every sum is accumulated in fp64 and rounded
// once, so the result is within an ulp or two of the exact value for any problem size.
//
// Every product runs on the fp64 matrix instruction (16x16x4, 64 cycles): its rate is that of the vector ALU's fp64 FMA, but one
// instruction replaces sixteen per lane and an operand element is converted once per 16 outputs.  The problems of this path
// are small (the fp32 configuration: 256 tokens, 256 x 256, 72 MFLOP), so latency bounds it and the shape of
// the kernels follows from that: small output tiles for many workgroups, the contraction of a tile dealt to its waves in
// pairs of chunks of 16, operands straight from memory into registers (no staging, no barrier until the waves' sums meet in LDS), the
// next two chunks (16 x 16 outputs: five) in flight while one is multiplied.  Four waves per SIMD: an operand of 16 elements a chunk and
// nothing kept across tiles leaves room for that (one form, the forward with W [d_out][d_in] in 32 x 32 tiles, spills two registers, outside its
// main loop), and then the tiles of a batch are on the chip all at once (two waves, chunks of 32: 600 tiles took two rounds of 512).
// Measured (256-token configuration, then 777 tokens, 500 -> 750, in us; a launch that does nothing takes 2.5 - 3): base product 49 and 145 with 64 x 64 tiles on the vector ALU, 11 and 29 at two waves per SIMD, now 6 and 23
// (the matrix instructions alone: 8.3 on average over the SIMDs, 12 where three tiles meet; a wave lives 15, of which it waits 58 % to issue,
// mostly for the matrix instructions of the others on its SIMD, and 26 % for loads and the LDS); weight gradients with the gradient
// of x 11 and 29.5, now 7 and 24.5; low-rank products beside the preparation 5.7 and 8.2.  The whole step: 322 -> 33 -> 22.8 and 1948 -> 73 -> 60.
// Larger ones, 4 adapters of rank 16: 1024 tokens, 1024 -> 1024 138 -> 103; 4096 tokens, 4096 -> 4096 5500 -> 4380 (63 TFLOP/s of
// the nominal 78.6).
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

constexpr int64_t kF32SmallTiles = 1024;    // see f32_tile_side
constexpr int64_t kF32MaxTiles = 1 << 22;   // workgroups of a launch

// ---- base products with the low-rank term, and the weight gradients: four waves per workgroup ------------------------------
// forward : C[t][n] = sum_i x[t][i]  W[i][n] + scale_k sum_j h[t][j] B_k[j][n]
// backward: C[t][i] = sum_n dy[t][n] W[i][n] +         sum_j g[t][j] A_k[i][j]     (g carries scale_k)
// WK: the contraction index is W's row index (forward with W [d_in][d_out], backward with W [d_out][d_in]).  16 NB x 16 NB
// outputs per workgroup.  The low-rank terms of the segments in a tile are further chunks of its contraction, added to
// the rows of that segment alone.
template <bool FWD, bool WK, int NB>
__device__ inline void f32_gemm_tile(const MetaView &mv, int n_seg, int64_t T, int64_t Kd, int64_t N, const float *__restrict__ S,
                                     const float *__restrict__ W, const float *__restrict__ side, float *Cout, int accumulate,
                                     int64_t m0, int n0, double *lds)
{
    constexpr int TS = 16 * NB, DEPTH = NB == 1 ? 6 : 3;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), q = lane >> 4;
    const int64_t m1 = m0 + TS < T ? m0 + TS : T;
    const int rows_here = (int)(m1 - m0), cols_here = (int)N - n0 < TS ? (int)N - n0 : TS;
    F32Operand<false, NB> rows{S + m0 * Kd, Kd, {}};
    F32Operand<WK, NB> cols{WK ? W + n0 : W + n0 * Kd, WK ? N : Kd, {}};
    auto clamped = [](int i, int n) { return i < n ? i : n - 1; };   // rows and columns past the end are not stored
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        rows.row(b, clamped(b * 16 + rows.own_row(), rows_here));
        cols.row(b, clamped(b * 16 + cols.own_row(), cols_here));
    }
    // the segments from the row tile's first one on, one per lane, with what the low-rank terms need of them: requested ahead of
    // the contraction (one after the other behind it, segment and adapter, they were 3 us for each segment of a tile)
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
    f64x4 acc[NB][NB];
    clear<NB, NB>(acc);
    contract<NB, NB, DEPTH>(wave, F32_NW, Kd, rows, cols, acc);
    int turn = (int)((Kd + 2 * F32_CK - 1) / (2 * F32_CK));            // pairs, then chunks, handed out so far, to keep the waves level
    for (int win = first_seg; win < n_seg; win += 64) {
        if (win > first_seg) load_window(win + lane);
        const bool last = __ballot(s_past) != 0;
        for (uint64_t todo = __ballot(s_in); todo; todo &= todo - 1) {
            const int l = __builtin_ctzll(todo);
            const int row0 = __builtin_amdgcn_readlane(s_row0, l), row1 = __builtin_amdgcn_readlane(s_row1, l), r = __builtin_amdgcn_readlane(s_r, l);
            const float mult = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(s_mult), l));
            const float *op = reinterpret_cast<const float *>((uintptr_t)readlane64(s_op, l));
            const int64_t h_off = readlane64(s_h, l);
            const int lo = row0 > m0 ? (int)(row0 - m0) : 0, hi = row1 < m1 ? (int)(row1 - m0) : rows_here;    // the segment's rows of the tile
            F32Operand<FWD, NB> low_cols{FWD ? op + n0 : op + n0 * r, FWD ? N : r, {}};
#pragma unroll
            for (int b = 0; b < NB; ++b) low_cols.row(b, clamped(b * 16 + low_cols.own_row(), cols_here));
            F32Operand<false, NB> low_rows{side + h_off + (m0 + lo - row0) * r, r, {}};
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const int i = b * 16 + low_rows.own_row();
                low_rows.row(b, i >= lo && i < hi ? i - lo : 0);
            }
            for (int k0 = 0; k0 < r; k0 += F32_CK, ++turn) {
                if (turn % F32_NW != wave) continue;
                float a[NB][4], b[NB][4];
                low_rows.load_part(k0, r, a);
                low_cols.load_part(k0, r, b);
                low_rows.arrange(a);
                low_cols.arrange(b);
                f64x4 low[NB][NB];
                clear<NB, NB>(low);
                multiply_chunk<NB, NB>(a, b, low);
                settle<NB, NB>(low);
                settle<NB, NB>(acc);
#pragma unroll
                for (int rb = 0; rb < NB; ++rb)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int row = rb * 16 + q + 4 * i;
                        if (row < lo || row >= hi) continue;                  // rows of other segments: untouched, also by NaN and infinities
#pragma unroll
                        for (int cb = 0; cb < NB; ++cb) acc[rb][cb][i] += (double)mult * low[rb][cb][i];
                    }
            }
        }
        if (last) break;
    }
    sum_waves<NB, NB, F32_NW>(acc, lds, [&](int rr, int cc, double v) {
        if (rr >= rows_here || cc >= cols_here) return;
        float *dst = Cout + m0 * N + n0 + ((int64_t)rr * N + cc);
        *dst = (float)(accumulate ? v + (double)*dst : v);
    });
}

// want_dA: dA_k[c][j] = sum_t x[t][c]  g[t][j]                (case 3; g carries scale_k)
// else   : dB_k[j][c] = scale_k sum_t h[t][j] dy[t][c]        (case 1)
// summed over every segment of adapter k; 32 hidden columns c0 .. and 16 ranks j0 .. of adapter k.
template <bool WANT_DA>
__device__ inline void f32_wgrad_tile(const MetaView &mv, const float *__restrict__ S, int64_t C, const float *__restrict__ side,
                                      int k, int64_t c0, int j0, double *lds)
{
    const AdapterInfo ad = mv.ad[k];
    const int r = ad.r;
    if (j0 >= r) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), i16 = lane & 15;
    constexpr int RB = WANT_DA ? 2 : 1, CB = WANT_DA ? 1 : 2;
    f64x4 acc[RB][CB];
    clear<RB, CB>(acc);
    int turn = 0;
    for (int li = 0; li < ad.n_own; ++li) {
        const SegInfo g = mv.seg[mv.seg_list[ad.seg_list0 + li]];
        const int len = g.row1 - g.row0;
        F32Operand<true, 2> s{S + (int64_t)g.row0 * C + c0, C, {}};
        F32Operand<true, 1> z{side + g.h_off + j0, r, {}};
#pragma unroll
        for (int b = 0; b < 2; ++b) s.row(b, b * 16 + i16 < C - c0 ? b * 16 + i16 : (int)(C - 1 - c0));
        z.row(0, j0 + i16 < r ? i16 : r - 1 - j0);
        const int first = (wave + F32_NW - turn % F32_NW) % F32_NW;
        if constexpr (WANT_DA) contract<RB, CB, 4>(first, F32_NW, len, s, z, acc);     // rows c, columns j
        else contract<RB, CB, 4>(first, F32_NW, len, z, s, acc);                       // rows j, columns c
        turn += (len + 2 * F32_CK - 1) / (2 * F32_CK);
    }
    const double mult = WANT_DA ? 1.0 : (double)ad.scale;
    sum_waves<RB, CB, F32_NW>(acc, lds, [&](int rr, int cc, double v) {
        if (WANT_DA) {
            if (c0 + rr < C && j0 + cc < r) ad.dA[(c0 + rr) * r + j0 + cc] = (float)v;
        } else {
            if (j0 + rr < r && c0 + cc < C) ad.dB[(int64_t)(j0 + rr) * C + c0 + cc] = (float)(v * mult);
        }
    });
}

template <bool FWD, bool WK, int NB>
__global__ void __launch_bounds__(64 * F32_NW, 4) k_f32_gemm(MetaView mv, int n_seg, int64_t T, int64_t Kd, int64_t N, const float *S,
                                                         const float *W, const float *side, float *Cout, int accumulate,
                                                         uint32_t tiles_n, uint32_t tile0)
{
    __shared__ double lds[F32_NW * 256 * NB * NB];
    const uint32_t tile = tile0 + blockIdx.x;                             // one per workgroup: what a loop would keep across tiles spills
    f32_gemm_tile<FWD, WK, NB>(mv, n_seg, T, Kd, N, S, W, side, Cout, accumulate, (int64_t)(tile / tiles_n) * (16 * NB), (int)(tile % tiles_n) * (16 * NB), lds);
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
    const int c = (int)(unit % across), jk = (int)(unit / across), j0 = jk % w.tiles_j * 16, k = jk / w.tiles_j;
    if (c < w.tiles_b) f32_wgrad_tile<false>(mv, w.dy, w.K, w.hf, k, (int64_t)c * 32, j0, lds);
    else f32_wgrad_tile<true>(mv, w.x, w.D, w.gf, k, (int64_t)(c - w.tiles_b) * 32, j0, lds);
}
__global__ void __launch_bounds__(64 * F32_NW, 4) k_f32_wgrad(MetaView mv, F32Wgrad w)
{
    __shared__ double lds[F32_NW * 32 * 16];
    f32_wgrad_unit(mv, w, (int64_t)blockIdx.y * gridDim.x + blockIdx.x, lds);
}

// The weight gradients and the gradient of x in one launch (they need g and nothing of each other): the units of the gradients
// first, each walks all tokens of an adapter.
template <bool WK, int NB>
__global__ void __launch_bounds__(64 * F32_NW, 4) k_f32_bwd(MetaView mv, F32Wgrad w, uint32_t n_units, int n_seg, int64_t T, const float *W,
                                                        float *dx, uint32_t tiles_n)
{
    __shared__ double lds[F32_NW * 256 * (NB == 1 ? 2 : NB * NB)];
    if (blockIdx.x < n_units) { f32_wgrad_unit(mv, w, blockIdx.x, lds); return; }
    const uint32_t tile = blockIdx.x - n_units;
    f32_gemm_tile<false, WK, NB>(mv, n_seg, T, w.K, w.D, w.dy, W, w.gf, dx, 0, (int64_t)(tile / tiles_n) * (16 * NB), (int)(tile % tiles_n) * (16 * NB), lds);
}

// Tiles of 16 x 16 outputs while all of them are on the chip at once (four workgroups on each of 256 compute units): then nothing but
// the length of a wave's chain counts.  30 shapes, against 32 x 32 alone: 1.20 times as fast on average, up to 1.4 (25 tokens, 385 -> 550
// 35 -> 25 us); up to 2048 instead of 1024 small tiles gains 2 % or loses 4 %.
static int f32_tile_side(int64_t T, int64_t N) { return ((T + 15) / 16) * ((N + 15) / 16) <= kF32SmallTiles ? 16 : 32; }

hipError_t launch_f32_gemm(const MetaView &mv, const MetaHeader &h, bool forward, const float *S, const float *W,
                           const float *side, float *C, bool accumulate, hipStream_t st)
{
    if (h.T == 0) return hipSuccess;
    const int acc = accumulate ? 1 : 0;
    const int64_t Kd = forward ? h.D : h.K, N = forward ? h.K : h.D;
    const int side_len = f32_tile_side(h.T, N);
    const int64_t tiles_n = (N + side_len - 1) / side_len, n_tiles = tiles_n * ((h.T + side_len - 1) / side_len);
    const bool wk = forward != (h.w_out_in != 0);
#define PL_F32G1(F_, W_, NB_) hipLaunchKernelGGL((k_f32_gemm<F_, W_, NB_>), dim3(n), dim3(64 * F32_NW), 0, st, mv, (int)h.n_seg, h.T, Kd, N, S, W, side, C, acc, (uint32_t)tiles_n, (uint32_t)tile0)
#define PL_F32G(F_, W_) do { if (side_len == 16) PL_F32G1(F_, W_, 1); else PL_F32G1(F_, W_, 2); } while (0)
    for (int64_t tile0 = 0; tile0 < n_tiles; tile0 += kF32MaxTiles) {      // (2^32 of 32 x 32 are 17 TB of outputs)
        const unsigned n = (unsigned)(n_tiles - tile0 < kF32MaxTiles ? n_tiles - tile0 : kF32MaxTiles);
        if (forward && wk) PL_F32G(true, true);
        else if (forward) PL_F32G(true, false);
        else if (wk) PL_F32G(false, true);
        else PL_F32G(false, false);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
#undef PL_F32G
#undef PL_F32G1
    return hipSuccess;
}

static F32Wgrad wgrad_of(const MetaHeader &h, int max_rank, const float *x, const float *gf, const float *dy, const float *hf)
{
    return F32Wgrad{x, gf, dy, hf, h.D, h.K, (max_rank + 15) / 16, (int32_t)((h.K + 31) / 32), (int32_t)((h.D + 31) / 32), 0};
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
    return (int64_t)(w.tiles_b + w.tiles_a) * w.tiles_j * h.n_adapters <= kF32MaxTiles && (h.D + 31) / 32 * ((h.T + 31) / 32) <= kF32MaxTiles;
}

hipError_t launch_f32_bwd(const MetaView &mv, const MetaHeader &h, int max_rank, const float *x, const float *gf, const float *dy,
                          const float *hf, const float *W, float *dx, hipStream_t st)
{
    const F32Wgrad w = wgrad_of(h, max_rank, x, gf, dy, hf);
    const int64_t units = (int64_t)(w.tiles_b + w.tiles_a) * w.tiles_j * h.n_adapters;
    const int side_len = f32_tile_side(h.T, h.D);
    const int64_t tiles_n = (h.D + side_len - 1) / side_len, n_tiles = tiles_n * ((h.T + side_len - 1) / side_len);
    const dim3 grid((unsigned)(units + n_tiles));
#define PL_F32B(W_, NB_) hipLaunchKernelGGL((k_f32_bwd<W_, NB_>), grid, dim3(64 * F32_NW), 0, st, mv, w, (uint32_t)units, (int)h.n_seg, h.T, W, dx, (uint32_t)tiles_n)
    if (h.w_out_in && side_len == 16) PL_F32B(true, 1);
    else if (h.w_out_in) PL_F32B(true, 2);
    else if (side_len == 16) PL_F32B(false, 1);
    else PL_F32B(false, 2);
#undef PL_F32B
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
