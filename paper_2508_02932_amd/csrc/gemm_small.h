// The tile routine of gemm_small_bf16.hip (see there for what it is for), also run beside the preparation of a short batch
// (gemm_short_bf16.hip).
#pragma once
#include "plora_internal.h"

namespace plora {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

#define LDS_PTR(T, p) ((__attribute__((address_space(3))) T *)(p))

constexpr int GS_BN = 128;                 // output columns per workgroup
constexpr int GS_BK = 64;                  // contraction elements per stage
// Ring slots of the two tiles; two workgroups share the 160 KB of a compute unit.  deep: a third slot of the W tile (80 KB).
constexpr int gs_ring_x(int bm) { return bm == 128 ? 2 : 3; }
inline bool gemm_small_deep(int64_t T) { return T <= 512; }      // measured in gemm_small_bf16.hip
constexpr int gs_ring_w(int bm, bool deep) { return bm == 128 && !deep ? 2 : 3; }

__device__ inline uint32_t gs_pack_bf16x2(float lo, float hi)
{
    typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
    typedef float v2f __attribute__((ext_vector_type(2)));
    const v2f f = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, v2bf));
}

// 2 bf16 + 2 bf16 in fp32, rounded to nearest even (the accumulating epilogue)
__device__ inline uint32_t gs_add_bf16x2(uint32_t a, uint32_t b)
{
    return gs_pack_bf16x2(__uint_as_float(a << 16) + __uint_as_float(b << 16),
                          __uint_as_float(a & 0xffff0000u) + __uint_as_float(b & 0xffff0000u));
}

template <int N> __device__ inline void gs_wait_vmcnt()
{
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit field");
    __builtin_amdgcn_s_waitcnt(0x0f70 | (N & 15) | ((N >> 4) << 14));
}

__device__ inline int64_t gs_readlane64(int64_t v, int l)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), l);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// FWD names the form of the weight operand as in gemm_bf16.hip: W[Kd][N] (contraction index = row index), else W[N][Kd].
// One workgroup per (row tile of BM, column tile of 128, split z of the contraction); BM / 32 waves, each 64 (32 when
// BM = 64) x 64 outputs on MFMA 16x16x32.  Stages of 64 contraction elements go HBM -> LDS directly, through one ring for the token tile and one for W.
// Split z multiplies its share of the main steps and every n_split-th extension step; without EXT main steps alone, always to part.
// row_tile0 > 0: the rows are those of the 256-row tiles from entry row_tile0 of the tile order on (tiles_m counts them).
// id: the workgroup's number among the tiles.  part != nullptr: the fp32 partial tile goes to part[z][M][N] (summed by k_gemm_finish), else bf16 to Cout.
struct GemmSmallArgs {
    const uint16_t *S, *W, *side, *ap, *zero;
    uint16_t *Cout;
    float *part;
    int tiles_m, tiles_n, n_split, row_tile0, M, Kd, N, n_seg;
};
template <bool FWD, int BM, bool DEEP, bool ACC, bool EXT>
__device__ __forceinline__ void gemm_small_tile(const MetaView &mv, const GemmSmallArgs &ga, int id, char *lds)
{
    static_assert(BM == 64 || BM == 128, "");
    constexpr int NW = 4;                                      // waves, two by two
    constexpr int WM = BM / 2;                                 // rows per wave
    constexpr int MB = WM / 16;                                // 16-row blocks per wave
    constexpr int XT = BM * GS_BK * 2, WT = GS_BN * GS_BK * 2;
    constexpr int NX = gs_ring_x(BM), NWR = gs_ring_w(BM, DEEP);               // ring slots of the token tile and of the W tile
    // equal rings: the two tiles of a stage side by side; deep: the W ring behind the token ring
    constexpr int XSLOT = DEEP ? XT : XT + WT, WSLOT = DEEP ? WT : XT + WT, kW = DEEP ? NX * XT : XT;
    constexpr int XL = BM / 8 / NW, WL = 16 / NW, LPS = XL + WL;   // load instructions (1 KB) per wave per stage
    const uint16_t *__restrict__ S = ga.S, *__restrict__ W = ga.W, *__restrict__ side = ga.side, *__restrict__ ap = ga.ap, *__restrict__ zero = ga.zero;
    uint16_t *__restrict__ Cout = ga.Cout;
    float *__restrict__ part = ga.part;
    const int tiles_m = ga.tiles_m, tiles_n = ga.tiles_n, n_split = ga.n_split, row_tile0 = ga.row_tile0, M = ga.M, Kd = ga.Kd, N = ga.N, n_seg = ga.n_seg;

    // workgroup -> (row tile, column tile, split).  Workgroups are dealt round-robin to the 8 XCDs; every XCD gets a
    // contiguous range of ids with the row tiles fastest, so that the workgroups that stream the same part of W share its L2.
    const int n_wg = tiles_m * tiles_n * n_split;
    {
        const int per = n_wg / 8;
        if (id < per * 8) id = (id % 8) * per + id / 8;
    }
    int m0 = (id % tiles_m) * BM;
    if (EXT && row_tile0 > 0) {                                       // the rest of a product that the 256-row kernel began
        m0 = mv.tile_order[row_tile0 + m0 / kGemmTileRows] * kGemmTileRows + m0 % kGemmTileRows;
        if (m0 >= M) return;
    }
    const int rest = id / tiles_m;
    const int n0 = (rest % tiles_n) * GS_BN, z = rest / tiles_n;
    const int m1 = m0 + BM < M ? m0 + BM : M;
    const int ldw = FWD ? N : Kd;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t lds_base = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)LDS_PTR(char, lds));

    // ---- the segments that overlap this row tile: a window of up to 64 records of the segment table, one per lane, from
    // which the extension steps are looked up (tiles with segments beyond the window move it; rare)
    const int win0 = !EXT || n_seg <= 64 ? 0 : mv.tile[m0 / kGemmTileRows].first_seg;
    int win = win0;
    int s_row0, s_row1, s_rp, s_r, s_cnt, s_cum, win_first = 0, win_ext;
    int64_t s_hb, s_op;                                        // s_op: GemmSeg::B (as address) or ap_off
    auto load_window = [&]() {
        const int idx = win + lane;
        SegInfo g;
        g.row0 = 0; g.row1 = 0; g.adapter = -1; g.r = 0; g.rp = 0; g.hb_off = 0;
        if (idx < n_seg) g = mv.seg[idx];
        const bool in = g.adapter >= 0 && g.row1 > g.row0 && g.row0 < m1 && g.row1 > m0;
        s_row0 = g.row0; s_row1 = g.row1; s_rp = g.rp; s_r = g.r; s_hb = g.hb_off; s_op = 0;
        if (in) {
            const AdapterInfo *a = mv.ad + g.adapter;
            s_op = FWD ? (int64_t)(uintptr_t)a->ext_b : a->ap_off;
        }
        s_cnt = in ? g.rp / kRankPadGemm : 0;
        int c = s_cnt;                                         // inclusive prefix sum over the wave
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int v = __shfl_up(c, d);
            if (lane >= d) c += v;
        }
        s_cum = c - s_cnt;
        win_ext = __builtin_amdgcn_readlane(c, 63);
        asm volatile("" : "+v"(s_op));                         // the records have arrived: nothing below waits for them again
    };
    int n_ext = 0;
    if constexpr (EXT) {
        load_window();
        n_ext = win_ext;
    }
    if (EXT && n_seg > 64) {                                          // count the extension steps of the segments beyond the window
        for (int w = win0 + 64; w < n_seg; w += 64) {
            const int idx = w + lane;
            int cnt = 0, past = 1;
            if (idx < n_seg) {
                const SegInfo g = mv.seg[idx];
                past = g.row0 >= m1;
                if (!past && g.adapter >= 0 && g.row1 > g.row0 && g.row1 > m0) cnt = g.rp / kRankPadGemm;
            }
#pragma unroll
            for (int d = 32; d; d >>= 1) cnt += __shfl_xor(cnt, d);
            n_ext += __builtin_amdgcn_readfirstlane(cnt);
            if (__builtin_amdgcn_readlane(past, 0)) break;
        }
    }

    // steps of this split: main steps [k_lo, k_hi), then extension steps z, z + n_split, ...
    const int nk_main = (Kd + GS_BK - 1) / GS_BK;
    const int k_lo = (int)((int64_t)nk_main * z / n_split), k_hi = (int)((int64_t)nk_main * (z + 1) / n_split);
    const int n_main = k_hi - k_lo;
    const int n_it = n_main + (n_ext > z ? (n_ext - z + n_split - 1) / n_split : 0);

    // ---- loader.  Token tile [BM][8 chunks]: instruction q covers rows 8q .. 8q+7, lane -> (row 8q + lane/8, slot lane%8),
    // slot c' of row u holds chunk c' ^ ((u >> 1) & 7).  W tile [128 n][8 chunks]: the same.  FWD W tile [64 k][16 chunks]:
    // instruction q covers k rows 4q .. 4q+3, slot c' of row u holds chunk c' ^ (2 (u & 3) + 8 ((u >> 3) & 1)).
    uint32_t off_x[XL], off_w[WL];
    const int lrow = lane >> 3;
    auto row_chunk = [&](int u) { return (lane & 7) ^ ((u >> 1) & 7); };
    auto kw_chunk = [&](int u) { return (lane & 15) ^ (2 * (u & 3) + 8 * ((u >> 3) & 1)); };
#pragma unroll
    for (int jj = 0; jj < XL; ++jj) {
        const int u = (wave + NW * jj) * 8 + lrow;
        int row = m0 + u;
        row = row < M ? row : M - 1;                           // clamped rows and columns only feed outputs that are not stored
        off_x[jj] = (uint32_t)(row - m0) * (uint32_t)Kd * 2u + (uint32_t)row_chunk(u) * 16u;
    }
#pragma unroll
    for (int jj = 0; jj < WL; ++jj) {
        if (FWD) {
            const int u = (wave + NW * jj) * 4 + (lane >> 4);
            int n = n0 + kw_chunk(u) * 8;
            n = n < N ? n : N - 8;
            off_w[jj] = (uint32_t)u * (uint32_t)ldw * 2u + (uint32_t)(n - n0) * 2u;
        } else {
            const int u = (wave + NW * jj) * 8 + lrow;
            int n = n0 + u;
            n = n < N ? n : N - 1;
            off_w[jj] = (uint32_t)(n - n0) * (uint32_t)ldw * 2u + (uint32_t)row_chunk(u) * 16u;
        }
    }
    const char *base_x = reinterpret_cast<const char *>(S) + (int64_t)m0 * Kd * 2;
    const char *base_w = reinterpret_cast<const char *>(W) + (FWD ? (int64_t)n0 * 2 : (int64_t)n0 * ldw * 2);
    auto load_ptr = [&](const void *g, uint32_t dst) {
        asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(g), "s"(dst));
    };
    auto load_off = [&](uint32_t off, const char *base, uint32_t dst) {
        asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(dst));
    };
    // extension step e -> lane that holds its segment's record, and the rank column it starts at
    auto find_ext = [&](int e, int &kk) {
        if (DEEP && e < win_first) { win = win0; win_first = 0; load_window(); }
        while (e - win_first >= win_ext) { win_first += win_ext; win += 64; load_window(); }
        const int le = e - win_first;
        const int l = __builtin_ctzll(__ballot(s_cum <= le && le < s_cum + s_cnt));
        kk = (le - __builtin_amdgcn_readlane(s_cum, l)) * kRankPadGemm;
        return l;
    };
    auto main_w = [&](int it, int slot) {
        const uint32_t dw = lds_base + kW + slot * WSLOT + wave * 1024;
        const int k0 = (k_lo + it) * GS_BK;
        const char *gw = base_w + (FWD ? (int64_t)k0 * ldw * 2 : (int64_t)k0 * 2);
        if (k0 + GS_BK <= Kd) {
#pragma unroll
            for (int jj = 0; jj < WL; ++jj) load_off(off_w[jj], gw, dw + jj * (NW * 1024));
        } else {                                           // last, partial step: chunks past the end read the zero page
#pragma unroll
            for (int jj = 0; jj < WL; ++jj) {
                const int u = FWD ? (wave + NW * jj) * 4 + (lane >> 4) : (wave + NW * jj) * 8 + lrow;
                const bool ok = FWD ? k0 + u < Kd : k0 + row_chunk(u) * 8 < Kd;
                load_ptr(ok ? static_cast<const void *>(gw + off_w[jj]) : zero, dw + jj * (NW * 1024));
            }
        }
    };
    auto ext_w = [&](int l, int kk, int slot) {
        const uint32_t dw = lds_base + kW + slot * WSLOT + wave * 1024;
        const int rp = __builtin_amdgcn_readlane(s_rp, l), r = __builtin_amdgcn_readlane(s_r, l);
        const int64_t op = gs_readlane64(s_op, l);
#pragma unroll
        for (int jj = 0; jj < WL; ++jj) {
            const uint16_t *gw;
            if (FWD) {
                const int u = (wave + NW * jj) * 4 + (lane >> 4);
                int n = n0 + kw_chunk(u) * 8;
                n = n < N ? n : N - 8;
                const int j = kk + u;                          // row of the [r][N] operand
                gw = j < r ? reinterpret_cast<const uint16_t *>((uintptr_t)op) + ((uint32_t)j * (uint32_t)ldw + (uint32_t)n) : zero;
            } else {
                const int u = (wave + NW * jj) * 8 + lrow;
                int n = n0 + u;
                n = n < N ? n : N - 1;                         // row of the padded [N][rp] operand
                gw = ap + op + (int64_t)n * rp + kk + row_chunk(u) * 8;
            }
            load_ptr(gw, dw + jj * (NW * 1024));
        }
    };
    auto main_x = [&](int it, int slot) {
        const uint32_t dx = lds_base + slot * XSLOT + wave * 1024;
        const int k0 = (k_lo + it) * GS_BK;
        const char *gx = base_x + (int64_t)k0 * 2;
        if (k0 + GS_BK <= Kd) {
#pragma unroll
            for (int jj = 0; jj < XL; ++jj) load_off(off_x[jj], gx, dx + jj * (NW * 1024));
        } else {
#pragma unroll
            for (int jj = 0; jj < XL; ++jj) {
                const int u = (wave + NW * jj) * 8 + lrow;
                load_ptr(k0 + row_chunk(u) * 8 < Kd ? static_cast<const void *>(gx + off_x[jj]) : zero, dx + jj * (NW * 1024));
            }
        }
    };
    auto ext_x = [&](int l, int kk, int slot) {
        const uint32_t dx = lds_base + slot * XSLOT + wave * 1024;
        const int row0 = __builtin_amdgcn_readlane(s_row0, l), row1 = __builtin_amdgcn_readlane(s_row1, l);
        const int rp = __builtin_amdgcn_readlane(s_rp, l);
        const int64_t hb = gs_readlane64(s_hb, l);
#pragma unroll
        for (int jj = 0; jj < XL; ++jj) {
            const int u = (wave + NW * jj) * 8 + lrow;
            const int row = m0 + u;
            const bool in = row >= row0 && row < row1;         // rows of other segments contribute nothing
            load_ptr(in ? side + hb + (int64_t)(row - row0) * rp + kk + row_chunk(u) * 8 : zero, dx + jj * (NW * 1024));
        }
    };

    auto issue_w = [&](int it, int slot) {
        if (!EXT || it < n_main) { main_w(it, slot); return; }
        int kk;
        const int l = find_ext(z + (it - n_main) * n_split, kk);
        ext_w(l, kk, slot);
    };
    auto issue_x = [&](int it, int slot) {
        if (!EXT || it < n_main) { main_x(it, slot); return; }
        int kk;
        const int l = find_ext(z + (it - n_main) * n_split, kk);
        ext_x(l, kk, slot);
    };
    auto issue = [&](int it, int slot) {                       // both tiles of a stage (rings of equal length)
        if (!EXT || it < n_main) { main_w(it, slot); main_x(it, slot); return; }
        int kk;
        const int l = find_ext(z + (it - n_main) * n_split, kk);
        ext_w(l, kk, slot);
        ext_x(l, kk, slot);
    };

    // ---- MFMA operands: lane (lm, kg) reads row lm of its 16-row block, chunk 4 ks + kg
    const int lm = lane & 15, kg = lane >> 4;
    const int wm0 = (wave >> 1) * WM, wn0 = (wave & 1) * 64;
    int xoff[MB], woff[4];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        const int u = wm0 + mb * 16 + lm;
        xoff[mb] = u * 128 + ((kg ^ ((u >> 1) & 7)) * 16);
    }
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) {
        if (FWD) {                                             // transposing read: see tokcontract_bf16.hip
            const int u = kg * 8 + (lm >> 2);
            const int cl = wn0 + nb * 16 + (lm & 3) * 4;
            woff[nb] = u * 256 + ((((cl >> 3) ^ (2 * (u & 3) + 8 * ((u >> 3) & 1))) * 16) + (cl & 7) * 2);
        } else {
            const int u = wn0 + nb * 16 + lm;
            woff[nb] = u * 128 + ((kg ^ ((u >> 1) & 7)) * 16);
        }
    }
    f32x4 acc[4][MB];
#pragma unroll
    for (int nb = 0; nb < 4; ++nb)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[nb][mb] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Stage `it` of the token tile is requested NX - 1 stages ahead, of the W tile NWR - 1.  Loads complete in order, so what
    // may still fly when stage `it` is needed is what was requested behind the later of its two tiles: the stages after it,
    // or - deep: the token tile goes out in front of a W tile that is one stage further on - that W tile.
    static_assert(!DEEP || (BM == 128 && NX == 2 && NWR == 3), "the deep ring is counted for these slots");
    constexpr int FLY = DEEP ? WL : (NX - 2) * LPS;
#pragma unroll
    for (int p = 0; p < NWR - 1; ++p) {
        if (p >= n_it) break;
        if constexpr (DEEP) {
            if (p < NX - 1) issue_x(p, p);
            issue_w(p, p);
        } else {
            issue(p, p);
        }
    }
    int rx = 0, rw = 0, wr = NX - 1;
    for (int it = 0; it < n_it; ++it) {
        // this wave's loads of stage `it` have landed ...
        if (it + NWR - 1 <= n_it) gs_wait_vmcnt<FLY>();
        else gs_wait_vmcnt<0>();
        __builtin_amdgcn_s_waitcnt(0xc07f);                    // ... its LDS reads of the slots about to be refilled are done ...
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();                          // ... and so are everyone else's
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (DEEP) {
            if (it + NX - 1 < n_it) issue_x(it + NX - 1, rx == 0 ? NX - 1 : rx - 1);
            if (it + NWR - 1 < n_it) issue_w(it + NWR - 1, rw == 0 ? NWR - 1 : rw - 1);
        } else {
            if (it + NX - 1 < n_it) issue(it + NX - 1, wr);
            wr = wr + 1 == NX ? 0 : wr + 1;
        }
        const char *sx = lds + rx * XSLOT, *sw = DEEP ? lds + kW + rw * WSLOT : sx + kW;
        rx = rx + 1 == NX ? 0 : rx + 1;
        if constexpr (DEEP) rw = rw + 1 == NWR ? 0 : rw + 1;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            bf16x8 xf[MB], wf[4];
#pragma unroll
            for (int nb = 0; nb < 4; ++nb) {
                if (FWD) {
                    const char *p = sw + woff[nb] + ks * 32 * 256;
                    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(LDS_PTR(bf16x4, p));
                    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(LDS_PTR(bf16x4, p + 4 * 256));
                    wf[nb] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                } else {
                    wf[nb] = *LDS_PTR(const bf16x8, sw + (woff[nb] ^ (ks * 64)));
                }
            }
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) xf[mb] = *LDS_PTR(const bf16x8, sx + (xoff[mb] ^ (ks * 64)));
            // the workgroup that multiplies goes first: its partner on the compute unit is then fetching, and they stay out of
            // step (128 rows: 4 - 6 % of the kernel; 64 rows: slower by 1 %, left alone)
            if constexpr (BM == 128) __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int nb = 0; nb < 4; ++nb)
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
                    acc[nb][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[nb], xf[mb], acc[nb][mb], 0, 0, 0);
            if constexpr (BM == 128) __builtin_amdgcn_s_setprio(0);
        }
    }

    // ---- epilogue: a lane holds, of token wm0 + 16 mb + lm, the columns wn0 + 16 nb + 4 kg .. + 3
    if (!EXT || part) {
        float *dst = part + (int64_t)z * M * N;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const int m = m0 + wm0 + mb * 16 + lm;
#pragma unroll
            for (int nb = 0; nb < 4; ++nb) {
                const int n = n0 + wn0 + nb * 16 + kg * 4;
                if (m < M && n < N) *reinterpret_cast<f32x4 *>(dst + (int64_t)m * N + n) = acc[nb][mb];
            }
        }
        return;
    }
    // bf16: each wave passes 16 x 64 blocks through 2 KB of LDS of its own and stores whole 128-byte rows
    __builtin_amdgcn_s_waitcnt(0xc07f);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();                              // the ring is free (every load has landed: the last wait was 0)
    __builtin_amdgcn_sched_barrier(0);
    char *stg = lds + wave * 2048;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) {
            uint2 v;
            v.x = gs_pack_bf16x2(acc[nb][mb][0], acc[nb][mb][1]);
            v.y = gs_pack_bf16x2(acc[nb][mb][2], acc[nb][mb][3]);
            const int chunk = nb * 2 + (kg >> 1);
            *reinterpret_cast<uint2 *>(stg + lm * 128 + ((chunk ^ (lm & 7)) * 16) + (kg & 1) * 8) = v;
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int row = (lane >> 3) + 8 * j, c = lane & 7;
            uint4 v = *reinterpret_cast<const uint4 *>(stg + row * 128 + ((c ^ (row & 7)) * 16));
            const int m = m0 + wm0 + mb * 16 + row, n = n0 + wn0 + c * 8;
            if (m < M && n < N) {
                uint4 *dst = reinterpret_cast<uint4 *>(Cout + (int64_t)m * N + n);
                if constexpr (ACC) {
                    const uint4 o = *dst;
                    v.x = gs_add_bf16x2(o.x, v.x); v.y = gs_add_bf16x2(o.y, v.y);
                    v.z = gs_add_bf16x2(o.z, v.z); v.w = gs_add_bf16x2(o.w, v.w);
                }
                *dst = v;
            }
        }
    }
}

// Sums the fp32 partial tiles [split][M][N] in split order and rounds to bf16 (ACC: added to what Cout holds, as the
// epilogue of an unsplit call does).  4 elements per thread, eight partial tiles requested at a time.
template <bool ACC>
__device__ inline void gemm_finish(const float *__restrict__ part, uint16_t *__restrict__ Cout, int64_t n_vec, int n_split, int64_t i)
{
    if (i >= n_vec) return;
    const float4 *p = reinterpret_cast<const float4 *>(part) + i;
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int z0 = 0; z0 < n_split; z0 += 8) {
        float4 v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (z0 + j < n_split) v[j] = p[(z0 + j) * n_vec];
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (z0 + j < n_split) { a.x += v[j].x; a.y += v[j].y; a.z += v[j].z; a.w += v[j].w; }
    }
    uint2 v;
    v.x = gs_pack_bf16x2(a.x, a.y); v.y = gs_pack_bf16x2(a.z, a.w);
    uint2 *dst = reinterpret_cast<uint2 *>(Cout) + i;
    if constexpr (ACC) {
        const uint2 o = *dst;
        v.x = gs_add_bf16x2(o.x, v.x); v.y = gs_add_bf16x2(o.y, v.y);
    }
    *dst = v;
}

}  // namespace plora
