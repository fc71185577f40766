// Forward of a short batch in two launches: what does not depend on each other, then what does.
//
// k_short_products: the metadata tables, the shrink x A_k in slices of 16 tokens (skinny_short.h, the sums of every share of the
// contraction as they are) and the base product x W in split small tiles (gemm_small.h, without low-rank steps) are workgroups of one
// launch.  k_short_finish adds up both sets of partial sums in order and the low-rank term behind them: per 16 tokens of one
// segment and 128 columns, s h is rounded to bf16 as everywhere, multiplied with B_k on MFMA 16x16x32 into the fp32 sum, which
// is rounded once.  No B_k^T is packed for it, whatever the order of W.
// Bound by two launches and, in the first, by the stream of W beside the shrink's chain of description, operands and sums.  Before, the
// shrink and the packing of B_k were a launch in front of the product (9 - 20 us), the product's sum a third.  Whole forward calls, us,
// before and now, W from HBM: 48 tokens, 4096 -> 4096, eight adapters 27.9 and 19.8; 1 token, 4696 -> 2816 21.4 and 15.1; 255 tokens,
// 3024 -> 3664 42.4 and 27.3; 8 tokens, 3296 -> 5776 24.3 and 17.1; the projections of a group together: three of 942 tokens, 640 ->
// 512, 128, 128 a step 115 and 82.  The finishing launch alone is 5 - 8 us, three trips to the description and one to the sums.
#include "gemm_small.h"
#include "prep.h"
#include "skinny_short.h"

#include <algorithm>
#include <cstring>

namespace plora {

// The 16-token slice `unit` of the segments with tokens, in order (one lane per segment, 64 at a time): its segment (rows, adapter, rank,
// h_off), its first token inside the segment and the scale.
template <class Src>
__device__ __forceinline__ SegInfo segment_of_slice(const DescReader<Src> &in, int unit, int &t0, float &scale)
{
    const int n_seg = in.n_seg(), lane = threadIdx.x & 63;
    int64_t h = 0;
    int first = 0;
    SegInfo g;
    g.row0 = 0; g.row1 = 0; g.adapter = -1; g.r = 0; g.rp = 0; g.r16 = 0; g.blk0 = 0; g.lp = 0; g.h_off = 0; g.hb_off = 0; g.zt_off = 0;
    t0 = 0; scale = 0.f;
    for (int s0 = 0; s0 < n_seg; s0 += 64) {
        const int s = s0 + lane;
        int len = 0, r = 0, row0 = 0, k = -1;
        if (s < n_seg) {
            k = in.seg_adapter(s);
            row0 = in.seg_row0(s);
            len = in.seg_row1(s) - row0;
            if (k >= 0) r = in.ad_rank(k);
        }
        const int n = (len + 15) / 16;
        const int64_t he = (int64_t)len * r;
        const int n_inc = wave_scan(n);
        const int64_t h_inc = wave_scan(he);
        const uint64_t own = __ballot(unit < first + n_inc && unit >= first + n_inc - n);
        if (own) {
            const int l = __builtin_ctzll(own);
            auto at = [&](int v) { return __builtin_amdgcn_readlane(v, l); };
            g.row0 = at(row0); g.row1 = g.row0 + at(len); g.adapter = at(k); g.r = at(r);
            g.r16 = pad_to(g.r, kRankPadMfma); g.lp = pad_to(g.row1 - g.row0, kTokPad);
            g.h_off = h + gs_readlane64(h_inc - he, l);
            t0 = (unit - first - at(n_inc) + at(n)) * 16;
            if (g.adapter >= 0) scale = in.ad_scale(g.adapter);
            break;
        }
        first += __builtin_amdgcn_readlane(n_inc, 63);
        h += gs_readlane64(h_inc, 63);
    }
    return g;
}

__device__ __attribute__((aligned(16))) const uint32_t g_short_zeros[4] = {0u, 0u, 0u, 0u};    // the zero page is written in the same launch

// One call, or the projections of a grouped call (NP of them) whose plans and weight orders agree.
struct ShortProducts {
    char *meta_dst;
    uint32_t *zero_page;
    ShortJob job;
    GemmSmallArgs ga;
    int32_t n_units, n_gemm;
    int32_t word0, wg0;           // first word of its description, first workgroup
};
template <int NP> struct ShortWords { uint32_t w[NP == 1 ? kChunkWords : 640]; };
template <int NP> struct ShortBatch {
    ShortProducts p[NP];
    int32_t n;
    ShortWords<NP> c;
};
static_assert(sizeof(ShortBatch<1>) <= 4000 && sizeof(ShortBatch<kMaxGroup>) <= 4000, "a kernel argument");

// Workgroups of a call: one for the tables, n_gemm of the base product, then the shares of the shrink, all slices of a share side by side.
template <bool FWD, int BM, bool DEEP, int NP>
__global__ void __launch_bounds__(256, 2) k_short_products(ShortBatch<NP> sb)
{
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    int q = 0;
    if constexpr (NP > 1)
        for (int i = 1; i < NP; ++i)
            if (i < sb.n && (int)blockIdx.x >= sb.p[i].wg0) q = i;
    const ShortProducts &sp = sb.p[q];
    const DescReader<WordsInArg> in{WordsInArg{sb.c.w + sp.word0}};
    int wg = (int)blockIdx.x - sp.wg0;
    if (wg == 0) {
        sp.zero_page[threadIdx.x] = 0u;                        // kZeroBytes = 256 * 4
        derive_on_device(in, sp.meta_dst, lds);
        return;
    }
    wg -= 1;
    if (wg < sp.n_gemm) {
        // the compiler lets the branches of this kernel run into one another, and without a wait here would wait in every stage for
        // loads of the shrink (283 tokens, 2192 -> 6272: 42 us instead of 28)
        __builtin_amdgcn_s_waitcnt(0);
        GemmSmallArgs ga = sp.ga;
        ga.zero = reinterpret_cast<const uint16_t *>(g_short_zeros);
        gemm_small_tile<FWD, BM, DEEP, false, false>(MetaView{}, ga, wg, lds);
        return;
    }
    wg -= sp.n_gemm;
    const int split = wg / sp.n_units, unit = wg - split * sp.n_units;
    int t0;
    float scale;
    const SegInfo g = segment_of_slice(in, unit, t0, scale);
    if (g.adapter < 0) return;
    const uint16_t *A = static_cast<const uint16_t *>(in.ad_ptr(g.adapter, 0));
    const ShortJob job = sp.job;
    const int nb = job.max_r16 / 16;
    if (nb <= 1) skinny_short<1, true>(job, g, scale, t0, unit, sp.n_units, split, A, true, lds);
    else if (nb <= 2) skinny_short<2, true>(job, g, scale, t0, unit, sp.n_units, split, A, true, lds);
    else if (nb <= 4) skinny_short<4, true>(job, g, scale, t0, unit, sp.n_units, split, A, true, lds);
    else skinny_short<8, true>(job, g, scale, t0, unit, sp.n_units, split, A, true, lds);
}

struct ShortFinish {
    const float *h_part, *y_part;
    uint16_t *y;
    float *hf;
    int32_t n_units, h_split, max_r16, y_split, M, N, max_steps, word0;
};
template <int NP> struct ShortFinishBatch {
    ShortFinish p[NP];
    ShortWords<NP> c;
};
// A wave takes CB blocks of 16 columns: two while that leaves the chip with one round of workgroups, whose chain of loads is what a launch
// costs then, else four.
template <int CB, int NP>
__global__ void __launch_bounds__(256, 4) k_short_finish(ShortFinishBatch<NP> fb)
{
    constexpr int BN = 64 * CB, PITCH = 32 * CB, LPR = 2 * CB, RPI = 64 / LPR, NI = 32 / RPI;    // columns of the workgroup; bytes and 16-byte loads of a wave's row, rows and instructions per step
    extern __shared__ __attribute__((aligned(16))) char fin_lds[];
    char *h_lds = fin_lds;                                     // s h as the second operand of up to four steps of 32 ranks
    const ShortFinish f = fb.p[NP > 1 ? blockIdx.z : 0];
    if (NP > 1 && (int)blockIdx.y * BN >= f.N) return;         // of a narrower projection
    const DescReader<WordsInArg> in{WordsInArg{fb.c.w + f.word0}};
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lm = lane & 15, kg = lane >> 4;
    const int unit = blockIdx.x, n0 = blockIdx.y * BN + wave * (16 * CB);
    int t0;
    float scale;
    const SegInfo g = segment_of_slice(in, unit, t0, scale);
    const int nt = g.row1 - g.row0 - t0, N = f.N;
    const int row = g.row0 + t0 + (lm < nt ? lm : nt - 1);     // rows past the end are not stored
    const int r = g.r, n_steps = (r + 31) / 32;
    char *b_lds = fin_lds + f.max_steps * (1024 + wave * (32 * PITCH));     // the wave's columns of B_k, 32 rows per step
    if (g.adapter >= 0) {
        const uint16_t *B = static_cast<const uint16_t *>(in.ad_ptr(g.adapter, 1));
        uint4 b[4][NI];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if (s >= n_steps) break;
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int j = s * 32 + i * RPI + lane / LPR, n = n0 + lane % LPR * 8;
                const bool ok = j < r && n < N;
                b[s][i] = *reinterpret_cast<const uint4 *>(B + (ok ? (int64_t)j * N + n : 0));
                if (!ok) b[s][i] = make_uint4(0u, 0u, 0u, 0u);
            }
        }
        if (wave < n_steps) {                                  // this wave's step of s h: the shares of the shrink in order
            const int j = wave * 32 + kg * 8;
            float h[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) h[i] = 0.f;
            if (j < g.r16) {
                const int64_t stride = (int64_t)f.n_units * 16 * f.max_r16;
                const float *src = f.h_part + (int64_t)unit * 16 * f.max_r16 + lm * g.r16 + j;
                for (int z0 = 0; z0 < f.h_split; z0 += 4) {
                    float4 v[4][2];
#pragma unroll
                    for (int z = 0; z < 4; ++z) {
                        if (z0 + z >= f.h_split) break;
                        v[z][0] = *reinterpret_cast<const float4 *>(src + (z0 + z) * stride);
                        v[z][1] = *reinterpret_cast<const float4 *>(src + (z0 + z) * stride + 4);
                    }
#pragma unroll
                    for (int z = 0; z < 4; ++z) {
                        if (z0 + z >= f.h_split) break;
                        h[0] += v[z][0].x; h[1] += v[z][0].y; h[2] += v[z][0].z; h[3] += v[z][0].w;
                        h[4] += v[z][1].x; h[5] += v[z][1].y; h[6] += v[z][1].z; h[7] += v[z][1].w;
                    }
                }
            }
            if (f.hf && blockIdx.y == 0 && lm < nt) {
                float *dst = f.hf + g.h_off + (int64_t)(t0 + lm) * r;
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (j + i < r) dst[j + i] = h[i];
            }
            union { uint4 q; uint16_t v[8]; } u;
#pragma unroll
            for (int i = 0; i < 8; ++i) u.v[i] = j + i < r ? bf16_rne(scale * h[i]) : (uint16_t)0;     // past the rank: sums of what lay behind A_k
            *reinterpret_cast<uint4 *>(h_lds + (wave * 64 + lane) * 16) = u.q;
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if (s >= n_steps) break;
#pragma unroll
            for (int i = 0; i < NI; ++i) *reinterpret_cast<uint4 *>(b_lds + s * (32 * PITCH) + i * 1024 + lane * 16) = b[s][i];
        }
    }
    sh_f32x4 acc[CB];
#pragma unroll
    for (int nb = 0; nb < CB; ++nb) acc[nb] = sh_f32x4{0.f, 0.f, 0.f, 0.f};
    const int64_t part_stride = (int64_t)f.M * N;
    constexpr int ZB = 16 / CB;                                // partial tiles requested at a time
    for (int z0 = 0; z0 < f.y_split; z0 += ZB) {
        sh_f32x4 v[ZB][CB];
#pragma unroll
        for (int z = 0; z < ZB; ++z) {
            if (z0 + z >= f.y_split) break;
#pragma unroll
            for (int nb = 0; nb < CB; ++nb) {
                const int n = n0 + nb * 16 + kg * 4;
                v[z][nb] = *reinterpret_cast<const sh_f32x4 *>(f.y_part + (z0 + z) * part_stride + (int64_t)row * N + (n < N ? n : 0));
            }
        }
#pragma unroll
        for (int z = 0; z < ZB; ++z) {
            if (z0 + z >= f.y_split) break;
#pragma unroll
            for (int nb = 0; nb < CB; ++nb) acc[nb] += v[z][nb];
        }
    }
    __syncthreads();
    if (g.adapter >= 0) {
        for (int s = 0; s < n_steps; ++s) {
            const sh_bf16x8 hf = *reinterpret_cast<const sh_bf16x8 *>(h_lds + (s * 64 + lane) * 16);
#pragma unroll
            for (int nb = 0; nb < CB; ++nb) {
                // transposing read: the 16 lanes of a group fetch a 4(k) x 16 block; lane i then holds column i
                const char *q = b_lds + s * (32 * PITCH) + (kg * 8 + (lm >> 2)) * PITCH + (nb * 16 + (lm & 3) * 4) * 2;
                const sh_bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(SH_LDS_PTR(sh_bf16x4, q));
                const sh_bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(SH_LDS_PTR(sh_bf16x4, q + 4 * PITCH));
                const sh_bf16x8 wf = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, hf, acc[nb], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int nb = 0; nb < CB; ++nb) {
        const int n = n0 + nb * 16 + kg * 4;
        if (lm >= nt || n >= N) continue;
        uint2 v;
        v.x = gs_pack_bf16x2(acc[nb][0], acc[nb][1]); v.y = gs_pack_bf16x2(acc[nb][2], acc[nb][3]);
        *reinterpret_cast<uint2 *>(f.y + (int64_t)row * N + n) = v;
    }
}

template <bool FWD, int BM, bool DEEP, int NP>
static hipError_t launch_products(ShortBatch<NP> &sb, size_t lds, int slot, hipStream_t st)
{
    constexpr size_t ring = (size_t)(gs_ring_x(BM) * BM + gs_ring_w(BM, DEEP) * GS_BN) * GS_BK * 2;
    if (lds < ring) lds = ring;
    int wgs = 0;
    for (int i = 0; i < sb.n; ++i) {
        ShortProducts &sp = sb.p[i];
        sp.ga.tiles_m = (sp.ga.M + BM - 1) / BM; sp.ga.tiles_n = (sp.ga.N + GS_BN - 1) / GS_BN;
        sp.n_gemm = sp.ga.tiles_m * sp.ga.tiles_n * sp.ga.n_split;
        sp.wg0 = wgs;
        wgs += 1 + sp.n_gemm + sp.n_units * sp.job.n_split;
    }
    auto kern = k_short_products<FWD, BM, DEEP, NP>;
    const hipError_t e = allow_full_lds(reinterpret_cast<const void *>(kern), slot + (NP > 1 ? 6 : 0));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)wgs), dim3(256), lds, st, sb);
    return hipGetLastError();
}

template <int NP>
static hipError_t launch_batch(const ShortForward *const *ops, int n, hipStream_t st)
{
    ShortBatch<NP> sb{};
    ShortFinishBatch<NP> fb{};
    sb.n = n;
    size_t lds = 0;
    int64_t widest = 0;
    int max_steps = 0, words = 0;
    for (int i = 0; i < n; ++i) {
        const ShortForward &o = *ops[i];
        const MetaHeader &h = o.h;
        ShortProducts &sp = sb.p[i];
        sp.meta_dst = o.meta_dev; sp.zero_page = static_cast<uint32_t *>(o.zero_dev);
        sp.n_units = o.slices;
        sp.job.S = static_cast<const uint16_t *>(o.x); sp.job.part = o.h_part;
        sp.job.C = (int32_t)h.D; sp.job.mode = 0; sp.job.max_r16 = h.max_r16;
        sp.job.n_split = o.shares.n; sp.job.per = o.shares.per;
        sp.ga = GemmSmallArgs{static_cast<const uint16_t *>(o.x), static_cast<const uint16_t *>(o.W), nullptr, nullptr, nullptr, nullptr, o.y_part,
                              0, 0, o.plan.n_split, 0, (int)h.T, (int)h.D, (int)h.K, (int)h.n_seg};
        sp.word0 = words;
        const int steps = (h.max_r16 + 31) / 32;
        fb.p[i] = ShortFinish{o.h_part, o.y_part, static_cast<uint16_t *>(o.y), o.hf, o.slices, o.shares.n, h.max_r16, o.plan.n_split, (int)h.T, (int)h.K, steps, words};
        std::memcpy(sb.c.w + words, o.desc_host, (size_t)o.n_words * 4);
        words += o.n_words;
        lds = std::max(lds, std::max(derive_lds_bytes(o.n_words, h.n_seg), short_lds_bytes(h.max_r16)));
        widest = std::max(widest, h.K); max_steps = std::max(max_steps, steps);
    }
    std::memcpy(fb.c.w, sb.c.w, (size_t)words * 4);
    const ShortForward &o = *ops[0];
    const bool deep = gemm_small_deep(o.h.T);
    hipError_t e;
#define PL_SP(FWD_, BM_, DEEP_, SLOT_) launch_products<FWD_, BM_, DEEP_, NP>(sb, lds, SLOT_, st)
    if (o.h.w_out_in) e = o.plan.bm == 64 ? PL_SP(false, 64, false, 36) : deep ? PL_SP(false, 128, true, 37) : PL_SP(false, 128, false, 38);
    else e = o.plan.bm == 64 ? PL_SP(true, 64, false, 39) : deep ? PL_SP(true, 128, true, 40) : PL_SP(true, 128, false, 41);
#undef PL_SP
    if (e != hipSuccess) return e;
    const int64_t narrow = (widest + 127) / 128, wide = (widest + 255) / 256;
    if (n * o.slices * narrow <= 1024) {
        hipLaunchKernelGGL((k_short_finish<2, NP>), dim3((unsigned)o.slices, (unsigned)narrow, (unsigned)n), dim3(256), (size_t)max_steps * (1024 + 4 * 2048), st, fb);
    } else {
        e = allow_full_lds(reinterpret_cast<const void *>(&k_short_finish<4, NP>), NP > 1 ? 55 : 54);       // 68 KB at ranks above 96
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((k_short_finish<4, NP>), dim3((unsigned)o.slices, (unsigned)wide, (unsigned)n), dim3(256), (size_t)max_steps * (1024 + 4 * 4096), st, fb);
    }
    return hipGetLastError();
}

hipError_t launch_short_forward(const ShortForward *ops, int n, hipStream_t st)
{
    if (n < 0 || n > kMaxGroup) return hipErrorInvalidValue;
    bool done[kMaxGroup] = {};
    for (int i = 0; i < n; ++i)
        if (ops[i].n_words > kChunkWords || ops[i].plan.bm == 0 || ops[i].plan.big_tiles != 0 || ops[i].slices < 1) return hipErrorInvalidValue;
    for (int i = 0; i < n; ++i) {
        if (done[i]) continue;
        const ShortForward *batch[kMaxGroup];
        int m = 0, words = 0;
        for (int q = i; q < n; ++q) {
            if (done[q] || ops[q].plan.bm != ops[i].plan.bm || ops[q].h.w_out_in != ops[i].h.w_out_in) continue;
            if (m > 0 && words + ops[q].n_words > (int)(sizeof(ShortWords<kMaxGroup>) / 4)) continue;
            batch[m++] = &ops[q]; words += ops[q].n_words; done[q] = true;
        }
        const hipError_t e = m == 1 ? launch_batch<1>(batch, m, st) : launch_batch<kMaxGroup>(batch, m, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace plora
