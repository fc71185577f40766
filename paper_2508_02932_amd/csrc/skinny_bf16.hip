// Skinny rank-r products of the packed multi-LoRA layer on bf16 inputs (gfx950):
//   shrink  h_t = x_t A_k            (section 2.4; the first half of the low-rank update)
//   dH      g_t = scale_k dy_t B_k^T (appendix C.2, case 2)
// Both stream one big [T][C] matrix once (C = d_in or d_out) against a small per-adapter matrix
// whose rows are output columns with the contraction index contiguous (A_k^T packed, or B_k as it
// is).  They are bound by HBM, so the kernel is built around keeping bytes in flight: operands go
// HBM -> LDS directly (global_load_lds) through a two-stage ring (more workgroups per compute unit
// pay more here than a deeper ring: measured), the contraction is split over
// workgroups when the batch has too few token blocks to fill the chip, and the arithmetic runs on
// 16x16x32 bf16 MFMA with fp32 accumulators so that ranks up to 128 stay far below the
// matrix-core roof.  The rank is never tiled (appendix C.2: tile the sequence and hidden
// dimensions, not the rank).  Partial tiles of the splits are summed in a fixed order by a small
// finishing kernel that also writes the bf16 copies the later kernels consume.
// Short batches, where a kernel's own time is mostly its start, take skinny_short.h instead.
#include "prep.h"
#include "skinny_short.h"
#include <algorithm>
#include <cstring>
#include <type_traits>

namespace plora {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

#define LDS_PTR(T, p) ((__attribute__((address_space(3))) T *)(p))

constexpr int SK_BK = 64;                              // contraction elements per stage
constexpr int SK_NST = 2;                              // ring stages: 32-64 KB of LDS per workgroup, so 2-3 fit on a compute unit
constexpr int SK_XT = kSkinnyRows * SK_BK * 2;         // 16 KB: [128 tokens][64 k]
constexpr int SK_NW = kSkinnyRows / 32;                // waves per workgroup: a wave owns 32 tokens
constexpr int SK_XL = kSkinnyRows / 8 / SK_NW;         // token-tile load instructions per wave per stage (4)
constexpr int SK_MB = kSkinnyRows / 16 / SK_NW;        // 16-token MFMA blocks per wave (2)
constexpr int SK_BL = (PLORA_MAX_RANK / 8 + SK_NW - 1) / SK_NW;   // small-matrix load instructions per wave per stage, at most
constexpr int SK_MAXNB = PLORA_MAX_RANK / 16;
constexpr int64_t SH_MAX_BYTES = 64 << 20, SH_MAX_SMALL = 24000000, SH_MAX_SMALL_8 = 10000000;

// s_waitcnt vmcnt(n) for a wave-uniform runtime n (the instruction takes an immediate)
__device__ inline void wait_vmcnt_dyn(int n)
{
#define W_(N) case N: __builtin_amdgcn_s_waitcnt(0x0f70 | (N & 15) | ((N >> 4) << 14)); break;
    switch (n) {
        W_(0) W_(1) W_(2) W_(3) W_(4) W_(5) W_(6) W_(7) W_(8) W_(9) W_(10) W_(11) W_(12) W_(13) W_(14) W_(15)
        W_(16) W_(17) W_(18)
    default: __builtin_amdgcn_s_waitcnt(0x0f70); break;
    }
#undef W_
}

// One product of a launch.
struct SkinnyJob {
    const BlkInfo *blk;
    const uint16_t *S, *at;       // the big matrix [T][C]; mode 0: packed A_k^T
    float *part;                  // fp32 partial tiles
    SkinnyOut out;
    int32_t C, mode, per, n_split, max_r16;      // per: stages of 64 per split
    int32_t past;                 // S is read past the caches ...
    int32_t turn;                 // ... and from another stage in every workgroup
};
// How S is read, see k_skinny.  alone: of a stand-alone low-rank call; mean_r16: rank rows that a token reads on average.
static void set_past(SkinnyJob &j, const MetaHeader &h, bool alone, int mean_r16)
{
    const int64_t bytes = h.T * j.C * 2;
    const bool worth = bytes >= (170 << 20) || (bytes >= (64 << 20) && (j.mode == 0 ? h.K >= 1024 : j.max_r16 <= 64));
    j.past = (alone ? bytes >= (48 << 20) : worth) && rows_of_whole_lines(j.S, j.C);
    j.turn = j.past && (alone || j.mode == 1) && mean_r16 <= 52 && (int64_t)mean_r16 * j.C * 2 <= (3 << 19);
}
struct SkinnyBatch { SkinnyJob j[kMaxGroup]; };

// One workgroup (4 waves) per (token block of 128 rows of one segment, slice of the contraction).
// Stage = 64 contraction elements: the token tile [128][64] and the small-matrix tile [r16][64]
// land in LDS by direct loads (16-byte chunks XOR-swizzled by row so that MFMA operand reads are
// conflict free).  Wave w owns tokens 32w..32w+31 and every rank block, so nothing is reduced
// across waves.  Output: the fp32 partial tile [128][r16] of this slice.
//   mode 0: small matrix = packed A_k^T [r16][C] (rows >= r are zero),  mode 1: B_k [r][C].
// The big matrix may be read with the non-temporal hint, where its rows are whole lines of 128 bytes (rows_of_whole_lines; otherwise
// neighbouring stages share lines, which the hint lets go between them: 20000 tokens, 13000 columns 177 us, 195 with it).  With its
// finishing launch, us, without and with the hint: 32768 tokens, ranks 8 to 128, 8192 columns 147 and 133, 28672 columns 432 and 409;
// 16384 tokens of rank 64, 4096 columns 48 and 42, 14336 columns 127 and 116; of 142 shapes from 48 MB on none is slower with it.  But
// the product that reads the matrix next does not find it in the last cache (256 MB).  Whole steps over inputs that change, without
// and with the hint on all matrices from 48 MB on:
//   - from 170 MB on little would be left there: 21019 tokens, 8192 -> 512 (328 MB) 626 and 599, 20615 tokens, 512 -> 8192 (322 MB) 602
//     and 585
//   - x before a GEMM that is bound by its operations, from 64 MB on: 16462 tokens, 2048 -> 2048 (64 MB) 383 and 375, 17635 tokens, 2048 ->
//     1024 (69 MB) 271 and 264; a narrow one is not: 5912 tokens, 8192 -> 512 (92 MB) 256 and 266, 15639 tokens, 4096 -> 512 (122 MB) 405
//     and 420
//   - dy before k_tokc, which then reads it from memory: of small ranks dH gains more than that (16384 tokens, 4096 columns, rank 8 to 32 dH
//     48 -> 35, k_tokc 54 -> 62), of large ones less (4326 tokens, 14336 columns, rank 64 to 128 dH 61 -> 55, k_tokc 33 -> 44)
//   - in the stand-alone calls nothing but k_tokc reads it again: 9645 tokens, 8192 -> 1024 (151 MB) 283 and 275, 3812 tokens, 1024 -> 14336
//     (104 MB) 229 and 224
// With the hint, and where the ranks are small, every workgroup begins its slice at another stage: side by side from the same column on,
// the workgroups ask for 128-byte pieces whole rows apart, which lie in few of the memory channels (8192 tokens, rank 16, 16384 columns
// 59 -> 51, 32768 columns 118 -> 92; 16384 tokens, rank 8 to 64, 8192 columns 74 -> 69).  Side by side they also share each stage of the
// small matrix in the L2, which turned they read all over at once.  Rows of it per token on average, change over the widths from 4096
// to 49152 columns: 16 to 32 -22 to +4 %, 48 -7 to +6 %, 51 -5 %, 54 -3 to +3 %, 64 -1 to +18 %, 128 0 to +21 % (28672 columns 164 -> 191): up to
// 52, and 1.5 MB (26 rows, 49152 columns 338 -> 350).  Not the shrink of the other calls: a fused one has to sum as the plain ones of its
// projections do, whose ranks differ.
// grid.z: the jobs of the batch (dH of the projections of a grouped call).
// GROUP (mode 0 only): the small matrix of adapter k is the packed A_k^T of several projections, one below the other
// (GroupView); the tables are projection 0's, `at` is not used, and the jobs are where each projection's sums go.
// a: the token block blk of n_blocks; split: the share of the contraction.
template <bool GROUP>
__device__ __forceinline__ void skinny_tile(const SkinnyJob &job, const BlkInfo &a, const uint16_t *__restrict__ zero,
                                            const std::conditional_t<GROUP, GroupView, NoGroup> &gv, int blk, int n_blocks, int split, char *lds)
{
    const uint16_t *__restrict__ S = job.S, *__restrict__ at = job.at;
    float *__restrict__ part = job.part;
    const int C = job.C, mode = GROUP ? 0 : job.mode, stages_per_split = job.per, max_r16 = job.max_r16;
    const SegInfo g = a.g;
    const int t0 = a.t0;
    const int nt = (g.row1 - g.row0 - t0 < kSkinnyRows) ? g.row1 - g.row0 - t0 : kSkinnyRows;
    int r16 = g.r16;
    int p_r16[kMaxGroup];                              // GROUP: rows of each projection's block of the small matrix
    int64_t p_at[kMaxGroup];                           // ... and where the block starts in that projection's buffer
    if constexpr (GROUP) {
        r16 = 0;
#pragma unroll
        for (int p = 0; p < kMaxGroup; ++p) {
            p_r16[p] = 0; p_at[p] = 0;
            if (p < gv.n_proj) {
                const AdapterInfo ap = gv.mv[p].ad[g.adapter];
                p_r16[p] = ap.r16; p_at[p] = ap.at_off;
                r16 += ap.r16;
            }
        }
    }
    const int nb = r16 / 16;
    const int stage_bytes = SK_XT + max_r16 * SK_BK * 2;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t lds_base = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)LDS_PTR(char, lds));

    const int n_stage_all = (C + SK_BK - 1) / SK_BK;
    const int st0 = split * stages_per_split;
    int n_st = n_stage_all - st0;
    n_st = n_st < stages_per_split ? n_st : stages_per_split;
    if (n_st < 0) n_st = 0;

    const uint16_t *Bm = GROUP ? nullptr : (mode == 0) ? at + a.at_off : static_cast<const uint16_t *>(a.B);
    const int brows = (mode == 0) ? r16 : g.r;       // rows of the small matrix that exist

    // ---- loader: every load instruction moves 8 rows x 128 bytes; lane -> (row 8q + lane/8, slot
    // lane%8); slot c' of row u holds chunk c' ^ ((u >> 1) & 7).  Token tile: 16 instructions, wave w
    // issues w, w+4, w+8, w+12.  Small-matrix tile: r16/8 instructions, wave w issues w, w+4, ...
    const int lrow = lane >> 3;
    const uint16_t *xp[SK_XL];
    bool xok[SK_XL];
    int xchunk[SK_XL];
#pragma unroll
    for (int jj = 0; jj < SK_XL; ++jj) {
        const int u = (wave + SK_NW * jj) * 8 + lrow;
        xchunk[jj] = (lane & 7) ^ ((u >> 1) & 7);
        xok[jj] = u < nt;
        xp[jj] = S + (int64_t)(g.row0 + t0 + (xok[jj] ? u : 0)) * C + (int64_t)st0 * SK_BK + xchunk[jj] * 8;
    }
    const int nbi = r16 / 8;                                      // small-matrix load instructions per stage
    const int my_b = (nbi > wave) ? (nbi - wave + SK_NW - 1) / SK_NW : 0;     // ... of which this wave issues my_b
    const uint16_t *bp[SK_BL];
    bool bok[SK_BL];
    int bchunk[SK_BL];
#pragma unroll
    for (int jj = 0; jj < SK_BL; ++jj) {
        const int u = (wave + SK_NW * jj) * 8 + lrow;
        bchunk[jj] = (lane & 7) ^ ((u >> 1) & 7);
        bok[jj] = u < brows;
        if constexpr (GROUP) {
            // the 8 rows of an instruction lie in one projection's block (blocks are multiples of 16 rows)
            int first = 0, cum = 0;
            const uint16_t *base = gv.small[0] + p_at[0];
#pragma unroll
            for (int p = 1; p < kMaxGroup; ++p) {
                cum += p_r16[p - 1];
                if (p < gv.n_proj && u >= cum) { first = cum; base = gv.small[p] + p_at[p]; }
            }
            bp[jj] = base + (int64_t)(bok[jj] ? u - first : 0) * C + (int64_t)st0 * SK_BK + bchunk[jj] * 8;
        } else {
            bp[jj] = Bm + (int64_t)(bok[jj] ? u : 0) * C + (int64_t)st0 * SK_BK + bchunk[jj] * 8;
        }
    }
    const int lps = SK_XL + my_b;                                     // loads per stage issued by this wave

    auto load16 = [&](const uint16_t *gp, uint32_t dst) {
        asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(gp), "s"(dst));
    };
    const bool past = job.past != 0;
    auto load16_once = [&](const uint16_t *gp, uint32_t dst) {
        asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off nt" ::"v"(gp), "s"(dst));
    };
    const int turn = job.turn && n_st > 0 ? (int)(((unsigned)blk * 5u + (unsigned)split * 3u) % (unsigned)n_st) : 0;
    auto issue = [&](int st) {       // step of this split: stage st + turn, round the end; ring slot st % SK_NST
        const uint32_t base = lds_base + (st % SK_NST) * stage_bytes;
        const int sx = st + turn < n_st ? st + turn : st + turn - n_st;
        const int k0 = (st0 + sx) * SK_BK;
        if (past) {
#pragma unroll
            for (int jj = 0; jj < SK_XL; ++jj)
                load16_once(xok[jj] ? xp[jj] + (int64_t)sx * SK_BK : zero, base + (wave + SK_NW * jj) * 1024);
        } else {
#pragma unroll
            for (int jj = 0; jj < SK_XL; ++jj) {
                const bool ok = xok[jj] && (k0 + xchunk[jj] * 8 < C);
                load16(ok ? xp[jj] + (int64_t)sx * SK_BK : zero, base + (wave + SK_NW * jj) * 1024);
            }
        }
#pragma unroll
        for (int jj = 0; jj < SK_BL; ++jj) {
            if (jj < my_b) {
                const bool ok = bok[jj] && (k0 + bchunk[jj] * 8 < C);
                load16(ok ? bp[jj] + (int64_t)sx * SK_BK : zero, base + SK_XT + (wave + SK_NW * jj) * 1024);
            }
        }
    };

    // ---- MFMA operands: lane (lm, kg) reads row lm of its block, chunk 4*ks + kg
    const int lm = lane & 15, kg = lane >> 4;
    int xoff[SK_MB];
#pragma unroll
    for (int mb = 0; mb < SK_MB; ++mb) {
        const int u = (wave * SK_MB + mb) * 16 + lm;
        xoff[mb] = u * 128 + ((kg ^ ((u >> 1) & 7)) * 16);                  // ks*4 XORs in (bit 2 of the chunk)
    }
    int boff[SK_MAXNB];
#pragma unroll
    for (int b = 0; b < SK_MAXNB; ++b) {
        const int u = b * 16 + lm;
        boff[b] = SK_XT + u * 128 + ((kg ^ ((u >> 1) & 7)) * 16);
    }
    f32x4 acc[SK_MB][SK_MAXNB];
#pragma unroll
    for (int mb = 0; mb < SK_MB; ++mb)
#pragma unroll
        for (int b = 0; b < SK_MAXNB; ++b) acc[mb][b] = f32x4{0.f, 0.f, 0.f, 0.f};

    for (int p = 0; p < SK_NST - 1; ++p)
        if (p < n_st) issue(p);
    for (int st = 0; st < n_st; ++st) {
        const int ahead = (n_st - 1 - st < SK_NST - 2) ? n_st - 1 - st : SK_NST - 2;
        wait_vmcnt_dyn(ahead * lps);             // this wave's loads of stage st have landed ...
        __builtin_amdgcn_s_waitcnt(0xc07f);      // ... its LDS reads of the slot about to be refilled are done ...
        __builtin_amdgcn_sched_barrier(0);       // (nothing may be moved across the barrier)
        __builtin_amdgcn_s_barrier();            // ... and so are everyone else's; ring slot (st-1) is free
        __builtin_amdgcn_sched_barrier(0);
        if (st + SK_NST - 1 < n_st) issue(st + SK_NST - 1);
        const char *sb = lds + (st % SK_NST) * stage_bytes;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            bf16x8 xf[SK_MB];
#pragma unroll
            for (int mb = 0; mb < SK_MB; ++mb) xf[mb] = *LDS_PTR(const bf16x8, sb + (xoff[mb] ^ (ks * 64)));
#pragma unroll
            for (int b = 0; b < SK_MAXNB; ++b) {
                if (b < nb) {
                    const bf16x8 bf = *LDS_PTR(const bf16x8, sb + (boff[b] ^ (ks * 64)));
#pragma unroll
                    for (int mb = 0; mb < SK_MB; ++mb)
                        acc[mb][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf[mb], bf, acc[mb][b], 0, 0, 0);
                }
            }
        }
    }

    // partial tile [128][r16] of this (block, split): lane holds column 16b + lm, rows 16*(2w+mb) + 4kg + i
    float *dst = part + ((int64_t)split * n_blocks + blk) * (kSkinnyRows * max_r16);
#pragma unroll
    for (int mb = 0; mb < SK_MB; ++mb)
#pragma unroll
        for (int b = 0; b < SK_MAXNB; ++b)
            if (b < nb) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    dst[((wave * SK_MB + mb) * 16 + kg * 4 + i) * r16 + b * 16 + lm] = acc[mb][b][i];
            }
}

template <bool GROUP>
__global__ void __launch_bounds__(64 * SK_NW) k_skinny(SkinnyBatch batch, const uint16_t *__restrict__ zero,
                                               std::conditional_t<GROUP, GroupView, NoGroup> gv)
{
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    const SkinnyJob job = batch.j[GROUP ? 0 : blockIdx.z];
    if ((int)blockIdx.y >= job.n_split) return;
    const BlkInfo a = job.blk[blockIdx.x];
    skinny_tile<GROUP>(job, a, zero, gv, blockIdx.x, gridDim.x, blockIdx.y, lds);
}

// dH in the launch of the preparation: it reads B_k as it lies in memory and no table, a workgroup finds its token block in the
// description itself.  The tables come first (a long chain), then dH, and the short packing workgroups in what room it leaves: the other
// way round 8192 tokens, 4096 -> 4096 gained nothing, for dH then began its 512 workgroups behind 385 others (7 us of preparation saved, 0 to
// 8 of a step; backward_impl has the line).
__device__ __attribute__((aligned(16))) const uint32_t g_skinny_zeros[4] = {0u, 0u, 0u, 0u};     // the zero page is written in the same launch
__global__ void __launch_bounds__(64 * SK_NW) k_prep_dh(DescChunk c, PrepArgs pa, SkinnyJob job, int n_prep, int n_blocks)
{
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    const DescReader<WordsInArg> in{WordsInArg{c.w}};
    const int n_dh = (int)gridDim.x - n_prep, wg = (int)blockIdx.x - 1;      // the tables, then dH, then the rest of the preparation
    if (wg < 0 || wg >= n_dh) { prep_body(in, pa, wg < 0 ? 0 : wg - n_dh + 1, lds); return; }
    const int split = wg / n_blocks, blk = wg - split * n_blocks;
    BlkInfo a;
    a.g = segment_of_block(in, blk, a.t0, a.scale);
    a.at_off = 0; a.B = in.ad_ptr(a.g.adapter, 1);
    __builtin_amdgcn_s_waitcnt(0);                   // the compiler would wait in every stage for what the other branch has in flight
    skinny_tile<false>(job, a, reinterpret_cast<const uint16_t *>(g_skinny_zeros), NoGroup{0}, blk, n_blocks, split, lds);
}

// Sums the partial tiles of the splits (fixed order) and writes the outputs, 16 rows of a token block per workgroup.
// blockIdx.z: the job.  GROUP: the partial tiles are those of a fused pass (pitch = the fused rank of the segment's adapter) and the
// jobs are its projections; the columns of one start behind those of the projections before it.
template <bool GROUP>
__global__ void __launch_bounds__(256) k_skinny_finish(SkinnyBatch batch, std::conditional_t<GROUP, GroupView, NoGroup> gv)
{
    const int proj = blockIdx.z;
    const SkinnyJob job = batch.j[proj];
    const SkinnyOut out = job.out;
    const float *__restrict__ part = job.part;
    const int mode = job.mode, n_split = job.n_split, max_r16 = job.max_r16;
    constexpr int FR = 16;                            // token rows per workgroup (grid.y slices of a block)
    __shared__ float tile[FR * PLORA_MAX_RANK];       // [FR][r16], pitch r16
    const int blk = blockIdx.x;
    const BlkInfo bi = job.blk[blk];
    const SegInfo g = bi.g;
    const float mult = bi.scale;
    const int r0 = blockIdx.y * FR;                   // first row of this slice inside the block
    const int t0 = bi.t0 + r0;                        // first token of the slice inside the segment
    const int nt = g.row1 - g.row0 - t0;              // valid tokens from there on
    if (t0 >= g.lp) return;                           // slice lies past the padded segment: nothing to write
    const int r16 = g.r16;
    int pitch = r16, col0 = 0;
    const int64_t tile_elems = (int64_t)kSkinnyRows * max_r16;
    if constexpr (GROUP) {
        pitch = 0;
        for (int p = 0; p < gv.n_proj; ++p) {
            const int rp16 = gv.mv[p].ad[g.adapter].r16;
            if (p < proj) col0 += rp16;
            pitch += rp16;
        }
    }
    const int64_t split_stride = (int64_t)gridDim.x * tile_elems;
    const float *src = part + (int64_t)blk * tile_elems + (int64_t)r0 * pitch + col0;
    const int q = r16 / 4;                            // float4 per row of these columns
    for (int e = threadIdx.x; e < FR * q; e += 256) {
        const int row = e / q, c4 = e - row * q;
        const float *s0 = src + row * pitch + c4 * 4;
        float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int sp0 = 0; sp0 < n_split; sp0 += 8) {  // eight tiles requested at a time
            float4 v[8];
#pragma unroll
            for (int sp = 0; sp < 8; ++sp)
                if (sp0 + sp < n_split) v[sp] = *reinterpret_cast<const float4 *>(s0 + (sp0 + sp) * split_stride);
#pragma unroll
            for (int sp = 0; sp < 8; ++sp)
                if (sp0 + sp < n_split) { sum.x += v[sp].x; sum.y += v[sp].y; sum.z += v[sp].z; sum.w += v[sp].w; }
        }
        reinterpret_cast<float4 *>(tile)[e] = sum;
    }
    __syncthreads();
    write_outputs<FR>(g, mult, mode, tile, r16, t0, nt, out);
}

// Splits of the contraction over workgroups: three workgroups per compute unit, eight stages or more per split.  A short
// batch cannot fill the chip with eight splits, and one workgroup walks its stages at about 0.9 us each whatever the rest of
// the chip does, so up to 32 token blocks the contraction is cut further, to four stages: 512 tokens x 14336 columns, 28
// stages per split 24 us, 7 stages 9 us; 1024 tokens 26 -> 12.6 us.  (A function of the token blocks and the contraction alone; the workspace may
// allow fewer.)
int skinny_splits(const MetaHeader &h, int64_t C)
{
    if (h.n_blocks == 0) return 1;
    const int n_stage_all = (int)((C + SK_BK - 1) / SK_BK);
    const int want = (768 + h.n_blocks - 1) / h.n_blocks;
    int n = want < 8 ? want : 8;
    if (n > n_stage_all / 8) n = n_stage_all / 8;
    if (n < 1) n = 1;
    int fine = 256 / h.n_blocks;
    if (fine > kSkinnyMaxSplits) fine = kSkinnyMaxSplits;
    if (fine > n_stage_all / 4) fine = n_stage_all / 4;
    return fine > n ? fine : n;
}

// ---- short batches (skinny_short.h), with the tables in place: the projections of a grouped call ------------------------
struct ShortBatch { ShortJob j[kMaxGroup]; };
template <int NB>
__global__ void __launch_bounds__(64 * SH_NW, 4) k_skinny_short(ShortBatch batch)
{
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const ShortJob job = batch.j[blockIdx.z];
    if ((int)blockIdx.y >= job.n_split) return;
    const BlkInfo a = job.blk[blockIdx.x / kShortSlices];
    const uint16_t *small = job.mode == 0 ? job.small + a.at_off : static_cast<const uint16_t *>(a.B);
    skinny_short<NB>(job, a.g, a.scale, a.t0 + blockIdx.x % kShortSlices * 16, blockIdx.x, gridDim.x, blockIdx.y, small, false, lds);
}

// Which products are short.  k_skinny reads the small matrix once per 128 tokens, in a launch of its own with a finishing launch
// behind it.  The bounds, by whole steps with k_skinny and short, us:
//   - what the slices fetch of the small matrix and their own rows out of the L2s: 47 MiB (dH of 1852 tokens, 4096 columns, rank 32) 123 and
//     111, 54 MiB (1341 tokens, 4096 -> 512, rank 64) 83 and 77; above 64 MiB some gain and some lose: 72 MiB (2250 tokens, 1536 -> 8320,
//     rank 16) 191 and 179, 68 MiB (1209 tokens, 5120 -> 3072, rank 128) 163 and 173, 80 MiB (1301 tokens, 5120 -> 512, rank 64) 123 and
//     128, (1018 tokens, 14336 -> 8192, rank 64) 536 and 547
//   - A_k and B_k of all adapters, which come from memory and whose packing shares the launch.  Up to rank 64: 18 MB (1734 tokens,
//     4096 -> 512, 30 adapters) 108 and 97, 21 MB (187 tokens, 8192 -> 2048, 16 adapters) 114 and 111, 34 MB (450 tokens, 14336 -> 2048, 16
//     adapters) 217 and 226.  Above, where a wave has half a chunk in flight and its registers are those of the preparation: 8.6 MB (132
//     tokens, 2048 -> 1024, 24 adapters) 104 and 89, 10.1 MB (976 tokens, 3072 -> 4096, 16 adapters) 135 and 144, 25 MB (487 tokens,
//     4096 -> 4096, 16 adapters) 138 and 163, 67 MB (174 tokens, 8192 -> 1024, 30 adapters) 169 and 255
//   - above rank 64 at most two chunks for a wave: three or four (75 tokens, 14336 -> 1536, 4 adapters) 106 and 129
bool skinny_is_short(const MetaHeader &h, int slices16, int r16_total, int64_t C)
{
    if (h.n_blocks == 0 || h.n_blocks > kShortMaxBlocks) return false;
    if ((int64_t)slices16 * (16 + h.max_r16) * C * 2 > SH_MAX_BYTES) return false;
    const int most = std::max(8, std::max(skinny_splits(h, h.D), skinny_splits(h, h.K)));     // splits that the workspace has room for, uncut
    const int64_t small = (int64_t)r16_total * (h.D + h.K) * 2;
    if (h.max_r16 <= 64) return small <= SH_MAX_SMALL;
    return small <= SH_MAX_SMALL_8 && short_shares(h, slices16, C, most / 2).per <= 2 * SH_NW;
}

// Shares of the contraction: about two workgroups per compute unit (four where the rank makes a chunk long: 3000 tokens,
// 1024 -> 1024, rank 128 the step takes 95 and 92 us; 2048 tokens, 4096 -> 4096, rank 16 158 and 162), a chunk for every wave
// at least (one, two, four, eight chunks: 64 tokens, 2048 -> 2048 the step takes 41, 44, 47, 50 us, 300 tokens, 1024 -> 1024,
// rank 128 64, 73, 89, 89)
ShortShares short_shares(const MetaHeader &h, int slices16, int64_t C, int most)
{
    const int n_chunks = (int)((C + SH_BK - 1) / SH_BK);
    int n = (h.max_r16 > 64 ? 1024 : 512) / (slices16 > 0 ? slices16 : 1);
    if (n > n_chunks / SH_NW) n = n_chunks / SH_NW;
    if (n > most) n = most;
    if (n > kShortMaxSplits) n = kShortMaxSplits;
    if (n < 1) n = 1;
    const int per = (n_chunks + n - 1) / n;
    return ShortShares{(n_chunks + per - 1) / per, per};
}

ShortJob short_job(const SkinnyOperands &o)
{
    ShortJob j{};
    j.blk = o.mv.blk; j.S = static_cast<const uint16_t *>(o.S); j.small = static_cast<const uint16_t *>(o.at);
    j.part = o.part; j.flags = o.flags;
    j.out = SkinnyOut{o.hf, static_cast<uint16_t *>(o.hb), static_cast<uint16_t *>(o.zt), o.zt_scaled ? 1 : 0};
    j.C = (int32_t)o.C; j.mode = o.mode; j.max_r16 = o.h.max_r16;
    const ShortShares s = short_shares(o.h, o.slices16, o.C, o.n_split);
    j.n_split = s.n; j.per = s.per;
    j.number = launch_number();
    return j;
}

static hipError_t launch_short(const SkinnyOperands *ops, int n, hipStream_t st)
{
    ShortBatch batch{};
    int max_r16 = 0, grid_y = 0;
    for (int i = 0; i < n; ++i) {
        batch.j[i] = short_job(ops[i]);
        max_r16 = ops[i].h.max_r16 > max_r16 ? ops[i].h.max_r16 : max_r16;
        grid_y = batch.j[i].n_split > grid_y ? batch.j[i].n_split : grid_y;
    }
    const dim3 grid((unsigned)(ops[0].h.n_blocks * kShortSlices), (unsigned)grid_y, (unsigned)n);
    const size_t lds = short_lds_bytes(max_r16);
    const int nb = max_r16 / 16;
    if (nb <= 1) hipLaunchKernelGGL(k_skinny_short<1>, grid, dim3(64 * SH_NW), lds, st, batch);
    else if (nb <= 2) hipLaunchKernelGGL(k_skinny_short<2>, grid, dim3(64 * SH_NW), lds, st, batch);
    else if (nb <= 4) hipLaunchKernelGGL(k_skinny_short<4>, grid, dim3(64 * SH_NW), lds, st, batch);
    else hipLaunchKernelGGL(k_skinny_short<8>, grid, dim3(64 * SH_NW), lds, st, batch);
    return hipGetLastError();
}

static SkinnyJob skinny_job(const SkinnyOperands &o)
{
    SkinnyJob j{};
    j.blk = o.mv.blk; j.S = static_cast<const uint16_t *>(o.S); j.at = static_cast<const uint16_t *>(o.at);
    j.part = o.part;
    j.out = SkinnyOut{o.hf, static_cast<uint16_t *>(o.hb), static_cast<uint16_t *>(o.zt), o.zt_scaled ? 1 : 0};
    j.C = (int32_t)o.C; j.mode = o.mode; j.max_r16 = o.h.max_r16; j.n_split = o.n_split;
    set_past(j, o.h, o.alone, o.mean_r16);
    const int n_stage_all = (j.C + SK_BK - 1) / SK_BK;
    j.per = (n_stage_all + j.n_split - 1) / j.n_split;
    return j;
}

hipError_t launch_prep_dh(const PrepJob &p, hipStream_t st)
{
    const SkinnyOperands &o = *p.dh;
    if (o.mode != 1 || o.is_short || o.h.n_blocks == 0 || p.n_words > kChunkWords) return hipErrorInvalidValue;
    PrepArgs pa;
    int64_t n_wg;
    size_t lds;
    hipError_t e = prep_args(p, pa, n_wg, lds);
    if (e != hipSuccess) return e;
    SkinnyBatch batch{};
    batch.j[0] = skinny_job(o);
    DescChunk c;
    std::memcpy(c.w, p.desc_host, (size_t)p.n_words * 4);
    lds = std::max(lds, (size_t)SK_NST * (SK_XT + o.h.max_r16 * SK_BK * 2));
    e = allow_full_lds(reinterpret_cast<const void *>(k_prep_dh), 2);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_prep_dh, dim3((unsigned)(n_wg + (int64_t)o.h.n_blocks * o.n_split)), dim3(64 * SK_NW), lds, st, c, pa, batch.j[0], (int)n_wg, o.h.n_blocks);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_skinny_finish<false>, dim3((unsigned)o.h.n_blocks, kSkinnyRows / 16, 1), dim3(256), 0, st, batch, NoGroup{0});
    return hipGetLastError();
}

hipError_t launch_skinny_bf16(const SkinnyOperands *ops, int n, const void *zero, hipStream_t st)
{
    if (n < 0 || n > kMaxGroup) return hipErrorInvalidValue;
    SkinnyOperands brief[kMaxGroup];
    SkinnyBatch batch{};
    int n_brief = 0, m = 0, max_r16 = 0, grid_y = 0, n_blocks = 0;
    for (int i = 0; i < n; ++i) {
        const SkinnyOperands &o = ops[i];
        if (o.h.n_blocks == 0) continue;
        if (o.is_short) { brief[n_brief++] = o; continue; }
        batch.j[m++] = skinny_job(o);
        n_blocks = o.h.n_blocks;
        max_r16 = o.h.max_r16 > max_r16 ? o.h.max_r16 : max_r16;
        grid_y = o.n_split > grid_y ? o.n_split : grid_y;
    }
    if (n_brief > 0) {
        const hipError_t e = launch_short(brief, n_brief, st);
        if (e != hipSuccess) return e;
    }
    if (m == 0) return hipSuccess;
    const size_t lds = (size_t)SK_NST * (SK_XT + max_r16 * SK_BK * 2);
    hipError_t e = allow_full_lds(reinterpret_cast<const void *>(k_skinny<false>), 0);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_skinny<false>, dim3((unsigned)n_blocks, (unsigned)grid_y, (unsigned)m), dim3(64 * SK_NW), lds, st, batch,
                       static_cast<const uint16_t *>(zero), NoGroup{0});
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_skinny_finish<false>, dim3((unsigned)n_blocks, kSkinnyRows / 16, (unsigned)m), dim3(256), 0, st, batch, NoGroup{0});
    return hipGetLastError();
}

hipError_t launch_skinny_group(const GroupView &gv, const MetaHeader &hv, const void *x, int64_t C, const void *zero, float *part,
                               size_t part_bytes, int n_split, float *const *hf, void *const *hb, void *const *zt, hipStream_t st)
{
    if (hv.n_blocks == 0) return hipSuccess;
    if (gv.n_proj < 2 || gv.n_proj > kMaxGroup || gv.max_r16 > PLORA_MAX_RANK || hv.max_r16 != gv.max_r16) return hipErrorInvalidValue;
    if (n_split < 1 || (size_t)n_split * hv.n_blocks * kSkinnyRows * gv.max_r16 * 4 > part_bytes) return hipErrorInvalidValue;
    const int n_stage_all = (int)((C + SK_BK - 1) / SK_BK);
    SkinnyBatch batch{};
    for (int p = 0; p < gv.n_proj; ++p) {
        SkinnyJob &j = batch.j[p];
        j.blk = gv.mv[p].blk; j.S = static_cast<const uint16_t *>(x); j.part = part;
        j.out = SkinnyOut{hf[p], static_cast<uint16_t *>(hb[p]), static_cast<uint16_t *>(zt[p]), 0};
        j.C = (int32_t)C; j.mode = 0; j.per = (n_stage_all + n_split - 1) / n_split; j.n_split = n_split; j.max_r16 = gv.max_r16;
        set_past(j, hv, false, 0);
    }
    const size_t lds = (size_t)SK_NST * (SK_XT + gv.max_r16 * SK_BK * 2);
    hipError_t e = allow_full_lds(reinterpret_cast<const void *>(k_skinny<true>), 7);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_skinny<true>, dim3((unsigned)hv.n_blocks, (unsigned)n_split), dim3(64 * SK_NW), lds, st, batch,
                       static_cast<const uint16_t *>(zero), gv);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_skinny_finish<true>, dim3((unsigned)hv.n_blocks, kSkinnyRows / 16, (unsigned)gv.n_proj), dim3(256), 0, st, batch, gv);
    return hipGetLastError();
}

}  // namespace plora
