// Weight gradients of the packed multi-LoRA layer on bf16 inputs (gfx950): the two products that
// contract over the token axis (appendix C.2),
//   case 3   dA_k[c][j] =           sum_t x_t[c]  g_t[j]      (g carries scale_k)
//   case 1   dB_k[j][c] = scale_k * sum_t dy_t[c] h_t[j]
// summed over every segment of adapter k.  Each streams a big [T][C] matrix once (bound by HBM)
// against the small transposed bf16 factor zt[j][t] written by the skinny kernel.
//
// The token index is the slow index of the big matrix, so its MFMA operand needs a transpose; it
// is staged HBM -> LDS as it lies in memory (direct loads into a ring of stages that fills the LDS)
// and read with the transposing LDS load (ds_read_b64_tr_b16).  The rank stays whole in every tile;
// tiles are cut along the hidden dimension (128 columns per workgroup, one wave per 32
// columns) and a workgroup walks the tokens of one adapter, longest adapters first.  The MFMA code
// is specialised per number of 16-wide rank blocks so that every LDS read of a stage is in flight
// before the first MFMA.  Nothing in the loop may spill: a scratch reload waits on the same counter
// as the direct loads and would drain the ring.
// When that gives too few workgroups to fill the chip the token walk is split as well and
// the fp32 partial tiles are summed, in a fixed order, by a small finishing kernel; otherwise the
// result is written directly.  No atomics anywhere: the summation order is fixed.
#include "gemm_small.h"

#include <algorithm>
#include <type_traits>

namespace plora {

constexpr int TC_BC = kTokTileColumns;                 // columns of the big matrix per workgroup
constexpr int TC_BT = 64;                  // tokens per stage (TC_BT / 32 MFMA K steps)
constexpr int TC_MAX_NST = 8;              // LDS ring stages: as many as fit in the 160 KB of a compute unit, at most this
constexpr int TC_LDS_BYTES = 160 * 1024;
constexpr int TC_CB = 2;                                  // 16-column MFMA blocks per wave: a wave owns 32 columns
constexpr int TC_SL = TC_BT * 32 * 2 / 1024;              // big-matrix load instructions per wave per stage (4)
constexpr int TC_NB = PLORA_MAX_RANK / 16;
constexpr int TC_KS = TC_BT / 32;                         // MFMA K steps per stage
constexpr int TC_ZC = TC_BT / 8;                          // 16-byte chunks per small-factor row
constexpr int TC_ZR = 64 / TC_ZC;                         // small-factor rows per load instruction
constexpr int TC_ZSH = TC_ZC == 4 ? 2 : 1;                // rows that share a 256-byte LDS line: 4 or 2
static_assert(TC_BT == 32 || TC_BT == 64, "");

__device__ inline void tc_wait_vmcnt(int n)
{
#define W_(N) case N: __builtin_amdgcn_s_waitcnt(0x0f70 | (N & 15) | ((N >> 4) << 14)); break;
    switch (n) {
        W_(0) W_(1) W_(2) W_(3) W_(4) W_(5) W_(6) W_(7) W_(8) W_(9) W_(10) W_(11) W_(12) W_(13) W_(14) W_(15) W_(16)
        W_(17) W_(18) W_(19) W_(20) W_(21) W_(22) W_(23) W_(24) W_(25) W_(26) W_(27) W_(28) W_(29) W_(30) W_(31) W_(32)
        W_(33) W_(34) W_(35) W_(36) W_(37) W_(38) W_(39) W_(40) W_(41) W_(42) W_(43) W_(44) W_(45) W_(46) W_(47) W_(48)
    default: __builtin_amdgcn_s_waitcnt(0x0f70); break;    // never reached: at most (TC_MAX_NST - 2) * 6 loads stay in flight
    }
#undef W_
}

// One product of a launch: the big matrix [T][C], the small factor, and how the work is cut.
struct TokcPass {
    const TokJob *job;
    const int32_t *seg_list;
    const SegInfo *seg;
    const uint16_t *S, *zt;
    float *part;                  // fp32 partial tiles [split][r16_total][C]; null: the result is written directly
    int32_t C, tiles, n_split;    // tiles: of TC_BC columns
    int32_t r16_total, want_da;
    int32_t unit0, finish0;       // first workgroup along x of this product, in the main and in the finishing launch
    int32_t past;                 // S is read past the caches
};
struct TokcBatch { TokcPass p[kTokMaxPasses]; };

// grid (column tiles and token splits of every product of the batch; adapters).  dB and dA do not depend on each other, nor do
// those of the projections of a grouped call, and together they need fewer splits to fill the chip.  In two launches with a finishing launch each, and in one with one: 8192 tokens,
// 4096 -> 4096, four adapters of rank 8 to 64 47.6 and 34.1 us; 512 tokens, 4096 -> 14336 24.7 and 14.3; 1531 tokens, 1000 ->
// 2504, five adapters (no split) 22.1 and 12.1; 16384 tokens, 4096 -> 14336, eight adapters 143 and 122; dB of a grouped
// q / k / v call of 16384 tokens 60 and 46.
// GROUP (dA only): the small factor of adapter k is the transposed g of several projections that share x, one below
// the other (GroupView); the tables are projection 0's, `zt` is not used, every projection's dA_k gets its own columns.
template <bool GROUP>
__device__ __forceinline__ void tokc_tile(const TokcBatch &batch, int n_pass, const uint16_t *__restrict__ zero, int max_r16, int nst,
                                          const std::conditional_t<GROUP, GroupView, NoGroup> &gv, int bx, int by, char *lds)
{
    constexpr int TC_NW = TC_BC / 32, TC_S_BYTES = TC_BT * TC_BC * 2;     // one wave per 32 columns
    constexpr int CPRW = TC_BC / 8;                               // 16-byte chunks per row of the big-matrix tile
    constexpr int RPIW = 64 / CPRW;                               // rows per 1 KB load instruction
    // 16-byte chunk c of token row u is stored at slot c ^ swz(u); chosen so that the 8 rows (u..u+3 and
    // u+8..u+11) that one pass of a transposing read touches fall into 8 different 32-byte bank groups
    auto swz = [](int u) { return 2 * (u & 3) + 8 * ((u >> 3) & 1); };
    int pi = 0;
    for (int i = 1; i < n_pass; ++i)
        if (bx >= batch.p[i].unit0) pi = i;
    const TokcPass ps = batch.p[pi];
    const TokJob a = ps.job[by];                     // longest adapters first
    const int k = a.k;
    const bool want_da = GROUP || ps.want_da;
    const uint16_t *__restrict__ S = ps.S, *__restrict__ zt = ps.zt;
    float *__restrict__ part = ps.part;
    const int C = ps.C, n_split = ps.n_split, r16_total = ps.r16_total;
    const int unit = bx - ps.unit0, split = unit / ps.tiles;
    const int c0 = (unit - split * ps.tiles) * TC_BC;
    int r16 = a.r16;
    int p_r16[kMaxGroup];                            // GROUP: rank rows (padded to 16) of each projection
    if constexpr (GROUP) {
        r16 = 0;
#pragma unroll
        for (int p = 0; p < kMaxGroup; ++p) {
            p_r16[p] = p < gv.n_proj ? gv.mv[p].ad[k].r16 : 0;
            r16 += p_r16[p];
        }
    }
    const int nb = r16 / 16;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t lds_base = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)LDS_PTR(char, lds));
    const int stage_bytes = TC_S_BYTES + max_r16 * TC_BT * 2;

    // steps (TC_BT tokens each) of this adapter over its own segments, and the
    // slice of them that belongs to this split
    const int32_t *own = ps.seg_list + a.seg_list0;
    const int n_own = a.n_own, n_steps_all = a.n_steps;
    const int per = (n_steps_all + n_split - 1) / n_split;
    const int step0 = split * per;
    int n_steps = n_steps_all - step0;
    n_steps = n_steps < per ? n_steps : per;
    if (n_steps < 0) n_steps = 0;

    // cursor of the next stage to fetch: index into the adapter's segment list, token offset inside that
    // segment, and the fields of the segment that the loader needs (kept in registers so that the load
    // issue right behind the barrier does not wait for a metadata fetch)
    int cur_li = 0, cur_t = 0;
    for (int skip = step0; skip > 0 && cur_li < n_own;) {
        const int len = cur_li ? ps.seg[own[cur_li]].row1 - ps.seg[own[cur_li]].row0 : a.len;
        const int st_here = (len + TC_BT - 1) / TC_BT;
        if (skip >= st_here) { skip -= st_here; ++cur_li; }
        else { cur_t = skip * TC_BT; skip = 0; }
    }
    // GROUP: the 8 rows that small-factor load instruction q = wave + TC_NW jj covers lie in one projection: zp[jj], and
    // zfirst[jj] is the first of that projection's rows in the fused factor
    constexpr int ZL = (PLORA_MAX_RANK / TC_ZR + TC_NW - 1) / TC_NW;
    int zp[ZL], zfirst[ZL];
    if constexpr (GROUP) {
#pragma unroll
        for (int jj = 0; jj < ZL; ++jj) {
            const int u = (wave + TC_NW * jj) * TC_ZR;
            int cum = 0;
            zp[jj] = 0; zfirst[jj] = 0;
#pragma unroll
            for (int p = 1; p < kMaxGroup; ++p) {
                cum += p_r16[p - 1];
                if (p < gv.n_proj && u >= cum) { zp[jj] = p; zfirst[jj] = cum; }
            }
        }
    }
    int seg_row0 = 0, seg_len = 0, seg_lp = 0;
    int64_t seg_zt = 0;
    const uint16_t *seg_zp[ZL];                      // GROUP: start of the current segment's rows in projection zp[jj]'s buffer
    auto load_desc = [&]() {
        if (!GROUP && cur_li == 0) {                 // the first segment came with the job
            seg_row0 = a.row0; seg_len = a.len; seg_lp = a.lp; seg_zt = a.zt_off;
            return;
        }
        if (cur_li < n_own) {
            const int sidx = own[cur_li];
            const SegInfo g = ps.seg[sidx];
            seg_row0 = g.row0; seg_len = g.row1 - g.row0; seg_lp = g.lp; seg_zt = g.zt_off;
            if constexpr (GROUP) {
#pragma unroll
                for (int jj = 0; jj < ZL; ++jj) seg_zp[jj] = gv.small[zp[jj]] + gv.mv[zp[jj]].seg[sidx].zt_off;
            }
        }
    };
    load_desc();

    // ---- loader.  Big-matrix tile [TC_BT t][CPRW chunks]: instruction q covers token rows RPIW q ..,
    // lane -> (row RPIW q + lane / CPRW, slot lane % CPRW); wave w issues q = w, w + TC_NW, ...
    // Small-factor tile [r16 j][TC_ZC chunks]:
    // instruction q covers rows TC_ZR q.., lane -> (row TC_ZR q + lane/TC_ZC, slot lane%TC_ZC), slot c' of
    // row u holds chunk c' ^ ((u >> TC_ZSH) & (TC_ZC-1)); wave w issues q = w, w + TC_NW, ... below r16/TC_ZR.
    const int nzi = r16 / TC_ZR;
    const int my_z = (nzi > wave) ? (nzi - wave + TC_NW - 1) / TC_NW : 0;
    const int lps = TC_SL + my_z;
    auto load16 = [&](const uint16_t *gp, uint32_t dst) {
        asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(gp), "s"(dst));
    };
    // the big matrix with the non-temporal hint, as in k_skinny: 16384 tokens, 14336 and 4096 columns 157 -> 132 us (4.6 TB/s; 130
    // where dH had left the end of dy in the last cache), 32768 x 8192 twice 231 -> 206, 8192 x 4096 twice the same.  Not where
    // column tiles share lines (20000 x 11000 and 13000 210 -> 246), and not where the last cache holds the
    // matrices of the launch: the product that reads one next finds it there (dX of 1024 tokens 139 us, 134 without)
    const bool past = ps.past != 0;
    auto load16_once = [&](const uint16_t *gp, uint32_t dst) {
        asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off nt" ::"v"(gp), "s"(dst));
    };
    auto issue = [&](int slot) {
        const uint32_t base = lds_base + slot * stage_bytes;
        const int tbase = __builtin_amdgcn_readfirstlane(cur_t);
#pragma unroll
        for (int jj = 0; jj < TC_SL; ++jj) {
            const int q = wave + TC_NW * jj;
            const int u = q * RPIW + lane / CPRW;
            const int chunk = (lane % CPRW) ^ swz(u);
            int c = c0 + chunk * 8;
            c = c < C ? c : C - 8;                                  // columns past the end only feed outputs that are not stored
            const int t = tbase + u;
            const uint16_t *p = (t < seg_len) ? S + (int64_t)(seg_row0 + t) * C + c : zero;
            if (past) load16_once(p, base + q * 1024);
            else load16(p, base + q * 1024);
        }
#pragma unroll
        for (int jj = 0; jj < (PLORA_MAX_RANK / TC_ZR + TC_NW - 1) / TC_NW; ++jj) {
            if (jj < my_z) {
                const int q = wave + TC_NW * jj;
                const int u = q * TC_ZR + lane / TC_ZC;
                const int chunk = (lane % TC_ZC) ^ ((u >> TC_ZSH) & (TC_ZC - 1));
                if constexpr (GROUP) load16(seg_zp[jj] + (int64_t)(u - zfirst[jj]) * seg_lp + tbase + chunk * 8, base + TC_S_BYTES + q * 1024);
                else load16(zt + seg_zt + (int64_t)u * seg_lp + tbase + chunk * 8, base + TC_S_BYTES + q * 1024);
            }
        }
        cur_t = tbase + TC_BT;
        if (cur_t >= seg_len) { ++cur_li; cur_t = 0; load_desc(); }
    };

    // ---- MFMA operands.  Wave w owns columns 32w..32w+31 (two 16-column blocks) and every rank block.
    // Transposing read of the big-matrix operand: the 16 lanes of group kg fetch the 4(t) x 16(c) block
    // at tokens 32*ks + 8*kg (+4 for the second read), 8 bytes each; lane i then holds column i.
    const int i16 = lane & 15, kg = lane >> 4;
    int soff[TC_CB];
#pragma unroll
    for (int cb = 0; cb < TC_CB; ++cb) {
        const int u = kg * 8 + (i16 >> 2);                            // token row fetched by this lane (first read)
        const int cl = wave * (TC_CB * 16) + cb * 16 + (i16 & 3) * 4; // first column fetched by this lane
        soff[cb] = u * (TC_BC * 2) + ((((cl >> 3) ^ swz(u)) * 16) + (cl & 7) * 2);
    }
    // second read (token row u+4) and later K steps (u+32): (u&3) and (u>>3)&1 unchanged, plain adds
    // small-factor operand: rank row j = 16b + i16, chunk 4*ks + kg; the swizzle term only depends on
    // i16, so block b sits 16 rows behind block b-1 and K step ks flips one offset bit
    const int zoff0 = TC_S_BYTES + i16 * (TC_BT * 2) + ((kg ^ ((i16 >> TC_ZSH) & (TC_ZC - 1))) * 16);

    f32x4 acc[TC_CB][TC_NB];
#pragma unroll
    for (int cb = 0; cb < TC_CB; ++cb)
#pragma unroll
        for (int b = 0; b < TC_NB; ++b) acc[cb][b] = f32x4{0.f, 0.f, 0.f, 0.f};

    auto compute = [&](auto nbc, const char *sb) {
        constexpr int NBC = decltype(nbc)::value;
#pragma unroll
        for (int ks = 0; ks < TC_KS; ++ks) {
            bf16x8 sf[TC_CB], zf[NBC];
#pragma unroll
            for (int cb = 0; cb < TC_CB; ++cb) {
                const char *p = sb + soff[cb] + ks * 32 * (TC_BC * 2);
                bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(LDS_PTR(bf16x4, p));
                bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(LDS_PTR(bf16x4, p + 4 * (TC_BC * 2)));
                sf[cb] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            }
#pragma unroll
            for (int b = 0; b < NBC; ++b) zf[b] = *LDS_PTR(const bf16x8, sb + (zoff0 ^ (ks * 64)) + b * 16 * (TC_BT * 2));
#pragma unroll
            for (int b = 0; b < NBC; ++b)
#pragma unroll
                for (int cb = 0; cb < TC_CB; ++cb)
                    acc[cb][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(sf[cb], zf[b], acc[cb][b], 0, 0, 0);
        }
    };

    // ring of nst stages: stage `it` lives in slot it % nst; nst - 1 stages are in flight ahead of the reader
    for (int p = 0; p < nst - 1; ++p)
        if (p < n_steps) issue(p);
    int rd_slot = 0, wr_slot = nst - 1;
    for (int it = 0; it < n_steps; ++it) {
        const int ahead = (n_steps - 1 - it < nst - 2) ? n_steps - 1 - it : nst - 2;
        tc_wait_vmcnt(ahead * lps);
        __builtin_amdgcn_s_waitcnt(0xc07f);      // this wave's LDS reads of the slot about to be refilled are done
        __builtin_amdgcn_sched_barrier(0);       // (nothing may be moved across the barrier)
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        if (it + nst - 1 < n_steps) issue(wr_slot);
        const char *sb = lds + rd_slot * stage_bytes;
        rd_slot = (rd_slot + 1 == nst) ? 0 : rd_slot + 1;
        wr_slot = (wr_slot + 1 == nst) ? 0 : wr_slot + 1;
        // straight-line code for each possible number of rank blocks: every LDS read of the stage is
        // issued before the first MFMA, so their latencies overlap instead of adding up per block
        switch (nb) {
        case 1: compute(std::integral_constant<int, 1>{}, sb); break;
        case 2: compute(std::integral_constant<int, 2>{}, sb); break;
        case 3: compute(std::integral_constant<int, 3>{}, sb); break;
        case 4: compute(std::integral_constant<int, 4>{}, sb); break;
        case 5: compute(std::integral_constant<int, 5>{}, sb); break;
        case 6: compute(std::integral_constant<int, 6>{}, sb); break;
        case 7: compute(std::integral_constant<int, 7>{}, sb); break;
        default: compute(std::integral_constant<int, 8>{}, sb); break;
        }
    }

    // ---- epilogue.  Lane holds rank column j = 16b + i16 and big-matrix columns c = cbase + 4*kg + i.
    const float mult = want_da ? 1.f : a.scale;
    int r16_off = a.r16_off;
    if constexpr (GROUP) {
        r16_off = 0;                                  // rows of the fused factors of the adapters before this one
        for (int p = 0; p < gv.n_proj; ++p) r16_off += gv.mv[p].ad[k].r16_off;
    }
#pragma unroll
    for (int cb = 0; cb < TC_CB; ++cb) {
        const int c = c0 + wave * (TC_CB * 16) + cb * 16 + kg * 4;
#pragma unroll
        for (int b = 0; b < TC_NB; ++b) {
            const int j = b * 16 + i16;
            if (b < nb && c < C) {
                if (part) {
                    float4 v;
                    v.x = acc[cb][b][0]; v.y = acc[cb][b][1]; v.z = acc[cb][b][2]; v.w = acc[cb][b][3];
                    *reinterpret_cast<float4 *>(part + ((int64_t)split * r16_total + r16_off + j) * C + c) = v;
                } else if constexpr (GROUP) {
                    int pj = 0, first = 0, cum = 0;   // the projection that owns rank block b, and its first row
#pragma unroll
                    for (int p = 1; p < kMaxGroup; ++p) {
                        cum += p_r16[p - 1];
                        if (p < gv.n_proj && b * 16 >= cum) { pj = p; first = cum; }
                    }
                    const AdapterInfo ap = gv.mv[pj].ad[k];
                    const int jl = j - first;
                    if (jl < ap.r) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) ap.dA[(int64_t)(c + i) * ap.r + jl] = acc[cb][b][i];
                    }
                } else if (j < a.r) {
                    if (want_da) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) a.dA[(int64_t)(c + i) * a.r + j] = acc[cb][b][i];
                    } else {
                        float4 v;
                        v.x = mult * acc[cb][b][0]; v.y = mult * acc[cb][b][1];
                        v.z = mult * acc[cb][b][2]; v.w = mult * acc[cb][b][3];
                        *reinterpret_cast<float4 *>(a.dB + (int64_t)j * C + c) = v;
                    }
                }
            }
        }
    }
}

template <bool GROUP>
__global__ void __launch_bounds__(2 * TC_BC) __attribute__((amdgpu_waves_per_eu(2, 2))) k_tokc(TokcBatch batch, int n_pass,
                                             const uint16_t *__restrict__ zero, int max_r16, int nst,
                                             std::conditional_t<GROUP, GroupView, NoGroup> gv)
{
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    tokc_tile<GROUP>(batch, n_pass, zero, max_r16, nst, gv, blockIdx.x, blockIdx.y, lds);
}

// dB, dA and, in small tiles, dX of a call (of the first projection of a grouped one): the three need g and nothing of one another.  The
// product's workgroups come first, they are the longer ones; the token walks fill the compute units beside and behind them.  Either part
// takes two workgroups of a compute unit alone, so the larger LDS and the 208 registers cost neither anything.  Taken wherever dX runs in
// small tiles alone: of 46 steps none that takes it was slower.  Whole steps, us, apart and together: 1531 tokens, 1000 -> 2504 88.0 and
// 76.4; 1024 tokens, 1024 -> 1024 49.5 and 38.4; 700 tokens, 4224 -> 2712 101 and 90; 74 tokens, 2688 -> 20224 159 and 142; 24 groups 1.05 on
// average; 1024 tokens, 4096 -> 14336, where 512 tiles fill the chip by themselves, the same.
template <bool FWD, int BM, bool DEEP>
__global__ void __launch_bounds__(2 * TC_BC) __attribute__((amdgpu_waves_per_eu(2, 2))) k_grads(TokcBatch batch, int n_pass, int units, int max_r16, int nst,
                                             MetaView mv, GemmSmallArgs ga, int n_gemm)
{
    static_assert(2 * TC_BC == 256, "both parts have four waves");
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    int id = blockIdx.x;
    // the compiler lets the branches run into one another: without these waits it would wait for loads of one in every stage of the other
    __builtin_amdgcn_s_waitcnt(0);
    if (id < n_gemm) {
        gemm_small_tile<FWD, BM, DEEP, false, true>(mv, ga, id, lds);
        return;
    }
    __builtin_amdgcn_s_waitcnt(0);
    id -= n_gemm;
    const int by = id / units;
    tokc_tile<false>(batch, n_pass, ga.zero, max_r16, nst, NoGroup{0}, id - by * units, by, lds);
}

// Sums the partial tiles [split][r16 rows][C] of one matrix in split order, for 64 columns and all of its r rows (the first
// at row0): dB_k[j][c] scaled by scale_k straight from the sums, dA_k[c][j] through LDS, so that both leave in whole rows.
// 16 threads x 4 columns per row, all splits of a row requested at once.
constexpr int TF_COLS = 64;
template <bool WANT_DA>
__device__ inline void finish_matrix(const float *__restrict__ part, int64_t split_stride, int n_split, int row0, int r, int C, int c0,
                                     float scale, float *__restrict__ dst, float *lds)
{
    const int c = c0 + (threadIdx.x & 15) * 4, jt = threadIdx.x >> 4;
    const int pitch = r | 1;                         // LDS rows of one column: an odd pitch keeps the banks apart
    for (int j = jt; j < r; j += 16) {
        if (c < C) {
            const float *src = part + (int64_t)(row0 + j) * C + c;
            float4 v[kTokMaxSplits];
#pragma unroll
            for (int sp = 0; sp < kTokMaxSplits; ++sp)
                if (sp < n_split) v[sp] = *reinterpret_cast<const float4 *>(src + sp * split_stride);
            float4 sum = v[0];
#pragma unroll
            for (int sp = 1; sp < kTokMaxSplits; ++sp)
                if (sp < n_split) { sum.x += v[sp].x; sum.y += v[sp].y; sum.z += v[sp].z; sum.w += v[sp].w; }
            if (WANT_DA) {
                float *q = lds + (c - c0) * pitch + j;
                q[0] = sum.x; q[pitch] = sum.y; q[2 * pitch] = sum.z; q[3 * pitch] = sum.w;
            } else {
                sum.x *= scale; sum.y *= scale; sum.z *= scale; sum.w *= scale;
                *reinterpret_cast<float4 *>(dst + (int64_t)j * C + c) = sum;
            }
        }
    }
    if (WANT_DA) {
        __syncthreads();
        const int cols = C - c0 < TF_COLS ? C - c0 : TF_COLS;
        float *out = dst + (int64_t)c0 * r;
        for (int e = threadIdx.x; e < cols * r; e += 256) {
            const int cc = e / r;
            out[e] = lds[cc * pitch + e - cc * r];
        }
        __syncthreads();
    }
}

__device__ inline void tokc_finish(const TokcBatch &batch, int n_pass, int bx, int by, float *lds)
{
    int pi = 0;
    for (int i = 1; i < n_pass; ++i)
        if (bx >= batch.p[i].finish0) pi = i;
    const TokcPass ps = batch.p[pi];
    const TokJob a = ps.job[by];
    const int c0 = (bx - ps.finish0) * TF_COLS;
    const int64_t stride = (int64_t)ps.r16_total * ps.C;
    if (ps.want_da) finish_matrix<true>(ps.part, stride, ps.n_split, a.r16_off, a.r, ps.C, c0, 1.f, a.dA, lds);
    else finish_matrix<false>(ps.part, stride, ps.n_split, a.r16_off, a.r, ps.C, c0, a.scale, a.dB, lds);
}

// grid (64-column tiles of the products that were split; adapters)
__global__ void __launch_bounds__(256) k_tokc_finish(TokcBatch batch, int n_pass)
{
    extern __shared__ __attribute__((aligned(16))) float tf_lds[];
    tokc_finish(batch, n_pass, blockIdx.x, blockIdx.y, tf_lds);
}

// The same and the sums of a split dX: finish x n_adapters workgroups, then the product's.
__global__ void __launch_bounds__(256) k_grads_finish(TokcBatch batch, int n_pass, int finish, int n_adapters, const float *__restrict__ part,
                                                      uint16_t *__restrict__ C, int64_t n_vec, int n_split)
{
    extern __shared__ __attribute__((aligned(16))) float tf_lds[];
    const int id = (int)blockIdx.x - finish * n_adapters;
    if (id < 0) tokc_finish(batch, n_pass, blockIdx.x % finish, blockIdx.x / finish, tf_lds);
    else gemm_finish<false>(part, C, n_vec, n_split, (int64_t)id * 256 + threadIdx.x);
}

// The same for the partial tiles of a fused dA pass: the rows of adapter k's projections lie one below the other.
__global__ void __launch_bounds__(256) k_tokc_finish_group(GroupView gv, const float *__restrict__ part, int C, int n_split)
{
    extern __shared__ __attribute__((aligned(16))) float tf_lds[];
    const int k = blockIdx.y;
    int row = 0;
    for (int p = 0; p < gv.n_proj; ++p) row += gv.mv[p].ad[k].r16_off;
    for (int p = 0; p < gv.n_proj; ++p) {
        const AdapterInfo a = gv.mv[p].ad[k];
        finish_matrix<true>(part, (int64_t)gv.r16_total * C, n_split, row, a.r, C, blockIdx.x * TF_COLS, 1.f, a.dA, tf_lds);
        row += a.r16;
    }
}

// Token splits.  128-column tiles throughout: two workgroups then share a compute unit, which pays more than the wider rows of
// 256-column tiles (measured: dB 8-19 % faster at the wide layers, the rest within a few percent either way).  When the tiles
// alone give fewer than about two workgroups per compute unit the token walk is split as well; the split is capped so that a
// split keeps about four stages, and so that the fp32 partial tiles (written once, read once) stay below half of the bytes of
// the big matrix.  Short walks gain from it too: a stage takes about 1 us, the finishing launch 5 us, and both products of 768
// tokens, 1024 -> 1024 take 12 us in splits against 16 whole, 2048 tokens, 4096 -> 4096 16 against 34 (512 tokens, 4096 -> 14336
// the same 14).
// other: workgroups that the other product brings to the same launch.
static int tokc_plan(const MetaHeader &h, int64_t C, int n_active_adapters, int64_t other)
{
    if (n_active_adapters < 1) return 1;
    const int64_t wgs = (C + TC_BC - 1) / TC_BC * n_active_adapters + other;
    const int steps = (int)(h.T / TC_BT / n_active_adapters);
    int want = (int)((512 + wgs - 1) / wgs);
    int cap = steps / 4;
    const int64_t r16_sum = (int64_t)h.n_adapters * (h.max_r16 > 0 ? h.max_r16 : 16);   // upper bound of the partial rows
    const int cap_bytes = (int)(h.T / (8 * r16_sum));
    if (cap > cap_bytes) cap = cap_bytes;
    if (cap < 1) cap = 1;
    if (want > cap) want = cap;
    if (want > kTokMaxSplits) want = kTokMaxSplits;
    if (want < 1) want = 1;
    return want;
}

int tokc_splits(const MetaHeader &h, int64_t C, int64_t C_other, int n_active_adapters)
{
    return tokc_plan(h, C, n_active_adapters, (C_other + TC_BC - 1) / TC_BC * n_active_adapters);
}

// Ring depth: the share of the 160 KB of LDS that lets two workgroups sit on a compute unit, but two stages at least (a second
// workgroup on the compute unit pays more than a third stage: measured).
static void tokc_ring(int max_r16, int *nst, size_t *lds)
{
    const size_t stage = (size_t)TC_BT * TC_BC * 2 + (size_t)max_r16 * TC_BT * 2;
    size_t budget = (size_t)TC_LDS_BYTES / 2;
    if (budget < 2 * stage) budget = 2 * stage;
    const int n = (int)(budget / stage);
    *nst = n > TC_MAX_NST ? TC_MAX_NST : n;
    *lds = *nst * stage;
}

template <bool GROUP>
static hipError_t launch_tokc(TokcBatch &batch, int n_pass, int n_adapters, const void *zero, int max_r16,
                              const std::conditional_t<GROUP, GroupView, NoGroup> &gv, hipStream_t st)
{
    int nst;
    size_t lds;
    max_r16 = max_r16 > 0 ? max_r16 : 16;
    tokc_ring(max_r16, &nst, &lds);
    auto kern = k_tokc<GROUP>;
    const hipError_t e = allow_full_lds(reinterpret_cast<const void *>(kern), GROUP ? 8 : 1);
    if (e != hipSuccess) return e;
    int units = 0;
    for (int i = 0; i < n_pass; ++i) { batch.p[i].unit0 = units; units += batch.p[i].tiles * batch.p[i].n_split; }
    hipLaunchKernelGGL(kern, dim3((unsigned)units, (unsigned)n_adapters), dim3(2 * TC_BC), lds, st, batch, n_pass,
                       static_cast<const uint16_t *>(zero), max_r16, nst, gv);
    return hipGetLastError();
}

static TokcPass make_pass(const MetaView &mv, const void *S, int64_t C, const void *zt, float *part, int n_split, int r16_total, bool want_dA, int64_t bytes)
{
    TokcPass p{};
    p.past = bytes > kLastCacheBytes && rows_of_whole_lines(S, C);
    p.job = mv.job; p.seg_list = mv.seg_list; p.seg = mv.seg;
    p.S = static_cast<const uint16_t *>(S); p.zt = static_cast<const uint16_t *>(zt);
    p.part = n_split > 1 ? part : nullptr;
    p.C = (int32_t)C; p.tiles = (int32_t)((C + TC_BC - 1) / TC_BC); p.n_split = n_split;
    p.r16_total = r16_total; p.want_da = want_dA ? 1 : 0;
    return p;
}

hipError_t launch_tokc_group_dA(const GroupView &gv, const MetaHeader &hv, const void *x, int64_t C, const void *zero,
                                float *part, size_t part_bytes, int n_split, int n_active_adapters, hipStream_t st)
{
    if (hv.n_adapters == 0) return hipSuccess;
    if (gv.n_proj < 2 || gv.n_proj > kMaxGroup || gv.max_r16 > PLORA_MAX_RANK || hv.max_r16 != gv.max_r16) return hipErrorInvalidValue;
    if (tokc_splits(hv, C, 0, n_active_adapters) != n_split) return hipErrorInvalidValue;
    if (n_split > 1 && (size_t)n_split * gv.r16_total * C * 4 > part_bytes) return hipErrorInvalidValue;
    TokcBatch batch{};
    batch.p[0] = make_pass(gv.mv[0], x, C, nullptr, part, n_split, gv.r16_total, true, hv.T * C * 2);
    const hipError_t e = launch_tokc<true>(batch, 1, hv.n_adapters, zero, gv.max_r16, gv, st);
    if (e != hipSuccess || n_split <= 1) return e;
    hipLaunchKernelGGL(k_tokc_finish_group, dim3((unsigned)((C + TF_COLS - 1) / TF_COLS), (unsigned)hv.n_adapters), dim3(256),
                       TF_COLS * (PLORA_MAX_RANK + 1) * 4, st, gv, part, (int)C, n_split);
    return hipGetLastError();
}

template <bool FWD, int BM, bool DEEP>
static hipError_t launch_grads_and_dx(TokcBatch &batch, int n_pass, int n_adapters, int max_r16, const GradsDx &g, hipStream_t st)
{
    constexpr size_t ring = (size_t)(gs_ring_x(BM) * BM + gs_ring_w(BM, DEEP) * GS_BN) * GS_BK * 2;
    int nst;
    size_t lds;
    max_r16 = max_r16 > 0 ? max_r16 : 16;
    tokc_ring(max_r16, &nst, &lds);
    auto kern = k_grads<FWD, BM, DEEP>;
    const hipError_t e = allow_full_lds(reinterpret_cast<const void *>(kern), 48 + (FWD ? 3 : 0) + (BM == 64 ? 0 : DEEP ? 1 : 2));
    if (e != hipSuccess) return e;
    int units = 0;
    for (int i = 0; i < n_pass; ++i) { batch.p[i].unit0 = units; units += batch.p[i].tiles * batch.p[i].n_split; }
    GemmSmallArgs ga{static_cast<const uint16_t *>(g.S), static_cast<const uint16_t *>(g.W), static_cast<const uint16_t *>(g.side),
                     static_cast<const uint16_t *>(g.ap), static_cast<const uint16_t *>(g.zero), static_cast<uint16_t *>(g.C),
                     g.plan.n_split > 1 ? g.part : nullptr, (int)((g.h.T + BM - 1) / BM), (int)((g.N + GS_BN - 1) / GS_BN), g.plan.n_split, 0,
                     (int)g.h.T, (int)g.Kd, (int)g.N, (int)g.h.n_seg};
    const int n_gemm = ga.tiles_m * ga.tiles_n * ga.n_split;
    hipLaunchKernelGGL(kern, dim3((unsigned)(n_gemm + units * n_adapters)), dim3(2 * TC_BC), std::max(lds, ring), st, batch, n_pass, units, max_r16, nst,
                       g.mv, ga, n_gemm);
    return hipGetLastError();
}

hipError_t launch_tokcontract_bf16(const TokcOperands *ops, int n, int n_adapters, const void *zero, const GradsDx *dx, hipStream_t st)
{
    if (n_adapters == 0 || n == 0) return hipSuccess;
    if (n < 0 || n > kTokMaxPasses) return hipErrorInvalidValue;
    TokcBatch batch{};
    int finish = 0, max_r16 = 0;
    bool finish_dA = false;
    int64_t bytes = 0;
    for (int i = 0; i < n; ++i) bytes += ops[i].T * ops[i].C * 2;
    for (int i = 0; i < n; ++i) {
        const TokcOperands &o = ops[i];
        batch.p[i] = make_pass(o.mv, o.S, o.C, o.zt, o.part, o.n_split, o.r16_total, o.want_dA, bytes);
        batch.p[i].finish0 = finish;
        if (o.n_split > 1) { finish += (int)((o.C + TF_COLS - 1) / TF_COLS); finish_dA = finish_dA || o.want_dA; }
        max_r16 = o.max_r16 > max_r16 ? o.max_r16 : max_r16;
    }
    hipError_t e;
    if (dx) {
        const bool deep = gemm_small_deep(dx->h.T);
#define PL_GD(FWD_, BM_, DEEP_) launch_grads_and_dx<FWD_, BM_, DEEP_>(batch, n, n_adapters, max_r16, *dx, st)
        if (dx->w_rows_contract) e = dx->plan.bm == 64 ? PL_GD(true, 64, false) : deep ? PL_GD(true, 128, true) : PL_GD(true, 128, false);
        else e = dx->plan.bm == 64 ? PL_GD(false, 64, false) : deep ? PL_GD(false, 128, true) : PL_GD(false, 128, false);
#undef PL_GD
        if (e != hipSuccess) return e;
        if (finish == 0) return dx->plan.n_split > 1 ? launch_gemm_finish(dx->part, dx->C, dx->h.T * dx->N, dx->plan.n_split, false, st) : hipSuccess;
    } else {
        e = launch_tokc<false>(batch, n, n_adapters, zero, max_r16, NoGroup{0}, st);
        if (e != hipSuccess || finish == 0) return e;
    }
    // k_tokc_finish looks for the last product that starts at or before its workgroup: those without a split are left out
    int m = 0;
    for (int i = 0; i < n; ++i)
        if (batch.p[i].n_split > 1) batch.p[m++] = batch.p[i];
    const size_t lds = finish_dA ? TF_COLS * (PLORA_MAX_RANK + 1) * 4 : 0;
    if (dx && dx->plan.n_split > 1) {
        const int64_t n_vec = dx->h.T * dx->N / 4;
        hipLaunchKernelGGL(k_grads_finish, dim3((unsigned)(finish * n_adapters + (n_vec + 255) / 256)), dim3(256), lds, st, batch, m, finish, n_adapters,
                           dx->part, static_cast<uint16_t *>(dx->C), n_vec, dx->plan.n_split);
    } else {
        hipLaunchKernelGGL(k_tokc_finish, dim3((unsigned)finish, (unsigned)n_adapters), dim3(256), lds, st, batch, m);
    }
    return hipGetLastError();
}

}  // namespace plora
