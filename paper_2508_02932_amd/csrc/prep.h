// The preparation kernels' device code (see small_kernels.hip, which launches them): derivation of the metadata tables from the
// compact description, packing of the adapter matrices, transposed copy of a saved activation.
#pragma once
#include "plora_internal.h"
#include "skinny_short.h"

namespace plora {

// ---- what the workgroups of the preparation kernel read of the description -------------------------
// Offsets are prefix sums over adapters or segments.  Every lane of a wave takes one entry and the wave sums or scans them
// in registers: one trip to memory instead of one per entry (a loop over 32 adapters and 32 segments on one thread was
// 25 us of every call).
__device__ inline int wave_scan(int v)                    // inclusive; lane moves inside the vector ALU (DPP)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);       // row_shr 1, 2, 4, 8 within 16 lanes
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);       // last lane of a row into the next row
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);       // lane 31 into the upper half
    return v;
}

__device__ inline int wave_sum(int v) { return __builtin_amdgcn_readlane(wave_scan(v), 63); }

__device__ inline int64_t wave_scan(int64_t v)
{
    // three 22-bit digits: 64 of them sum to 28 bits, so each digit is scanned in 32 bits (v < 2^63)
    const int64_t a = wave_scan((int)(v & 0x3fffff)), b = wave_scan((int)((v >> 22) & 0x3fffff)), c = wave_scan((int)(v >> 44));
    return a + (b << 22) + (c << 44);
}

// Sum over the adapters before k of their ranks, each padded to a multiple of `pad`.
template <class Src> __device__ inline int64_t rank_rows_before(const DescReader<Src> &in, int k, int pad)
{
    if (k == 0) return 0;
    const int lane = threadIdx.x & 63;
    int v = 0;
    for (int j = lane; j < k; j += 64) v += pad_to(in.ad_rank(j), pad);
    return wave_sum(v);
}

// ---- packing of A_k ------------------------------------------------------------------------------
// at: A_k^T as [r16][D] (rows j >= r are zero) - the "row = output column, contraction contiguous"
//     operand of the shrink kernel.
// ap: A_k as [D][rp] with columns j >= r zero - the low-rank K-extension operand of the dX GEMM.
// One block handles 64 rows i of one adapter; the tile goes through LDS so that both the reads of
// A_k (contiguous in j) and the writes of A_k^T (contiguous in i) are coalesced, 16 bytes per thread.
struct PackJob {
    const uint16_t *A;
    int r, rp, r16;
    int64_t at_off, ap_off;
};

__device__ inline void pack_block(const PackJob &a, int64_t D, int bx, uint16_t *at, uint16_t *ap, int want_at,
                                  int want_ap, uint16_t *tile)
{
    // The 64 rows of A_k handled here are one contiguous slab of 64 r elements: copy it to LDS as it is
    // (16 bytes per thread and step), then write both layouts from there.
    const int64_t i0 = (int64_t)bx * 64;
    const int r = a.r;
    const int rows = (int)((D - i0 < 64) ? D - i0 : 64);                 // a multiple of 8
    const uint4 *src = reinterpret_cast<const uint4 *>(a.A + i0 * r);
    const int n_vec = rows * r / 8;                                      // rows * r * 2 bytes is a multiple of 16
    for (int v = threadIdx.x; v < n_vec; v += 256) reinterpret_cast<uint4 *>(tile)[v] = src[v];
    __syncthreads();
    if (want_at) {
        // A_k^T rows j: 64 consecutive elements each, 8 per thread
        uint16_t *dst = at + a.at_off + i0;
        const int ii0 = (threadIdx.x & 7) * 8;
        if (ii0 < rows)
            for (int j = threadIdx.x >> 3; j < a.r16; j += 32) {
                union { uint4 q; uint16_t h[8]; } u;
                u.q = make_uint4(0u, 0u, 0u, 0u);
                if (j < r) {
#pragma unroll
                    for (int t = 0; t < 8; ++t) u.h[t] = tile[(ii0 + t) * r + j];
                }
                *reinterpret_cast<uint4 *>(dst + (int64_t)j * D + ii0) = u.q;
            }
    }
    if (want_ap) {
        // padded A_k: rows of rp elements, 8 elements (16 bytes) per thread and step
        uint16_t *dst = ap + a.ap_off + i0 * a.rp;
        const int vec_per_row = a.rp / 8, lanes_per_row = 8;         // rp is a multiple of 64
        const int ii0 = threadIdx.x / lanes_per_row, l = threadIdx.x % lanes_per_row;
        for (int ii = ii0; ii < rows; ii += 256 / lanes_per_row)
            for (int v = l; v < vec_per_row; v += lanes_per_row) {
                union { uint4 q; uint16_t h[8]; } u;
                if ((r & 7) == 0) {
                    u.q = v * 8 < r ? *reinterpret_cast<const uint4 *>(tile + ii * r + v * 8) : make_uint4(0u, 0u, 0u, 0u);
                } else {
#pragma unroll
                    for (int t = 0; t < 8; ++t) { const int j = v * 8 + t; u.h[t] = (j < r) ? tile[ii * r + j] : (uint16_t)0; }
                }
                reinterpret_cast<uint4 *>(dst + (int64_t)ii * a.rp)[v] = u.q;
            }
    }
}

// ---- packing of B_k when W is stored [d_out][d_in] -------------------------------------------------
// bp: B_k^T as [K][rp] with columns j >= r zero - the low-rank K-extension operand of the forward GEMM,
//     which then reads W (and with it this operand) with the contraction index contiguous.
// One block handles 64 columns n of one adapter: rows of B_k come in as 128-byte pieces, go through
// LDS, and leave as whole rows of rp elements.
struct PackBJob {
    const uint16_t *B;
    int r, rp;
    int64_t bp_off;
};

__device__ inline void pack_bt_block(const PackBJob &a, int64_t K, int bx, uint16_t *bp, uint16_t *tile)
{
    const int64_t n0 = (int64_t)bx * 64;
    const int cols = (int)((K - n0 < 64) ? K - n0 : 64);               // a multiple of 8
    const int l = threadIdx.x & 7;
    for (int j = threadIdx.x >> 3; j < a.r; j += 32) {
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (l * 8 < cols) v = *reinterpret_cast<const uint4 *>(a.B + (int64_t)j * K + n0 + l * 8);
        reinterpret_cast<uint4 *>(tile + j * 64)[l] = v;
    }
    __syncthreads();
    uint16_t *dst = bp + a.bp_off + n0 * a.rp;
    const int vec_per_row = a.rp / 8;                                   // rp is a multiple of 64
    for (int e = threadIdx.x; e < cols * vec_per_row; e += 256) {
        const int nn = e / vec_per_row, v = e % vec_per_row;
        union { uint4 q; uint16_t h[8]; } u;
#pragma unroll
        for (int t = 0; t < 8; ++t) { const int j = v * 8 + t; u.h[t] = (j < a.r) ? tile[j * 64 + nn] : (uint16_t)0; }
        reinterpret_cast<uint4 *>(dst + (int64_t)nn * a.rp)[v] = u.q;
    }
}

// ---- transposed bf16 copy of a saved fp32 activation ------------------------------------------------
// zt[j][t] = bf16(h[t][j]); rows j >= r and the padding tokens are written as zero.  One workgroup per
// (token block of kSkinnyRows rows, half of it): 64 tokens, so that every row of zt is written in whole 128-byte pieces.
struct TransposeJob {
    int len, r, r16, lp, t_block;    // segment length and rank; first token of the block inside the segment
    int64_t h_off, zt_off;
};
constexpr int kTrRows = 64;
typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x4_a16 __attribute__((ext_vector_type(4)));

__device__ inline void h_to_zt_slice(const TransposeJob &g, int slice, const float *hf, uint16_t *zt, float *tile)
{
    const int t0 = g.t_block + slice * kTrRows;     // first token of the slice inside the segment
    if (t0 >= g.lp) return;
    int nt = g.len - t0;
    nt = nt < 0 ? 0 : (nt < kTrRows ? nt : kTrRows);
    // the nt rows of r floats are contiguous: flat copy, then transposed reads
    const float *src = hf + g.h_off + (int64_t)t0 * g.r;
    const int n = nt * g.r;
    for (int e = threadIdx.x * 4; e + 4 <= n; e += 1024)
        *reinterpret_cast<f32x4_a16 *>(tile + e) = *reinterpret_cast<const f32x4_a4 *>(src + e);
    if ((int)threadIdx.x < (n & 3)) tile[(n & ~3) + threadIdx.x] = src[(n & ~3) + threadIdx.x];
    __syncthreads();
    const int tt = (threadIdx.x & 7) * 8;
    uint16_t *dst = zt + g.zt_off + t0 + tt;
    for (int j = threadIdx.x >> 3; j < g.r16; j += 32) {
        union { uint4 q; uint16_t h[8]; } u;
#pragma unroll
        for (int t = 0; t < 8; ++t) u.h[t] = (j < g.r && tt + t < nt) ? bf16_rne(tile[(tt + t) * g.r + j]) : (uint16_t)0;
        *reinterpret_cast<uint4 *>(dst + (int64_t)j * g.lp) = u.q;
    }
}

// ---- derivation of the metadata tables by one workgroup of 256 threads --------------------------------
// LDS of that workgroup.  The sizes that depend on the description come behind it: the description's words, then per
// segment the offsets h_off, hb_off and zt_off, then the first token block.
struct DeriveShared {
    int64_t at_off[PLORA_MAX_ADAPTERS], ap_off[PLORA_MAX_ADAPTERS];
    int32_t tokens[PLORA_MAX_ADAPTERS], n_own[PLORA_MAX_ADAPTERS], list0[PLORA_MAX_ADAPTERS], by_tokens[PLORA_MAX_ADAPTERS];
    int32_t r16_off[PLORA_MAX_ADAPTERS], rp_off[PLORA_MAX_ADAPTERS], n_steps[PLORA_MAX_ADAPTERS], first_seg[PLORA_MAX_ADAPTERS];
    int64_t wave_tot[4][4];
    int32_t totals[kSortKeys], base[kSortKeys], wave_cnt[4][kSortKeys], max_r16;
};
inline size_t derive_lds_bytes(int n_words, int n_seg)
{
    return align_up(sizeof(DeriveShared) + align_up((size_t)n_words * 4, 8) + (size_t)n_seg * 28, 16);
}

// Exclusive prefix sums of four values per thread over the workgroup; tot receives the sums.
__device__ inline void block_scan4(int64_t v[4], int64_t tot[4], int64_t (*wave_tot)[4])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int64_t inc[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) inc[i] = wave_scan(v[i]);
    if (lane == 63) {
#pragma unroll
        for (int i = 0; i < 4; ++i) wave_tot[wave][i] = inc[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        int64_t before = 0;
        tot[i] = 0;
        for (int w = 0; w < 4; ++w) {
            if (w < wave) before += wave_tot[w][i];
            tot[i] += wave_tot[w][i];
        }
        v[i] = before + inc[i] - v[i];
    }
    __syncthreads();
}

template <class Src> __device__ __forceinline__ void derive_on_device(const DescReader<Src> &src, char *meta_dst, char *shared_mem)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    DeriveShared &sh = *reinterpret_cast<DeriveShared *>(shared_mem);
    uint32_t *words = reinterpret_cast<uint32_t *>(shared_mem + sizeof(DeriveShared));
    const int n_seg = src.n_seg(), n_ad = src.n_adapters(), n_words = desc_words(n_seg, n_ad);
    int64_t *seg_hb = reinterpret_cast<int64_t *>(shared_mem + sizeof(DeriveShared) + align_up((size_t)n_words * 4, 8));
    int64_t *seg_h = seg_hb + n_seg, *seg_zt = seg_h + n_seg;
    int32_t *seg_blk0 = reinterpret_cast<int32_t *>(seg_zt + n_seg);
    for (int i = tid; i < n_words; i += 256) words[i] = src.src.word(i);
    sh.tokens[tid] = 0; sh.n_own[tid] = 0; sh.n_steps[tid] = 0; sh.first_seg[tid] = n_seg;
    if (tid < kSortKeys) sh.totals[tid] = 0;
    if (tid == 0) sh.max_r16 = 0;
    __syncthreads();
    const DescReader<WordsInMemory> in{WordsInMemory{words}};
    const int64_t T = in.T(), D = in.D(), K = in.K(), ap_rows = in.w_out_in() ? K : D;
    const TableLayout lay = table_layout(T, n_seg, n_ad, in.n_blocks(), in.records() != 0);
    const Tables t = tables_at(meta_dst, lay);
    const int64_t n_tiles = lay.n_tiles;
    const int n_blocks = in.n_blocks();

    // segments: 256 at a time, running sums carried along
    int64_t carry[4] = {0, 0, 0, 0};                 // token blocks, h, hb, zt
    for (int s0 = 0; s0 < n_seg; s0 += 256) {
        const int s = s0 + tid;
        SegInfo g;
        int64_t v[4] = {0, 0, 0, 0}, tot[4];
        if (s < n_seg) {
            g.row0 = in.seg_row0(s); g.row1 = in.seg_row1(s); g.adapter = in.seg_adapter(s);
            const int len = g.row1 - g.row0;
            g.r = g.adapter >= 0 ? in.ad_rank(g.adapter) : 0;
            g.rp = pad_to(g.r, kRankPadGemm); g.r16 = pad_to(g.r, kRankPadMfma); g.lp = pad_to(len, kTokPad);
            if (g.adapter >= 0) {
                v[0] = (len + kSkinnyRows - 1) / kSkinnyRows;
                v[1] = (int64_t)len * g.r; v[2] = (int64_t)len * g.rp; v[3] = (int64_t)g.r16 * g.lp;
                if (len > 0) {
                    atomicMax(&sh.max_r16, g.r16);
                    atomicAdd(&sh.tokens[g.adapter], len);
                    atomicAdd(&sh.n_own[g.adapter], 1);
                    atomicAdd(&sh.n_steps[g.adapter], g.lp / kTokPad);
                    atomicMin(&sh.first_seg[g.adapter], s);
                }
            }
        }
        block_scan4(v, tot, sh.wave_tot);
        if (s < n_seg) {
            g.blk0 = (int32_t)(carry[0] + v[0]);
            g.h_off = carry[1] + v[1]; g.hb_off = carry[2] + v[2]; g.zt_off = carry[3] + v[3];
            seg_h[s] = g.h_off; seg_hb[s] = g.hb_off; seg_zt[s] = g.zt_off; seg_blk0[s] = g.blk0;
            t.seg[s] = g;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) carry[i] += tot[i];
    }
    // adapters: one per thread.  (The scan's barriers also publish the counts and the segments' LDS records.)
    {
        const int k = tid;
        AdapterInfo a;
        int64_t v[4] = {0, 0, 0, 0}, tot[4];
        __syncthreads();
        if (k < n_ad) {
            a.A = in.ad_ptr(k, 0); a.B = in.ad_ptr(k, 1);
            a.dA = static_cast<float *>(const_cast<void *>(in.ad_ptr(k, 2)));
            a.dB = static_cast<float *>(const_cast<void *>(in.ad_ptr(k, 3)));
            a.r = in.ad_rank(k); a.rp = pad_to(a.r, kRankPadGemm); a.r16 = pad_to(a.r, kRankPadMfma);
            a.scale = in.ad_scale(k);
            a.n_own = sh.n_own[k]; a.tokens = sh.tokens[k]; a.reserved = 0;
            v[0] = (int64_t)a.r16 * D; v[1] = a.rp; v[2] = a.r16; v[3] = a.n_own;
        }
        block_scan4(v, tot, sh.wave_tot);
        if (k < n_ad) {
            a.at_off = v[0]; a.ap_off = v[1] * ap_rows; sh.rp_off[k] = (int32_t)v[1]; a.r16_off = (int32_t)v[2]; a.seg_list0 = (int32_t)v[3];
            a.ext_b = in.ext_b(k, a.at_off);
            sh.at_off[k] = a.at_off; sh.ap_off[k] = a.ap_off; sh.list0[k] = a.seg_list0; sh.r16_off[k] = a.r16_off;
            // place of this adapter in the order by token count, longest first, ties by index
            int rank = 0;
            for (int j = 0; j < n_ad; ++j) rank += sh.tokens[j] > a.tokens || (sh.tokens[j] == a.tokens && j < k);
            sh.by_tokens[rank] = k;
        }
        __syncthreads();
        if (k < n_ad) {
            a.by_tokens = sh.by_tokens[k];
            t.ad[k] = a;
        }
        if (k < n_ad && in.records()) {
            const int kj = a.by_tokens, s = sh.first_seg[kj];          // entry k of the jobs is adapter kj
            TokJob j;
            j.dA = static_cast<float *>(const_cast<void *>(in.ad_ptr(kj, 2)));
            j.dB = static_cast<float *>(const_cast<void *>(in.ad_ptr(kj, 3)));
            j.zt_off = 0; j.row0 = 0; j.len = 0; j.lp = 0;
            if (s < n_seg) { j.zt_off = seg_zt[s]; j.row0 = in.seg_row0(s); j.len = in.seg_row1(s) - j.row0; j.lp = pad_to(j.len, kTokPad); }
            j.k = kj; j.r = in.ad_rank(kj); j.r16 = pad_to(j.r, kRankPadMfma); j.r16_off = sh.r16_off[kj];
            j.scale = in.ad_scale(kj); j.seg_list0 = sh.list0[kj]; j.n_own = sh.n_own[kj]; j.n_steps = sh.n_steps[kj]; j.reserved = 0;
            t.job[k] = j;
        }
    }
    if (tid == 0) {
        MetaHeader hd;
        hd.T = T; hd.D = D; hd.K = K;
        hd.n_seg = n_seg; hd.n_adapters = n_ad; hd.n_blocks = n_blocks; hd.max_r16 = sh.max_r16;
        hd.w_out_in = in.w_out_in(); hd.reserved = 0; hd.at_base = in.at_base();
        *t.hdr = hd;
    }
    // per-adapter lists of non-empty segments: a segment's place is the number of earlier ones of its adapter
    for (int s = tid; s < n_seg; s += 256) {
        const int k = in.seg_adapter(s);
        if (k < 0 || in.seg_row1(s) <= in.seg_row0(s)) continue;
        int place = sh.list0[k];
        for (int q = 0; q < s; ++q) place += in.seg_adapter(q) == k && in.seg_row1(q) > in.seg_row0(q);
        t.seg_list[place] = s;
    }
    for (int b = tid; b < n_blocks; b += 256) {      // the last segment with blk0 <= b owns block b
        int lo = 0, hi = n_seg - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) / 2;
            if (seg_blk0[mid] <= b) lo = mid; else hi = mid - 1;
        }
        t.blk_seg[b] = lo;
        if (!in.records()) continue;
        BlkInfo bi;
        const int k = in.seg_adapter(lo);
        bi.g.row0 = in.seg_row0(lo); bi.g.row1 = in.seg_row1(lo); bi.g.adapter = k;
        bi.g.r = in.ad_rank(k); bi.g.rp = pad_to(bi.g.r, kRankPadGemm); bi.g.r16 = pad_to(bi.g.r, kRankPadMfma);
        bi.g.blk0 = seg_blk0[lo]; bi.g.lp = pad_to(bi.g.row1 - bi.g.row0, kTokPad);
        bi.g.h_off = seg_h[lo]; bi.g.hb_off = seg_hb[lo]; bi.g.zt_off = seg_zt[lo];
        bi.t0 = (b - bi.g.blk0) * kSkinnyRows;
        bi.scale = in.ad_scale(k); bi.at_off = sh.at_off[k]; bi.B = in.ad_ptr(k, 1); bi.rp_off = sh.rp_off[k]; bi.reserved = 0;
        t.blk[b] = bi;
    }
    // row tiles of the GEMMs, and the order they are walked in
    struct FromLds {
        const DescReader<WordsInMemory> &in;
        const DeriveShared &sh;
        const int64_t *hb;
        __device__ int row0(int s) const { return in.seg_row0(s); }
        __device__ int row1(int s) const { return in.seg_row1(s); }
        __device__ int adapter(int s) const { return in.seg_adapter(s); }
        __device__ int rank(int s) const { return in.ad_rank(in.seg_adapter(s)); }
        __device__ int64_t hb_off(int s) const { return hb[s]; }
        __device__ const void *ext_b(int k) const { return in.ext_b(k, sh.at_off[k]); }
        __device__ int64_t ap_off(int k) const { return sh.ap_off[k]; }
    };
    const FromLds from{in, sh, seg_hb};
    const bool sorted = !in.order_is_identity();
    int key = -1;                                    // class of this thread's latest tile
    for (int64_t i = tid; i < n_tiles; i += 256) {
        const GemmTile gt = derive_tile(from, n_seg, T, i);
        t.tile[i] = gt;
        key = sort_key(gt.n_ext);
        if (sorted) atomicAdd(&sh.totals[key], 1);
        else t.tile_order[i] = (int32_t)i;
    }
    if (!sorted) return;
    // counting sort, 256 tiles at a time: the place of a tile is the start of its class, plus the tiles of that class in
    // the earlier rounds, the earlier waves and the earlier lanes
    __syncthreads();
    if (tid < kSortKeys) {
        int b = 0;
        for (int k = kSortKeys - 1; k > tid; --k) b += sh.totals[k];
        sh.base[tid] = b;
    }
    const bool one_round = n_tiles <= 256;
    for (int64_t i0 = 0; i0 < n_tiles; i0 += 256) {
        const int64_t i = i0 + tid;
        if (!one_round) key = i < n_tiles ? sort_key(t.tile[i].n_ext) : -1;     // written by this thread above
        int before = 0;
#pragma unroll
        for (int k = 0; k < kSortKeys; ++k) {
            const uint64_t m = __ballot(key == k);
            if (key == k) before = __popcll(m & ((1ull << lane) - 1));
            if (lane == 0) sh.wave_cnt[wave][k] = __popcll(m);
        }
        __syncthreads();
        if (key >= 0) {
            int place = sh.base[key] + before;
            for (int w = 0; w < wave; ++w) place += sh.wave_cnt[w][key];
            t.tile_order[place] = (int32_t)i;
        }
        __syncthreads();
        if (tid < kSortKeys)
            for (int w = 0; w < 4; ++w) sh.base[tid] += sh.wave_cnt[w][tid];
        __syncthreads();
    }
}

// ---- the preparation kernel ----------------------------------------------------------------------
// Workgroup 0 derives the metadata tables into the workspace and clears the zero page; the next
// n_pack workgroups pack the A_k, the next n_pack_b the B_k (only when W is stored [d_out][d_in]); the
// last ones make the transposed bf16 copy of a saved activation.  The packing and copy workgroups work out the few
// offsets they need from the compact description themselves, so they do not wait for workgroup 0.
// Bound by latency: a launch, one trip to the description, a handful of workgroup-wide scans.  Per call, before (tables by
// one thread, a serial counting sort, 2-byte stores in the packing) and now: 32 adapters in 32 ragged segments 60 and 57 us
// -> 22 and 28 us (forward, backward); 16 equal segments 18 -> 10 us; 8 segments in 7 row tiles, fp32, 23 -> 9 us.
// What one description's part of a preparation launch reads and writes.
struct PrepArgs {
    char *meta_dst;
    uint32_t *zero_page;
    uint16_t *at, *ap, *zt;
    const float *hf;
    int32_t want_at, want_ap, pack_bx, n_pack, pack_bx_b, n_pack_b;
    int32_t word0, block0;        // of this description: first word of the argument, first workgroup of the launch
};
// Several descriptions in one launch (the projections of a grouped call).
constexpr int kPrepBatchWords = 768;
struct PrepBatch {
    int32_t n, pad;
    PrepArgs a[kMaxGroup];
    uint32_t w[kPrepBatchWords];
};
static_assert(sizeof(PrepBatch) <= 3584, "the batch must fit a kernel argument");

struct WordsInArg {
    const uint32_t *w;
    __device__ inline uint32_t word(int i) const { return w[i]; }
};

// The segment that owns token block blk (one lane per segment, 64 at a time), with its offsets as in the tables; t_block: the
// block's first token inside the segment.
template <class Src>
__device__ inline SegInfo segment_of_block(const DescReader<Src> &in, int blk, int &t_block, float &scale)
{
    const int n_seg = in.n_seg(), lane = threadIdx.x & 63;
    int64_t h = 0, hb = 0, zto = 0;
    int blk0 = 0;
    SegInfo g;
    g.row0 = 0; g.row1 = 0; g.adapter = -1; g.r = 0; g.rp = 0; g.r16 = 0; g.blk0 = 0; g.lp = 0; g.h_off = 0; g.hb_off = 0; g.zt_off = 0;
    t_block = 0; scale = 0.f;
    for (int s0 = 0; s0 < n_seg; s0 += 64) {
        const int s = s0 + lane;
        int len = 0, r = 0, nb = 0, row0 = 0, k = -1;
        if (s < n_seg) {
            k = in.seg_adapter(s);
            if (k >= 0) {
                row0 = in.seg_row0(s);
                len = in.seg_row1(s) - row0;
                r = in.ad_rank(k);
                nb = (len + kSkinnyRows - 1) / kSkinnyRows;
            }
        }
        const int r16 = pad_to(r, kRankPadMfma), rp = pad_to(r, kRankPadGemm), lp = pad_to(len, kTokPad);
        const int64_t he = (int64_t)len * r, be = (int64_t)len * rp, ze = (int64_t)r16 * lp;
        const int nb_inc = wave_scan(nb);
        const int64_t h_inc = wave_scan(he), b_inc = wave_scan(be), z_inc = wave_scan(ze);
        const uint64_t own = __ballot(blk < blk0 + nb_inc && blk >= blk0 + nb_inc - nb);
        if (own) {
            const int l = __builtin_ctzll(own);
            auto at = [&](int v) { return __builtin_amdgcn_readlane(v, l); };
            auto at64 = [&](int64_t v) { return (int64_t)((uint64_t)(uint32_t)at((int)(uint32_t)v) | ((uint64_t)(uint32_t)at((int)(uint32_t)((uint64_t)v >> 32)) << 32)); };
            g.row0 = at(row0); g.row1 = g.row0 + at(len); g.adapter = at(k); g.r = at(r); g.rp = at(rp); g.r16 = at(r16); g.lp = at(lp);
            g.blk0 = blk0 + at(nb_inc) - at(nb);
            t_block = (blk - g.blk0) * kSkinnyRows;
            g.h_off = h + at64(h_inc - he); g.hb_off = hb + at64(b_inc - be); g.zt_off = zto + at64(z_inc - ze);
            scale = in.ad_scale(g.adapter);
            break;
        }
        blk0 += __builtin_amdgcn_readlane(nb_inc, 63);
        h += __shfl(h_inc, 63); hb += __shfl(b_inc, 63); zto += __shfl(z_inc, 63);
    }
    return g;
}

template <class Src>
__device__ inline void prep_body(const DescReader<Src> &in, const PrepArgs &pa, int b, char *shared_mem)
{
    if (b == 0) {
        pa.zero_page[threadIdx.x] = 0u;  // kZeroBytes = 256 * 4
        derive_on_device(in, pa.meta_dst, shared_mem);
        return;
    }
    b -= 1;
    if (b < pa.n_pack) {
        const int k = b / pa.pack_bx;
        const int64_t D = in.D();
        PackJob a;
        a.A = static_cast<const uint16_t *>(in.ad_ptr(k, 0));
        a.r = in.ad_rank(k);
        a.rp = pad_to(a.r, kRankPadGemm);
        a.r16 = pad_to(a.r, kRankPadMfma);
        a.at_off = rank_rows_before(in, k, kRankPadMfma) * D;
        a.ap_off = rank_rows_before(in, k, kRankPadGemm) * D;
        pack_block(a, D, b % pa.pack_bx, pa.at, pa.ap, pa.want_at, pa.want_ap, reinterpret_cast<uint16_t *>(shared_mem));
        return;
    }
    b -= pa.n_pack;
    if (b < pa.n_pack_b) {
        const int k = b / pa.pack_bx_b;
        const int64_t K = in.K();
        PackBJob a;
        a.B = static_cast<const uint16_t *>(in.ad_ptr(k, 1));
        a.r = in.ad_rank(k);
        a.rp = pad_to(a.r, kRankPadGemm);
        a.bp_off = rank_rows_before(in, k, kRankPadGemm) * K;
        pack_bt_block(a, K, b % pa.pack_bx_b, pa.ap, reinterpret_cast<uint16_t *>(shared_mem));
        return;
    }
    b -= pa.n_pack_b;
    constexpr int kSlices = kSkinnyRows / kTrRows;
    const int blk = b / kSlices, slice = b % kSlices;
    int t_block;
    float scale;
    const SegInfo g = segment_of_block(in, blk, t_block, scale);
    h_to_zt_slice(TransposeJob{g.row1 - g.row0, g.r, g.r16, g.lp, t_block, g.h_off, g.zt_off}, slice, pa.hf, pa.zt, reinterpret_cast<float *>(shared_mem));
}

// The launch arguments of one description, its number of workgroups and the LDS they need.
inline hipError_t prep_args(const PrepJob &j, PrepArgs &pa, int64_t &n_wg, size_t &lds)
{
    static_assert(PLORA_MAX_ADAPTERS == 256, "one adapter per thread of workgroup 0");
    static_assert(kZeroBytes == 1024, "the zero page is written by one 256-thread workgroup");
    if (j.want_ap && j.want_bp) return hipErrorInvalidValue;            // both live in `ap`
    const MetaHeader &h = j.h;
    const bool pack = h.n_adapters > 0 && (j.want_at || j.want_ap);
    pa.meta_dst = j.meta_dev; pa.zero_page = static_cast<uint32_t *>(j.zero_dev);
    pa.at = static_cast<uint16_t *>(j.at); pa.ap = static_cast<uint16_t *>(j.ap);
    pa.zt = static_cast<uint16_t *>(j.zt); pa.hf = j.hf;
    pa.want_at = j.want_at ? 1 : 0; pa.want_ap = j.want_ap ? 1 : 0;
    pa.pack_bx = (int)((h.D + 63) / 64);
    pa.n_pack = pack ? pa.pack_bx * h.n_adapters : 0;
    pa.pack_bx_b = (int)((h.K + 63) / 64);
    pa.n_pack_b = (j.want_bp && h.n_adapters > 0) ? pa.pack_bx_b * h.n_adapters : 0;
    pa.word0 = 0; pa.block0 = 0;
    const int n_tr = (j.hf && j.zt) ? h.n_blocks * (kSkinnyRows / kTrRows) : 0;
    n_wg = 1 + (int64_t)pa.n_pack + pa.n_pack_b + n_tr;
    // LDS: the derivation of workgroup 0, a pack tile of 64 rows, or 64 tokens of a saved activation
    lds = derive_lds_bytes(j.n_words, h.n_seg);
    if ((pa.n_pack || pa.n_pack_b) && lds < (size_t)128 * j.max_rank) lds = (size_t)128 * j.max_rank;
    if (n_tr && lds < (size_t)256 * j.max_rank) lds = (size_t)256 * j.max_rank;
    return hipSuccess;
}

}  // namespace plora
