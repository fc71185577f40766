// Internal declarations shared by the host entry points and the HIP kernels of libplora.
// Not part of the public interface (that is include/plora.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include "plora.h"

namespace plora {

constexpr int kSkinnyRows = 128;   // token block of the shrink / dH kernel (never straddles a segment)
constexpr int kRankPadGemm = 64;   // ranks are padded to one K-step of the GEMM in the bf16 side buffers
constexpr int kRankPadMfma = 16;   // ranks are padded to one MFMA block in the skinny kernels
constexpr int kTokPad = 64;        // segment lengths are padded to this in the transposed side buffers
constexpr int kZeroBytes = 1024;   // zero page at the head of the workspace
constexpr int kTokMaxSplits = 8;    // the dA / dB kernels split the token walk over at most this many workgroups
constexpr int kSkinnyMaxSplits = 32; // the skinny kernels split the contraction over at most this many workgroups
constexpr int kGemmTileRows = 256;  // row tile of the base GEMMs
constexpr int kGemmGroupRows = 4;   // row tiles that the GEMM's tile order keeps together on one XCD (they share W columns in its L2)

// ---------------------------------------------------------------------------------------------
// Segment-packing metadata (section 2.4: which rows belong to which adapter).
//
// The host validates the description and ships it to the device in a compact form (a few 32-bit
// words per segment and adapter, passed by value as a kernel argument).  The tables the kernels
// read are derived from it on both sides: the device does it inside the preparation kernel and writes
// the tables into the workspace; the host does it to size the workspace, to plan the launches and to
// export the tables for the brute-force tests.
// ---------------------------------------------------------------------------------------------

// One entry per segment of the call (empty and base-only segments included).
struct SegInfo {
    int32_t row0, row1;   // token rows [row0, row1)
    int32_t adapter;      // -1: base weight only
    int32_t r;            // rank of the adapter (0 if none)
    int32_t rp;           // rank padded to kRankPadGemm: row pitch of the bf16 side buffer (0 if none)
    int32_t r16;          // rank padded to kRankPadMfma
    int32_t blk0;         // index of this segment's first token block (blocks of kSkinnyRows rows)
    int32_t lp;           // segment length padded to kTokPad: row pitch of the transposed side buffers
    int64_t h_off;        // element offset of the segment in the fp32 activation  [len][r]
    int64_t hb_off;       // element offset in the bf16 side buffer                [len][rp]
    int64_t zt_off;       // element offset in the transposed bf16 side buffers    [r16][lp]
};

// One entry per adapter.
struct AdapterInfo {
    const void *A;        // [d_in][r]
    const void *B;        // [r][d_out]
    float *dA;            // [d_in][r]   (backward only)
    float *dB;            // [r][d_out]  (backward only)
    int32_t r, rp, r16;
    float scale;
    int64_t at_off;       // element offset of A^T  [r16][d_in]  in the packed-A^T buffer
    int64_t ap_off;       // element offset of A    [d_in][rp]   in the padded-A buffer; with W stored [d_out][d_in]:
                          // of B^T [d_out][rp] in that same buffer
    int32_t r16_off;      // sum of r16 over the adapters before this one (row offset in dA / dB partial tiles)
    int32_t by_tokens;    // entry i: the adapter with the i-th largest token count (ties by index)
    int32_t seg_list0;    // this adapter's non-empty segments: seg_list[seg_list0 .. seg_list0 + n_own), in segment order
    int32_t n_own;
    int32_t tokens;       // tokens of this adapter over all its segments
    int32_t reserved;
    const void *ext_b;    // what GemmSeg::B is for this adapter's segments: B, or the packed A^T when W is [d_out][d_in]
};

struct MetaHeader {
    int64_t T, D, K;
    int32_t n_seg, n_adapters;
    int32_t n_blocks;     // token blocks of kSkinnyRows rows over all segments
    int32_t max_r16;      // largest rank (padded to 16) among segments with tokens
    int32_t w_out_in;     // 1: W is stored [d_out][d_in]
    int32_t reserved;
    const void *at_base;  // device address of the packed-A^T buffer (only used when w_out_in)
};

// What a 256-row tile of the base GEMMs needs to know about one segment whose low-rank term it adds.
struct GemmSeg {
    int32_t row0, row1;   // rows of the segment
    int32_t rp, r;        // padded and true rank
    int64_t hb_off;       // element offset of the segment in the bf16 low-rank factor [len][rp]
    const void *B;        // operand of the GEMM that reads W with the contraction index as row index, [r][N]:
                          // W[d_in][d_out]: forward, B_k;  W[d_out][d_in]: backward, the packed A_k^T
    int64_t ap_off;       // operand of the other GEMM, [N][rp], as element offset in the padded buffer:
                          // W[d_in][d_out]: backward, padded A_k;  W[d_out][d_in]: forward, padded B_k^T
};

// One entry per 256-row tile of the base GEMMs.  The low-rank term enters the GEMM as extra steps of
// the contraction loop, one per 64 padded rank columns of every segment with an adapter that
// overlaps the tile.  The first two such segments are spelled out, so that a tile gets all it needs
// with one fetch, issued a whole tile ahead.
struct GemmTile {
    int32_t n_ext;        // extension steps of the tile: sum of rp / 64 over the segments counted in n_own
    int32_t n_own;        // segments with an adapter and rows that overlap the tile
    int32_t first_seg;    // the first of them (n_seg if none)
    int32_t third_seg;    // the third of them (n_seg if fewer): where the walk over the segment table resumes
    GemmSeg s[2];
};

// What the skinny kernels need to know about a token block of kSkinnyRows rows: one record, so that a workgroup waits for
// one load instead of a chain of three (block -> segment -> adapter; about 1 us each, in kernels of 5 to 10 us).
struct BlkInfo {
    SegInfo g;
    int32_t t0;           // first token of the block inside its segment
    float scale;
    int64_t at_off;       // of the adapter
    const void *B;
    int32_t rp_off;       // sum of rp over the adapters before this one (rows of the padded operand, in units of its row count)
    int32_t reserved;
};

// The same for the weight-gradient kernels, one entry per adapter in the order by token count: the adapter, and the first
// of its segments (most adapters have one).
struct TokJob {
    float *dA, *dB;
    int64_t zt_off;               // first segment: its transposed factor,
    int32_t row0, len, lp;        // first row, rows, pitch of that factor
    int32_t k;                    // the adapter
    int32_t r, r16, r16_off;
    float scale;
    int32_t seg_list0, n_own, n_steps;    // n_steps: 64-token steps over all of its segments
    int32_t reserved;
};

// Device view of the derived tables (all pointers into the workspace, laid out by table_layout).
struct MetaView {
    const MetaHeader *hdr;
    const SegInfo *seg;
    const AdapterInfo *ad;
    const GemmTile *tile;     // one per 256-row tile
    const int32_t *blk_seg;   // segment of each token block of kSkinnyRows rows
    const int32_t *seg_list;  // non-empty segments grouped by adapter (see AdapterInfo)
    const int32_t *tile_order;  // the GEMM row tiles ordered by extension steps, most first (ties: lower tile first)
    const BlkInfo *blk;       // one per token block
    const TokJob *job;        // one per adapter, longest first
};

// Several projections that read the same x (q / k / v, gate / up), fused along the rank: for adapter k the fused pass
// treats the rows of the projections' small factors, each padded to 16, as one factor of sum_p r16_{k,p} <= PLORA_MAX_RANK
// rows (appendix C.2's concatenation of adapters, applied across projections).  The rows stay where each projection's
// own kernels keep them; the fused kernels gather them 8 rows at a time.  The projections share the segments, so the
// token blocks, the per-adapter segment lists and the order by token count are those of projection 0.
constexpr int kMaxGroup = PLORA_MAX_GROUP;
struct GroupView {
    int32_t n_proj;               // projections fused in this launch (>= 2)
    int32_t max_r16;              // largest fused rank among the adapters with tokens
    int32_t r16_total;            // sum of the fused ranks over all adapters (rows of the dA partial tiles)
    int32_t reserved;
    MetaView mv[kMaxGroup];       // each projection's own tables
    const uint16_t *small[kMaxGroup];   // shrink: its packed-A^T buffer;  dA: its transposed bf16 g
};
struct NoGroup { int32_t unused; };

// ---- compact description -----------------------------------------------------------------------
// 32-bit words: [0,1] T  [2,3] D  [4,5] K  [6] n_seg  [7] n_adapters  [8] n_blocks (computed by the host, fixes the
// table layout)  [9] bit 0: W is stored [d_out][d_in], bit 1: the sorted order of the GEMM row tiles is the identity (the
// host knows from its own derivation; the device then skips the sort)  [10,11] device address of the packed-A^T buffer; then per segment
// {row1, adapter}; then per adapter {A lo, A hi, B lo, B hi, dA lo, dA hi, dB lo, dB hi, r, scale bits}.
constexpr int kDescHeadWords = 12, kDescSegWords = 2, kDescAdWords = 10;
constexpr int kChunkWords = 896;   // 3584 bytes: what one launch carries by value, below the 4 KB kernel-argument limit
struct DescChunk { uint32_t w[kChunkWords]; };

#define PLORA_HD __host__ __device__ inline

PLORA_HD int desc_words(int n_seg, int n_adapters) { return kDescHeadWords + kDescSegWords * n_seg + kDescAdWords * n_adapters; }

// Where the compact description lies: word(i) returns word i.
struct WordsInMemory {
    const uint32_t *p;
    PLORA_HD uint32_t word(int i) const { return p[i]; }
};

template <class Src> struct DescReader {
    Src src;
    PLORA_HD int64_t w64(int i) const { return (int64_t)((uint64_t)src.word(i) | ((uint64_t)src.word(i + 1) << 32)); }
    PLORA_HD int64_t T() const { return w64(0); }
    PLORA_HD int64_t D() const { return w64(2); }
    PLORA_HD int64_t K() const { return w64(4); }
    PLORA_HD int n_seg() const { return (int)src.word(6); }
    PLORA_HD int n_adapters() const { return (int)src.word(7); }
    PLORA_HD int n_blocks() const { return (int)src.word(8); }
    PLORA_HD int w_out_in() const { return (int)(src.word(9) & 1u); }
    PLORA_HD int records() const { return (int)((src.word(9) >> 2) & 1u); }
    PLORA_HD int order_is_identity() const { return (int)((src.word(9) >> 1) & 1u); }
    PLORA_HD const void *at_base() const { return reinterpret_cast<const void *>((uintptr_t)w64(10)); }
    PLORA_HD int seg_row1(int s) const { return (int)src.word(kDescHeadWords + kDescSegWords * s); }
    PLORA_HD int seg_row0(int s) const { return s ? seg_row1(s - 1) : 0; }
    PLORA_HD int seg_adapter(int s) const { return (int)src.word(kDescHeadWords + kDescSegWords * s + 1); }
    PLORA_HD int ad_base(int k) const { return kDescHeadWords + kDescSegWords * n_seg() + kDescAdWords * k; }
    PLORA_HD const void *ad_ptr(int k, int which) const { return reinterpret_cast<const void *>((uintptr_t)w64(ad_base(k) + 2 * which)); }
    // operand of the GEMM form with the contraction index as row index (GemmSeg::B) of adapter k, whose packed A^T starts
    // at element at_off (integer arithmetic: the host derives the tables with a null base)
    PLORA_HD const void *ext_b(int k, int64_t at_off) const
    {
        return w_out_in() ? reinterpret_cast<const void *>((uintptr_t)at_base() + 2 * (uintptr_t)at_off) : ad_ptr(k, 1);
    }
    PLORA_HD int ad_rank(int k) const { return (int)src.word(ad_base(k) + 8); }
    PLORA_HD float ad_scale(int k) const
    {
        union { uint32_t u; float f; } c;
        c.u = src.word(ad_base(k) + 9);
        return c.f;
    }
};

PLORA_HD int32_t pad_to(int32_t v, int32_t a) { return (v + a - 1) / a * a; }
PLORA_HD size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Byte offsets of the derived tables inside the metadata region of the workspace.
struct TableLayout {
    size_t hdr, seg, ad, tile, blk_seg, seg_list, tile_order, blk, job, bytes;
    int64_t n_tiles;
};

PLORA_HD TableLayout table_layout(int64_t T, int n_seg, int n_adapters, int n_blocks, bool records)
{
    TableLayout l;
    size_t o = 0;
    l.n_tiles = (T + kGemmTileRows - 1) / kGemmTileRows;
    l.hdr = o;      o = align_up(o + sizeof(MetaHeader), 64);
    l.seg = o;      o = align_up(o + (size_t)n_seg * sizeof(SegInfo), 64);
    l.ad = o;       o = align_up(o + (size_t)n_adapters * sizeof(AdapterInfo), 64);
    l.tile = o;     o = align_up(o + (size_t)l.n_tiles * sizeof(GemmTile), 64);
    l.blk_seg = o;  o = align_up(o + (size_t)n_blocks * sizeof(int32_t), 64);
    l.seg_list = o; o = align_up(o + (size_t)n_seg * sizeof(int32_t), 64);
    l.tile_order = o; o = align_up(o + (size_t)l.n_tiles * sizeof(int32_t), 64);
    l.blk = o;      o = align_up(o + (records ? (size_t)n_blocks * sizeof(BlkInfo) : 0), 64);
    l.job = o;      o = align_up(o + (records ? (size_t)n_adapters * sizeof(TokJob) : 0), 64);
    l.bytes = o;
    return l;
}

// Mutable pointers to the tables (a host buffer or the workspace).
struct Tables {
    MetaHeader *hdr;
    SegInfo *seg;
    AdapterInfo *ad;
    GemmTile *tile;
    int32_t *blk_seg;
    int32_t *seg_list;
    int32_t *tile_order;
    BlkInfo *blk;
    TokJob *job;
};

PLORA_HD Tables tables_at(char *base, const TableLayout &l)
{
    Tables t;
    t.hdr = reinterpret_cast<MetaHeader *>(base + l.hdr);
    t.seg = reinterpret_cast<SegInfo *>(base + l.seg);
    t.ad = reinterpret_cast<AdapterInfo *>(base + l.ad);
    t.tile = reinterpret_cast<GemmTile *>(base + l.tile);
    t.blk_seg = reinterpret_cast<int32_t *>(base + l.blk_seg);
    t.seg_list = reinterpret_cast<int32_t *>(base + l.seg_list);
    t.tile_order = reinterpret_cast<int32_t *>(base + l.tile_order);
    t.blk = reinterpret_cast<BlkInfo *>(base + l.blk);
    t.job = reinterpret_cast<TokJob *>(base + l.job);
    return t;
}

PLORA_HD MetaView view_of(const Tables &t)
{
    MetaView v;
    v.hdr = t.hdr; v.seg = t.seg; v.ad = t.ad; v.tile = t.tile; v.blk_seg = t.blk_seg; v.seg_list = t.seg_list; v.tile_order = t.tile_order;
    v.blk = t.blk; v.job = t.job;
    return v;
}

// ---- derivation of the tables ------------------------------------------------------------------------
// The host walks segments and adapters one after the other (derive_tables); the preparation kernel derives the same
// tables in parallel (small_kernels.hip) and a test compares the two byte for byte.  The record of a row tile is built by
// one routine for both (derive_tile).

PLORA_HD bool seg_has_lowrank(const SegInfo &g) { return g.adapter >= 0 && g.row1 > g.row0; }

// Extension steps and the first segments of one GEMM row tile.  in: row0(s), row1(s), adapter(s), rank(s) and hb_off(s) of a
// segment, ext_b(k) and ap_off(k) of an adapter.
template <class In> PLORA_HD GemmTile derive_tile(const In &in, int n_seg, int64_t T, int64_t tile)
{
    const int64_t m0 = tile * kGemmTileRows;
    const int64_t m1 = m0 + kGemmTileRows < T ? m0 + kGemmTileRows : T;
    int lo = 0, hi = n_seg;                     // first segment with row1 > m0
    while (lo < hi) {
        const int mid = (lo + hi) / 2;
        if (in.row1(mid) > m0) hi = mid; else lo = mid + 1;
    }
    GemmTile gt;
    gt.n_ext = 0; gt.n_own = 0; gt.first_seg = n_seg; gt.third_seg = n_seg;
    for (int i = 0; i < 2; ++i) {
        gt.s[i].row0 = 0; gt.s[i].row1 = 0; gt.s[i].rp = 0; gt.s[i].r = 0;
        gt.s[i].hb_off = 0; gt.s[i].B = nullptr; gt.s[i].ap_off = 0;
    }
    for (int s = lo; s < n_seg && in.row0(s) < m1; ++s) {
        const int k = in.adapter(s);
        if (k < 0 || in.row1(s) <= in.row0(s)) continue;
        const int r = in.rank(s);
        if (gt.n_own < 2) {
            GemmSeg q;
            q.row0 = in.row0(s); q.row1 = in.row1(s); q.rp = pad_to(r, kRankPadGemm); q.r = r; q.hb_off = in.hb_off(s);
            q.B = in.ext_b(k); q.ap_off = in.ap_off(k);
            if (gt.n_own == 0) { gt.s[0] = q; gt.first_seg = s; }     // (no indexed access: the record stays in registers)
            else gt.s[1] = q;
        } else if (gt.n_own == 2) {
            gt.third_seg = s;
        }
        gt.n_own += 1;
        gt.n_ext += pad_to(r, kRankPadGemm) / kRankPadGemm;
    }
    return gt;
}

// The order in which the GEMMs walk their row tiles.  Workgroups that run side by side on one XCD work on a group of
// kGemmGroupRows consecutive entries of this order and share the columns of W they stream; they only stay in step if
// their tiles have the same number of contraction steps, so the row tiles are sorted by their extension steps, most
// first, tiles of equal length in row order (lengths of kSortKeys - 1 steps and more count as one class).
constexpr int kSortKeys = 9;

PLORA_HD int sort_key(int32_t n_ext) { return n_ext < kSortKeys - 1 ? n_ext : kSortKeys - 1; }

// The host's derivation.  tokens: scratch, two ints per adapter.
template <class Src> inline void derive_tables(const DescReader<Src> &in, const Tables &t, int32_t *tokens)
{
    const int n_seg = in.n_seg(), n_ad = in.n_adapters();
    const int64_t D = in.D(), T = in.T();
    const int64_t ap_rows = in.w_out_in() ? in.K() : D;   // rows of the padded operand [rows][rp], see GemmSeg
    int32_t *cursor = tokens + n_ad;
    for (int k = 0; k < n_ad; ++k) { tokens[k] = 0; cursor[k] = 0; t.ad[k].n_own = 0; }
    int64_t h = 0, hb = 0, zt = 0;
    int32_t blk = 0, max_r16 = 0;
    for (int s = 0; s < n_seg; ++s) {
        SegInfo g;
        g.row0 = in.seg_row0(s); g.row1 = in.seg_row1(s);
        g.adapter = in.seg_adapter(s);
        const int32_t len = g.row1 - g.row0;
        g.r = g.adapter >= 0 ? in.ad_rank(g.adapter) : 0;
        g.rp = pad_to(g.r, kRankPadGemm);
        g.r16 = pad_to(g.r, kRankPadMfma);
        g.lp = pad_to(len, kTokPad);
        g.blk0 = blk;
        g.h_off = h; g.hb_off = hb; g.zt_off = zt;
        if (g.adapter >= 0) {
            const int32_t nb = (len + kSkinnyRows - 1) / kSkinnyRows;
            for (int32_t b = 0; b < nb; ++b) t.blk_seg[blk + b] = s;
            blk += nb;
            if (len > 0 && g.r16 > max_r16) max_r16 = g.r16;
            h += (int64_t)len * g.r;
            hb += (int64_t)len * g.rp;
            zt += (int64_t)g.r16 * g.lp;
            tokens[g.adapter] += len;
            t.ad[g.adapter].n_own += len > 0;
        }
        t.seg[s] = g;
    }
    int64_t at = 0, ap = 0;
    int32_t r16_off = 0, list0 = 0;
    for (int k = 0; k < n_ad; ++k) {
        AdapterInfo a;
        a.A = in.ad_ptr(k, 0);
        a.B = in.ad_ptr(k, 1);
        a.dA = static_cast<float *>(const_cast<void *>(in.ad_ptr(k, 2)));
        a.dB = static_cast<float *>(const_cast<void *>(in.ad_ptr(k, 3)));
        a.r = in.ad_rank(k);
        a.rp = pad_to(a.r, kRankPadGemm);
        a.r16 = pad_to(a.r, kRankPadMfma);
        a.scale = in.ad_scale(k);
        a.at_off = at; at += (int64_t)a.r16 * D;
        a.ext_b = in.ext_b(k, a.at_off);
        a.ap_off = ap; ap += (int64_t)a.rp * ap_rows;
        a.r16_off = r16_off; r16_off += a.r16;
        a.by_tokens = 0;                    // filled in below
        a.seg_list0 = list0; a.n_own = t.ad[k].n_own; a.tokens = tokens[k]; a.reserved = 0;
        cursor[k] = list0;
        list0 += a.n_own;
        t.ad[k] = a;
    }
    // per-adapter lists of non-empty segments, in segment order
    for (int s = 0; s < n_seg; ++s)
        if (seg_has_lowrank(t.seg[s])) t.seg_list[cursor[t.seg[s].adapter]++] = s;
    // place of each adapter in the order by token count, longest first (the weight-gradient kernels hand out
    // adapters in that order, so the last workgroups are short)
    for (int k = 0; k < n_ad; ++k) {
        int rank = 0;
        for (int j = 0; j < n_ad; ++j) rank += tokens[j] > tokens[k] || (tokens[j] == tokens[k] && j < k);
        t.ad[rank].by_tokens = k;
    }
    for (int s = 0; s < n_seg && in.records(); ++s) {
        const SegInfo &g = t.seg[s];
        if (!seg_has_lowrank(g)) continue;
        const AdapterInfo &a = t.ad[g.adapter];
        for (int32_t t0 = 0, b = g.blk0; t0 < g.row1 - g.row0; t0 += kSkinnyRows, ++b)
            t.blk[b] = BlkInfo{g, t0, a.scale, a.at_off, a.B, (int32_t)(a.ap_off / ap_rows), 0};
    }
    for (int i = 0; i < n_ad && in.records(); ++i) {
        const int k = t.ad[i].by_tokens;
        const AdapterInfo &a = t.ad[k];
        TokJob j{a.dA, a.dB, 0, 0, 0, 0, k, a.r, a.r16, a.r16_off, a.scale, a.seg_list0, a.n_own, 0, 0};
        for (int li = 0; li < a.n_own; ++li) {
            const SegInfo &g = t.seg[t.seg_list[a.seg_list0 + li]];
            if (li == 0) { j.zt_off = g.zt_off; j.row0 = g.row0; j.len = g.row1 - g.row0; j.lp = g.lp; }
            j.n_steps += g.lp / kTokPad;
        }
        t.job[i] = j;
    }
    MetaHeader hd;
    hd.T = T; hd.D = D; hd.K = in.K();
    hd.n_seg = n_seg; hd.n_adapters = n_ad; hd.n_blocks = blk; hd.max_r16 = max_r16;
    hd.w_out_in = in.w_out_in(); hd.reserved = 0; hd.at_base = in.at_base();
    *t.hdr = hd;
    struct FromTables {
        const Tables &t;
        int row0(int s) const { return t.seg[s].row0; }
        int row1(int s) const { return t.seg[s].row1; }
        int adapter(int s) const { return t.seg[s].adapter; }
        int rank(int s) const { return t.seg[s].r; }
        int64_t hb_off(int s) const { return t.seg[s].hb_off; }
        const void *ext_b(int k) const { return t.ad[k].ext_b; }
        int64_t ap_off(int k) const { return t.ad[k].ap_off; }
    };
    const FromTables from{t};
    const int64_t n_tiles = (T + kGemmTileRows - 1) / kGemmTileRows;
    int32_t start[kSortKeys + 1];
    for (int k = 0; k <= kSortKeys; ++k) start[k] = 0;
    for (int64_t i = 0; i < n_tiles; ++i) {
        t.tile[i] = derive_tile(from, n_seg, T, i);
        start[sort_key(t.tile[i].n_ext)] += 1;
    }
    for (int k = kSortKeys - 1, base = 0; k >= 0; --k) { const int n = start[k]; start[k] = base; base += n; }
    for (int64_t i = 0; i < n_tiles; ++i) t.tile_order[start[sort_key(t.tile[i].n_ext)]++] = (int32_t)i;
}

// Byte offsets of the workspace regions, each 256-byte aligned.
struct WorkspaceLayout {
    size_t zero, meta, desc, flags, at, ap, hb, zt_h, zt_g, hf, gf, part, wpart, gpart, total;
    size_t meta_bytes;
};

// ---- launch wrappers implemented in the kernel files; all enqueue on `st` and return the HIP status ----

// Compute units of the current device (thread-safe, looked up once per device); 0 with *err set on failure.
int device_cu_count(hipError_t *err);
// Lets `kernel` use up to the 160 KB of LDS of a compute unit; done once per device and kernel (slot: a small
// index that is unique per kernel), thread-safe.
hipError_t allow_full_lds(const void *kernel, int slot);
constexpr int kLdsSlots = 56;

// Metadata and the small jobs in front of the heavy kernels, in one launch when the compact description fits a
// kernel argument (otherwise it is first uploaded in chunks to desc_stage): derived tables and zero page into the
// workspace; packing of A_k (bf16 path: A_k^T [r16][d_in] with zero rows beyond r, and / or A_k padded to rp
// columns); transposed bf16 copy of a saved activation, zt[j][t] = bf16(h[t][j]) (bf16 backward).
// want_bp (instead of want_ap, W stored [d_out][d_in]): B_k^T [d_out][rp] with zero columns beyond r into `ap`.
// A grouped call prepares its projections in one launch when their descriptions fit one kernel argument together.
// An NF4 weight to expand in the same launch (the two do not depend on each other).
struct Nf4Job {
    const uint32_t *codes;
    const float *absmax;
    void *out;
    int64_t n_elems;
};
int nf4_workgroups(int64_t n_elems);      // 0: no device

// bf16 path -------------------------------------------------------------------------------------
// Skinny product over token blocks: acc[t][j] = sum_c S[t][c] * Bm_k[j][c]  (c < C).
//   mode 0 (shrink): S = x (C = d_in), Bm_k = packed A_k^T;  mode 1 (dH): S = dy (C = d_out), Bm_k = B_k.
//   Several products in one launch (shrink and dH of a call, dH of the projections of a group: same segments, same adapters).
//   `part` receives the fp32 partial tiles of up to n_split contraction splits (skinny_splits; short batches take what suits
//   them, at most this), summed by a finishing launch or the last workgroup of a slice, which writes (each optional): hf
//   fp32 [len][r] (unscaled in mode 0); hb bf16 [len][rp] = scale_k*acc; zt bf16 [r16][lp] transposed, = (zt_scaled ? scale_k : 1) * acc.
struct SkinnyOperands {
    MetaView mv;
    MetaHeader h;
    int mode;
    const void *S;
    int64_t C;
    const void *at;
    float *part;
    int n_split;
    unsigned long long *flags;    // short products: kShortSlices * kShortMaxSplits per token block
    int slices16;                 // 16-token slices with tokens, over all segments
    float *hf;
    void *hb, *zt;
    bool zt_scaled, is_short;     // is_short: skinny_short.h
    bool alone;                   // of a stand-alone low-rank call: no base product reads S afterwards
    int mean_r16;                 // rank rows that a token reads on average
};
hipError_t launch_skinny_bf16(const SkinnyOperands *ops, int n, const void *zero, hipStream_t st);
// Whether a product takes the routine for short batches (skinny_short.h; such products of a grouped call are not fused).
bool skinny_is_short(const MetaHeader &h, int slices16, int r16_total, int64_t C);
struct ShortShares { int n, per; };       // workgroups that a slice's contraction is dealt to, chunks of 64 for each
ShortShares short_shares(const MetaHeader &h, int slices16, int64_t C, int most);
struct SkinnyOut {                // where the sums go, see above
    float *hf;
    uint16_t *hb, *zt;
    int32_t zt_scaled;
};
constexpr int kShortSlices = kSkinnyRows / 16, kShortMaxSplits = 16, kShortMaxBlocks = 64;
struct ShortJob {
    const BlkInfo *blk;
    const uint16_t *S, *small;    // small: packed A_k^T (mode 0, unless A_k is read as it is)
    float *part;
    unsigned long long *flags, number;
    SkinnyOut out;
    int32_t C, mode, per, n_split, max_r16;      // per: chunks of 64 per split
    int32_t wg0;                  // first workgroup, where the job shares a launch with the preparation
};
ShortJob short_job(const SkinnyOperands &o);
unsigned long long launch_number();       // never twice the same in a process, never 0
struct F32LowRank {               // one low-rank product: mode 0 h = x A_k, mode 1 g = scale_k dy B_k^T
    const float *S;
    float *out;
    int64_t C;
    int32_t mode;
};
struct PrepJob {
    const uint32_t *desc_host;    // the compact description
    int n_words, max_rank;        // max_rank: over all adapters
    MetaHeader h;
    char *meta_dev;
    uint32_t *desc_stage;
    void *zero_dev, *at, *ap;
    bool want_at, want_ap, want_bp;
    const float *hf;
    void *zt;
    const SkinnyOperands *brief;  // short products to run in the same launch (A_k read as it is); n_brief of them, at most kPrepShort
    int n_brief;
    const F32LowRank *f32;        // the same of the fp32 path
    int n_f32;
    const SkinnyOperands *dh;     // a dH that is not short, in the same launch and with its finishing launch behind it; or null
};
constexpr int kPrepShort = 2;
hipError_t launch_prep(const PrepJob *jobs, int n_jobs, hipStream_t st);
hipError_t launch_prep_dh(const PrepJob &job, hipStream_t st);
hipError_t launch_prep_nf4(const PrepJob &job, const Nf4Job &w, bool bf16, hipStream_t st);

// C[T][N] = S[T][Kd] * Wop + side[T][rp] * ext_k, rounded to bf16.
//   w_rows_contract : Wop = W [Kd][N] (contraction index is the row index),  ext_k = GemmSeg::B   [r][N]
//   otherwise       : Wop = W [N][Kd] (contraction index is contiguous),     ext_k = ap + GemmSeg::ap_off [N][rp]
//   W[d_in][d_out]: forward (S = x, Kd = d_in, N = d_out) is the first form, backward (S = dy, Kd = d_out, N = d_in)
//   the second; W[d_out][d_in]: the other way round.
//   row_tiles: how many row tiles to compute, in the order of the tile_order table
//   accumulate: C += the product (C is read in the epilogue and the sum rounded once more), otherwise C is overwritten
//   n_split > 1 (all row tiles): the contraction in that many parts, fp32 partial tiles [n_split][T][N] in part, then summed
hipError_t launch_gemm_bf16(const MetaView &mv, const MetaHeader &h, bool w_rows_contract, int64_t Kd, int64_t N,
                            const void *S, const void *W, const void *side, const void *ap, const void *zero, void *C,
                            bool accumulate, int row_tiles, float *part, int n_split, hipStream_t st);
// C = (accumulate: C +) the sum of n_split fp32 partial tiles [n_split][n] in order, rounded once.
hipError_t launch_gemm_finish(const float *part, void *C, int64_t n, int n_split, bool accumulate, hipStream_t st);
constexpr int64_t kLastCacheBytes = 256 << 20;     // shared by the XCDs of an MI355X
// Rows of a bf16 matrix begin and end on lines of 128 bytes: pieces of 64 columns that different workgroups or stages read share none.
inline bool rows_of_whole_lines(const void *p, int64_t columns)
{
    return columns % 64 == 0 && reinterpret_cast<uintptr_t>(p) % 128 == 0;
}
// The same product in small tiles with the contraction split over workgroups (gemm_small_bf16.hip).
struct GemmPlan {
    int bm;                   // rows of the output tile: 0: k_gemm's 256 x 256 tiles, otherwise tiles of bm x 128
    int n_split;              // splits of the contraction; above 1 the fp32 partial tiles take n_split * T * N * 4 bytes
    int big_tiles;            // row tiles that k_gemm computes (all of them when bm is 0); the small tiles compute the rest
};
struct GemmShape {
    int64_t T, Kd, N;
    bool w_rows_contract;     // as in launch_gemm_bf16
    bool w_cached;            // W has just been written, so that the last-level cache holds what fits of it
    bool short_shrink;        // behind a short shrink: small tiles may be part of a forward in two launches
    int max_ext;              // most extension steps of a 256-row tile
};
constexpr double kMaxSplitBytes = 64e6;       // fp32 partial tiles of a split product
// big_split_bytes: room for the partial tiles of split 256 x 256 tiles
GemmPlan gemm_plan(const GemmShape &s, double big_split_bytes = kMaxSplitBytes);
// Whether a base product with this plan can be part of a forward in two launches (gemm_short_bf16.hip): in small tiles alone that are
// split anyway, or whose one set of fp32 sums costs less than the launch saved (build_meta has the figures).
inline bool product_in_two_launches(const GemmPlan &p, int64_t T, int64_t N)
{
    return p.bm != 0 && p.big_tiles == 0 && (p.n_split > 1 || T * N <= 2250000);
}
hipError_t launch_gemm_small_bf16(const GemmPlan &p, const MetaView &mv, const MetaHeader &h, bool w_rows_contract, int64_t Kd, int64_t N,
                                  const void *S, const void *W, const void *side, const void *ap, const void *zero, void *C,
                                  bool accumulate, float *part, hipStream_t st);
// The forward of a short batch whose base product is split in small tiles, in two launches (gemm_short_bf16.hip).
struct ShortForward {
    const uint32_t *desc_host;
    int n_words;
    MetaHeader h;
    char *meta_dev;
    void *zero_dev;
    const void *x, *W;
    void *y;
    float *hf;                // h to keep, or null
    float *h_part, *y_part;   // [shares.n][slices][16][max_r16], [plan.n_split][T][K]
    int slices;               // of 16 tokens, over all segments
    ShortShares shares;
    GemmPlan plan;
};
hipError_t launch_short_forward(const ShortForward *ops, int n, hipStream_t st);      // one call, or projections of a group
// Stand-alone low-rank update C[T][N] += side * op_k (bf16, one rounding): side = bf16 low-rank factor [len][rp] per
// segment, opT = padded small matrices [N][rp], one behind the other.
hipError_t launch_expand_bf16(const MetaView &mv, const MetaHeader &h, void *C, int64_t N, const void *side, const void *opT,
                              const void *zero, hipStream_t st);
// Token contractions: out_k = mult * sum_t S[t][c] * zt[j][t] over all segments of adapter k, several products in one launch
// (dB and dA of a call; of every projection of a grouped call: their adapters and segments are the same).
//   want_dA: S = x, out = dA_k[c][j], mult = 1;  else S = dy, out = dB_k[j][c], mult = scale_k.
//   n_split > 1: the token walk is split, partial tiles go through `part` ([split][r16_total][C] fp32).
struct TokcOperands {
    MetaView mv;
    const void *S, *zt;
    int64_t C;
    float *part;
    int n_split, r16_total, max_r16;
    bool want_dA;
    int64_t T;
};
constexpr int kTokMaxPasses = 2 * kMaxGroup;
// dx: the dX product in small tiles, in the same launches; its fp32 partial tiles lie apart from those of the ops.
struct GradsDx {
    MetaView mv;
    MetaHeader h;
    GemmPlan plan;            // small tiles alone
    bool w_rows_contract;
    int64_t Kd, N;
    const void *S, *W, *side, *ap, *zero;
    void *C;
    float *part;
};
hipError_t launch_tokcontract_bf16(const TokcOperands *ops, int n, int n_adapters, const void *zero, const GradsDx *dx, hipStream_t st);
// The same two passes for several projections at once (see GroupView).  hv: projection 0's header with max_r16 replaced
// by the fused one.  Shrink: hf / hb / zt per projection as in launch_skinny_bf16 (mode 0);
// n_split: that of the projections' plain calls.  dA: the results go to each
// projection's own dA_k; n_split must be tokc_splits(hv, C, 0, n_active_adapters).
// part_bytes: size of `part`; a pass whose partial tiles do not fit is refused.
hipError_t launch_skinny_group(const GroupView &gv, const MetaHeader &hv, const void *x, int64_t C, const void *zero, float *part,
                               size_t part_bytes, int n_split, float *const *hf, void *const *hb, void *const *zt, hipStream_t st);
hipError_t launch_tokc_group_dA(const GroupView &gv, const MetaHeader &hv, const void *x, int64_t C, const void *zero,
                                float *part, size_t part_bytes, int n_split, int n_active_adapters, hipStream_t st);
// C_other: columns of the product that shares the launch (0: none).
int tokc_splits(const MetaHeader &h, int64_t C, int64_t C_other, int n_active_adapters);
constexpr int kTokTileColumns = 128;
int skinny_splits(const MetaHeader &h, int64_t C);

// fp32 path (fp64 accumulation) ---------------------------------------------------------------------
hipError_t launch_f32_lowrank(const MetaView &mv, const MetaHeader &h, int mode, const float *S, int64_t C,
                              float *out, hipStream_t st);
hipError_t launch_f32_gemm(const MetaView &mv, const MetaHeader &h, bool forward, const float *S, const float *W,
                           const float *side, float *C, bool accumulate, hipStream_t st);   // W's layout: h.w_out_in
// to_y: y += scale_k h B_k (side = h);  else dx += g A_k^T (side = g, which carries scale_k).
hipError_t launch_f32_expand(const MetaView &mv, const MetaHeader &h, bool to_y, float *C, const float *side, hipStream_t st);
// Both weight gradients: dB from dy and h, dA from x and g (which carries scale_k).  max_rank: over all adapters.
hipError_t launch_f32_wgrad(const MetaView &mv, const MetaHeader &h, int max_rank, const float *x, const float *gf, const float *dy,
                            const float *hf, hipStream_t st);
// The same and dx = dy W^T + g A_k^T in one launch, where that fits one (f32_bwd_fits).
bool f32_bwd_fits(const MetaHeader &h, int max_rank);
hipError_t launch_f32_bwd(const MetaView &mv, const MetaHeader &h, int max_rank, const float *x, const float *gf, const float *dy,
                          const float *hf, const float *W, float *dx, hipStream_t st);

// NF4 base weight: out[i] = level[index_i] * absmax[i / 64] for n_elems elements (a multiple of 64), bf16 or fp32.
hipError_t launch_nf4_dequant(const void *codes, const float *absmax, int64_t n_elems, bool bf16, void *out, hipStream_t st);

// optimizer ----------------------------------------------------------------------------------------
struct AdamwTensor {
    void *param; float *master; const float *grad; float *m, *v;
    uint64_t numel;
    float lr, beta1, beta2, eps, weight_decay;
    int32_t step;
    float grad_scale;
};
// AdamW step of n tensors (any sizes, each with its own hyperparameters); bf16 tells the type of `param`.
hipError_t launch_adamw(const AdamwTensor *t, int n, bool bf16, hipStream_t st);

}  // namespace plora
